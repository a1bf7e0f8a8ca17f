// How the planner carries out a layer on the kernel of small layers: reads lines "B T din dout dtype mode" (mode 7: identity and square
// together), prints "small_kw nsplit" (small_kw 0: not on that kernel).
#include <cstdio>

#include "pex_internal.h"

int main()
{
    long long B, T, din, dout;
    int dt, mode;
    while (scanf("%lld %lld %lld %lld %d %d", &B, &T, &din, &dout, &dt, &mode) == 6) {
        const pex::StatPlan p = pex::plan_stat(B, T, din, dout, (pex_dtype)dt, mode == 7 ? pex::MODE_SQUARE : (pex::Mode)mode, mode != 7);
        printf("%d %d\n", p.small_kw, p.nsplit);
    }
    return 0;
}
