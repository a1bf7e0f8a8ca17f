// Whether the planner runs an fp32 layer on the bf16 matrix cores if the kernel of small layers does not take it: reads lines "B T din dout mode pair", prints 0 or 1.
#include <cstdio>

#include "pex_internal.h"

int main()
{
    long long B, T, din, dout;
    int mode, pair;
    while (scanf("%lld %lld %lld %lld %d %d", &B, &T, &din, &dout, &mode, &pair) == 6)
        printf("%d\n", (int)pex::plan_stat(B, T, din, dout, PEX_F32, (pex::Mode)mode, !pair, true, false).f32_split);
    return 0;
}
