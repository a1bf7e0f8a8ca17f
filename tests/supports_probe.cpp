// Which layers the kernel of small layers takes at all, whatever the planner weighs: reads lines "T din dout dtype mode", prints 0 or 1.
#include <cstdio>

#include "pex_internal.h"

int main()
{
    long long T, din, dout;
    int dt, mode;
    while (scanf("%lld %lld %lld %d %d", &T, &din, &dout, &dt, &mode) == 5) printf("%d\n", (int)pex::small_supports(T, din, dout, (pex_dtype)dt, (pex::Mode)mode));
    return 0;
}
