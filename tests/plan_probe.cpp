// What the planner decides, for tests on a host without a GPU: reads lines "B T din dout dtype mode", prints
// "kernel nsplit per_split blocks threads" (blocks of one group; dtype 0 = fp32, 1 = bf16; mode = pex::Mode).
#include <cstdio>

#include "pex_internal.h"

int main()
{
    long long B, T, din, dout;
    int dt, mode;
    while (scanf("%lld %lld %lld %lld %d %d", &B, &T, &din, &dout, &dt, &mode) == 6) {
        const pex::StatPlan p = pex::plan_stat(B, T, din, dout, (pex_dtype)dt, (pex::Mode)mode);
        int bm = 64, bn = 64, threads = 256;
        if (p.kernel == 1) { pex::bf16_tile_shape((pex::Mode)mode, B, &bm, &bn); threads = 512; }
        if (p.kernel == 2) { pex::f32_tile_shape(p.din, p.dout, &bm, &bn); threads = bm / 64 * (bn / 64) * 64; }
        printf("%d %d %lld %lld %d\n", p.kernel, p.nsplit, (long long)p.per_split, (long long)((p.din + bm - 1) / bm * ((p.dout + bn - 1) / bn)), threads);
    }
    return 0;
}
