// How the planner carries out several statistics at once, for tests on a host without a GPU: reads lines "B T din dout dtype want", prints
// "examples nsplit per_split query plain small within odd" (examples: the M_b go through the workspace; the groups of the shared contraction; the bytes the
// call asks for, and asks for without any M_b; whether it is the kernel of small layers; the bytes of the plan of a call that has `plain` of them, and of
// one that has `query` at an address that is no multiple of 16).
#include <cstdio>

#include "pex_internal.h"

int main()
{
    long long B, T, din, dout;
    int dt;
    unsigned want;
    while (scanf("%lld %lld %lld %lld %d %u", &B, &T, &din, &dout, &dt, &want) == 6) {
        const pex::MultiPlan p = pex::plan_multi(B, T, din, dout, (pex_dtype)dt, want), plain = pex::plan_multi(B, T, din, dout, (pex_dtype)dt, want, true, true, false);
        const pex::MultiPlan within = pex::plan_multi_within(B, T, din, dout, (pex_dtype)dt, want, (void*)256, plain.query_bytes);
        const pex::MultiPlan odd = pex::plan_multi_within(B, T, din, dout, (pex_dtype)dt, want, (void*)264, p.query_bytes);
        printf("%d %d %lld %zu %zu %d %zu %zu\n", (int)p.examples, p.pair_plan.nsplit, (long long)p.pair_plan.per_split, p.query_bytes, plain.query_bytes,
               (int)(p.pair_plan.small_kw > 0), within.query_bytes, odd.query_bytes);
    }
    return 0;
}
