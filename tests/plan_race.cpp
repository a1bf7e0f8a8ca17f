// One host thread plans while another one changes an option: afterwards every kept plan must be the one a fresh thread makes
// under the same option.  Prints the number of plans that are not.
#include <atomic>
#include <cstdio>
#include <thread>

#include "pex_internal.h"

int main()
{
    std::atomic<bool> toggle{false}, idle{true}, stop{false};
    std::thread other([&] {
        while (!stop) {
            if (!toggle) { idle = true; continue; }
            idle = false;
            pex_set_option(PEX_OPT_MAX_SPLIT, 1);
            pex_set_option(PEX_OPT_MAX_SPLIT, 32);
        }
    });
    int wrong = 0;
    for (int k = 0; k < 2000; ++k) {
        const int64_t B = 64 + k;
        auto plan = [&] { return pex::plan_stat(B, 512, 768, 768, PEX_BF16, pex::MODE_SQUARE); };
        toggle = true;
        while (idle) {}
        plan();
        toggle = false;
        while (!idle) {}
        for (int split = 1; split <= 32; split += 31) {
            pex_set_option(PEX_OPT_MAX_SPLIT, split);
            const pex::StatPlan kept = plan();
            pex::StatPlan fresh;
            std::thread([&] { fresh = plan(); }).join();
            wrong += kept.nsplit != fresh.nsplit || kept.ws_bytes != fresh.ws_bytes;
        }
    }
    stop = true;
    other.join();
    printf("%d\n", wrong);
    return 0;
}
