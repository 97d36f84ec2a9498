// csrc/until_done.h: a preparation that fails is tried again by the next
// caller, one that succeeded is not repeated, and callers in several threads
// return only once it is done.
#include <stdio.h>

#include <atomic>
#include <thread>
#include <vector>

#include "../../paper_2509_02840_amd/csrc/until_done.h"

enum Status { kOk = 0, kNoMemory = 2 };

int main()
{
    bdu::UntilDone once;
    int calls = 0;
    auto prepare = [&] { return ++calls < 3 ? kNoMemory : kOk; };
    const bool first = once(prepare) == kNoMemory && once(prepare) == kNoMemory;
    const bool then = once(prepare) == kOk && once(prepare) == kOk && calls == 3;
    bdu::UntilDone shared;
    std::atomic<int> runs{0}, late{0};
    int made = 0;
    std::vector<std::thread> v;
    for (int k = 0; k < 8; ++k)
        v.emplace_back([&] {
            if (shared([&] { ++runs; made = 1; return kOk; }) != kOk || made != 1) ++late;
        });
    for (auto &t : v) t.join();
    const bool ok = first && then && runs == 1 && late == 0;
    printf("until done: %s\n", ok ? "all checks passed" : "failed");
    return ok ? 0 : 1;
}
