// Host model of how the workgroups of a grouped GEMM come to their work items, on the arithmetic of csrc/hand_out.h.
#define __host__
#define __device__
#include <stdint.h>

#include <condition_variable>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#include "hand_out.h"

using namespace moe::gg;

namespace {

enum { kOwn, kLook, kTake, kItem, kEnd };
struct Workgroup {
    int xcd, member, state, item, from;
};

// One step of a workgroup, at most one access to the counters in each (the kernel's settle_claim()).
template <bool OWN>
void step(Workgroup& w, const HandOut<OWN>& hand, int (&counter)[kXcds], bool steal, int* done, int stride, int& accesses) {
    if (w.state != kItem) ++accesses;
    switch (w.state) {
        case kItem:
            ++done[w.from * stride + w.item];
            w.state = hand.any() ? kOwn : kEnd;
            break;
        case kOwn: {
            w.item = hand.claimed(counter[w.from]++, w.from);
            w.state = w.item >= 0 ? kItem : steal ? kLook : kEnd;
            break;
        }
        case kLook: {
            int most = 0;
            for (int x = 0; x < kXcds; ++x)
                if (hand.open(x, counter[x]) > most) {
                    most = hand.open(x, counter[x]);
                    w.from = x;
                }
            w.state = most == 0 ? kEnd : kTake;
            break;
        }
        case kTake:
            w.item = hand.claimed(counter[w.from]++, w.from);
            w.state = w.item >= 0 ? kItem : kLook;
            break;
    }
}

template <bool OWN>
int run(int members, int n_whole, int left, int parts, const unsigned char* resident, bool steal, unsigned seed, int* done, int stride) {
    const HandOut<OWN> hand{members, n_whole, left, (left + kXcds - 1) / kXcds, parts};
    int counter[kXcds] = {0}, accesses = 0;
    std::mt19937 rng(seed);
    std::vector<Workgroup> live;
    for (int b = 0; b < members * kXcds; ++b) {
        if (!resident[b]) continue;
        Workgroup w{b % kXcds, b / kXcds, kOwn, hand.first(b / kXcds, b % kXcds), b % kXcds};
        if (w.item >= 0) w.state = kItem;
        else if (OWN) w.state = steal && hand.any() ? kLook : kEnd;  // (more workgroups than items)
        if (w.state != kEnd) live.push_back(w);
    }
    while (!live.empty()) {
        const size_t i = rng() % live.size();
        step(live[i], hand, counter, steal, done, stride, accesses);
        if (live[i].state == kEnd) {
            live[i] = live.back();
            live.pop_back();
        }
    }
    return accesses;
}

// Four wavefronts that each see the rank ready at another look of their own.
struct Workgroup4 {
    std::mutex m;
    std::condition_variable all;
    int arrived = 0, reports = 0;
    uint64_t told = 0;
};
struct Wavefront {
    Workgroup4& wg;
    int number, ready_at, looks;
    uint64_t bit;

    bool is_first() const { return number == 0; }
    void pause() const {}
    uint64_t look() { return ++looks >= ready_at ? bit : 0; }
    void report() const {
        std::lock_guard<std::mutex> l(wg.m);
        ++wg.reports;
    }
    uint64_t share(uint64_t r) const {
        std::unique_lock<std::mutex> l(wg.m);
        if (number == 0) wg.told = r;
        ++wg.arrived;
        wg.all.notify_all();
        wg.all.wait(l, [&] { return wg.arrived % 4 == 0; });
        return wg.told;
    }
};

}  // namespace

// Lets four wavefronts wait for one rank; answers[w]: what wavefront w goes on with.  Returns how many have reported a wait that ran out.
extern "C" int await_model(int rank, int spin_limit, const int* ready_at, int* answers, int* limit_after) {
    Workgroup4 wg;
    std::vector<std::thread> threads;
    for (int w = 0; w < 4; ++w)
        threads.emplace_back([&, w] {
            Wavefront f{wg, w, ready_at[w], 0, (uint64_t)1 << rank};
            uint64_t ready = 0;
            int limit = spin_limit;
            answers[w] = await_rank(rank, ready, limit, f) ? 1 : 0;
            limit_after[w] = limit;
        });
    for (std::thread& t : threads) t.join();
    return wg.reports;
}

// Lets the workgroups with resident[block] != 0 work until each finds nothing more; done[xcd * stride + item] counts what they have computed.
// Returns how often they have been at the counters.
extern "C" int hand_out_model(int linked, int mats, int members, int n_whole, int left, int parts, const unsigned char* resident, int steal,
                              unsigned seed, int* done, int stride) {
    const bool own = linked ? (mats == 2 ? owns_first(true, 2) : owns_first(true, 1)) : owns_first(false, mats);
    return own ? run<true>(members, n_whole, left, parts, resident, steal != 0, seed, done, stride)
               : run<false>(members, n_whole, left, parts, resident, steal != 0, seed, done, stride);
}
