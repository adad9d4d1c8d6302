// Host model of how the workgroups of a grouped GEMM come to their work items, on the arithmetic of csrc/hand_out.h.
#define __host__
#define __device__
#include <stdint.h>

#include <random>
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
void step(Workgroup& w, const HandOut<OWN>& hand, int (&counter)[kXcds], bool steal, int* done, int stride) {
    switch (w.state) {
        case kItem:
            ++done[w.from * stride + w.item];
            w.state = kOwn;
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
void run(int members, int n_whole, int left, int parts, const unsigned char* resident, bool steal, unsigned seed, int* done, int stride) {
    const HandOut<OWN> hand{members, n_whole, left, (left + kXcds - 1) / kXcds, parts};
    int counter[kXcds] = {0};
    std::mt19937 rng(seed);
    std::vector<Workgroup> live;
    for (int b = 0; b < members * kXcds; ++b) {
        if (!resident[b]) continue;
        Workgroup w{b % kXcds, b / kXcds, kOwn, hand.first(b / kXcds, b % kXcds), b % kXcds};
        if (w.item >= 0) w.state = kItem;
        else if (OWN) w.state = steal ? kLook : kEnd;  // (more workgroups than items)
        live.push_back(w);
    }
    while (!live.empty()) {
        const size_t i = rng() % live.size();
        step(live[i], hand, counter, steal, done, stride);
        if (live[i].state == kEnd) {
            live[i] = live.back();
            live.pop_back();
        }
    }
}

}  // namespace

// Lets the workgroups with resident[block] != 0 work until each finds nothing more; done[xcd * stride + item] counts what they have computed.
extern "C" int hand_out_model(int linked, int mats, int members, int n_whole, int left, int parts, const unsigned char* resident, int steal,
                              unsigned seed, int* done, int stride) {
    const bool own = linked ? (mats == 2 ? owns_first(true, 2) : owns_first(true, 1)) : owns_first(false, mats);
    if (own) run<true>(members, n_whole, left, parts, resident, steal != 0, seed, done, stride);
    else run<false>(members, n_whole, left, parts, resident, steal != 0, seed, done, stride);
    return own ? 1 : 0;
}
