// The products of backward_bf16.hip as orders of loads, stores, waits and reads of one wavefront, walked on the CPU: what a
// stage reads from LDS has to be older than what the last wait in front of it leaves in flight, and a load may go to a place
// in LDS only behind a wait (they are barriers too) that follows the last read of that place.
// Prints "ok <forms>" or the first read or load that is not covered.
#include <stdio.h>
#include <stdlib.h>
#include <map>
#include <utility>
#include <vector>
#include "../../paper_2104_06272_amd/csrc/backward_bf16_order.h"

using namespace ank;

enum Kind { LOW, DZ, MASK, HEAD };            // of the layer below; dZ_l (dW: all operands); top layer: mask words, head gradient

struct Walk {
    const char* form;
    int a, b, c;
    int waits = 0;
    std::vector<bool> landed;                  // by issue order: known to be done
    std::map<std::pair<int, int>, int> issued; // (kind, stage) -> issue order of its last load
    std::map<std::pair<int, int>, std::pair<int, int>> place;   // (kind, place in LDS) -> stage it holds, waits at the last read
    int op() { landed.push_back(false); return (int)landed.size() - 1; }
    [[noreturn]] void bad(const char* what, int kind, int stage, int i)
    {
        printf("%s<%d, %d, %d>: %s, kind %d of stage %d in stage %d\n", form, a, b, c, what, kind, stage, i);
        exit(1);
    }
    void load(int kind, int stage, int places, int i)
    {
        const auto at = std::make_pair(kind, stage % places);
        const auto held = place.find(at);
        // (held.first: what the place held; the same stage again is another piece of it)
        if (held != place.end() && held->second.first != stage && held->second.second >= waits) bad("overwritten before its last read", kind, stage, i);
        place[at] = {stage, -1};
        issued[{kind, stage}] = op();
    }
    void store() { op(); }
    void wait(int left)
    {
        for (int k = 0; k < (int)landed.size() - left; ++k) landed[k] = true;
        ++waits;
    }
    void barrier() { ++waits; }
    void read(int kind, int stage, int places, int i)
    {
        const auto at = place.find({kind, stage % places});
        if (at == place.end() || at->second.first != stage) bad("not in its place", kind, stage, i);
        if (!landed[issued[{kind, stage}]]) bad("read before its load is known to have landed", kind, stage, i);
        at->second.second = waits;
    }
};

// dx_body: `n` stages, numbered on past the last as the kernel does (it asks for the last one again)
template <int NR, bool TOP, bool MASKW> static void walk_dx(int n)
{
    using O = DxOrder<NR, TOP, MASKW>;
    Walk w{"dX", NR, TOP, MASKW};
    auto load = [&](int p, int k, int i) {                       // piece k of packet p
        if (k < O::DL) w.load(LOW, p, O::NL, i);
        else if (!TOP) w.load(DZ, p, O::NY, i);
        else if (k < O::DL + O::DM) w.load(MASK, p + 2, O::NT, i);
        else w.load(HEAD, p + 2, O::NT, i);
    };
    if (TOP)
        for (int t = 0; t < 2; ++t) {
            for (int k = 0; k < O::DM; ++k) w.load(MASK, t, O::NT, -1);
            w.load(HEAD, t, O::NT, -1);
        }
    for (int p = 0; p < O::X; ++p)
        for (int k = 0; k < O::D; ++k) load(p, k, -1);
    w.wait(0);
    if (TOP) { w.read(HEAD, 0, O::NT, -1); w.read(HEAD, 1, O::NT, -1); w.read(MASK, 0, O::NT, -1); w.barrier(); }
    else w.read(DZ, 0, O::NY, -1);
    for (int i = 0; i < n; ++i)
        for (int s = 0; s < O::KS; ++s) {
            if (s == O::WAIT_AT) w.wait(i >= O::X ? O::LEFT : O::LEFT_FIRST);
            if (!TOP) w.read(DZ, s + O::LA < O::KS ? i : i + 1, O::NY, i);
            if (s < O::D) load(i + O::X, s, i);
            if (s < (MASKW ? 1 : 4)) w.read(LOW, i, O::NL, i);
            if (O::store_at(s) && i > 0) w.store();
            if (TOP && s % 16 == 0 && s / 16 < NR / 256) w.read(MASK, i + 1, O::NT, i);
            if (TOP && s == O::WAIT_AT - 6) w.read(HEAD, i + 2, O::NT, i);
        }
}

template <bool TOP, int PARTS> static void walk_dw(int n)
{
    using O = DwOrder<TOP, PARTS>;
    Walk w{"dW", TOP, PARTS, 0};
    auto load = [&](int p, int k, int i) {
        if (k < O::DP) w.load(DZ, p, O::NB, i);
        else w.load(k == O::DP ? MASK : HEAD, p + 2, O::NT, i);
    };
    if (TOP)
        for (int t = 0; t < 2; ++t) { w.load(MASK, t, O::NT, -1); w.load(HEAD, t, O::NT, -1); }
    for (int p = 0; p < O::NB; ++p)
        for (int k = 0; k < O::D; ++k) load(p, k, -1);
    if (TOP) {
        w.wait(0);
        for (int t = 0; t < 3; ++t) w.read(HEAD, t, O::NT, -1);
        for (int t = 0; t < 2; ++t) w.read(MASK, t, O::NT, -1);
        w.barrier();
    } else w.wait(O::D * (O::NB - 1));
    w.read(DZ, 0, O::NB, -1);
    for (int i = 0; i < n; ++i) {
        for (int s = 0; s < 8; ++s) w.read(DZ, i, O::NB, i);      // first half: the second step's operands, top: h_L for the head matrix
        w.wait(O::LEFT);
        for (int s = 0; s < 8; ++s) {
            if (TOP && s == 0) w.read(MASK, i + 2, O::NT, i);
            const int k = TOP ? s : s - 4;                       // loads in the first (top) or the last slots
            if (k >= 0 && k < O::D) load(i + O::NB, k, i);
            if (s < 6) w.read(DZ, i + 1, O::NB, i);
            if (TOP && s == 2) w.read(HEAD, i + 3, O::NT, i);
        }
    }
}

int main()
{
    for (int n = 1; n <= 40; ++n) {
        walk_dx<256, false, false>(n); walk_dx<256, false, true>(n); walk_dx<256, true, false>(n); walk_dx<256, true, true>(n);
        walk_dx<512, false, false>(n); walk_dx<512, false, true>(n); walk_dx<512, true, false>(n); walk_dx<512, true, true>(n);
        walk_dw<false, 0>(n); walk_dw<true, 0>(n); walk_dw<true, 1>(n); walk_dw<true, 2>(n);
    }
    printf("ok 12\n");
}
