// In which order a wavefront of backward_bf16.hip issues its loads and stores, and how many of them its waits leave in flight.
// The hardware counts both together and completes them in the order of issue, so a wait for "all but the last N" is a wait
// for whatever was issued before those N.  Plain constants, so that the order can be walked without a GPU.
#pragma once

namespace ank {

// The dX product.  A stage is KS slots, one matrix instruction each.  Packet i + X is asked for in stage i, its D loads in the
// slots 0 .. D - 1 (mask or activations of the layer below, then dZ_l, or for the top layer the mask words and the head gradient
// of stage i + X + 2).  From stage 1 on the result of the stage before is stored, 8 bytes a lane in the slots E0 + 1, + 3, + 5
// and + 7.  The wait stands in front of the reads of slot WAIT_AT and is for packet i + 1.
// (256 outputs, top layer: the stores ahead of the wait are faster than half of them behind it.  256-256, 262144 samples, both
// products 101 and 106 us; 512-256 165 and 171.)
template <int NR, bool TOP, bool MASKW>
struct DxOrder {
    static constexpr int KS = NR / 16, LA = 4;                   // operands are read LA slots ahead, the last ones of the next stage
    static constexpr int DL = MASKW ? 1 : 2, DM = TOP ? NR / 256 : NR / 128, D = DM + DL + (TOP ? 1 : 0);
    static constexpr int X = !TOP && NR == 512 && !MASKW ? 2 : 3;
    static constexpr int NY = TOP ? 2 : X + 1, NL = X + 1, NT = X + 2;   // places in LDS of dZ_l, of the layer below, of the top layer's
    static constexpr int STORES = 4, E0 = TOP && NR == 512 ? 12 : 4, WAIT_AT = KS - LA;
    static constexpr bool store_at(int s) { return s > E0 && s < E0 + 2 * STORES && (s - E0) % 2 == 1; }
    static constexpr int stores_before_wait()
    {
        int n = 0;
        for (int s = 0; s < WAIT_AT; ++s) n += store_at(s);
        return n;
    }
    // since packet i + 1: the stores of stage i + 1 - X, the loads and stores of the stages between, the loads of stage i and
    // those of its stores that stand before the wait
    static_assert(D - 1 <= E0 + 1 && D <= WAIT_AT, "loads before stores and before the wait");
    static constexpr int LEFT = stores_before_wait() + (X - 1) * (D + STORES);
    static constexpr int LEFT_FIRST = (X - 1) * D;               // stages 0 .. X - 1, some of whose stores do not exist
};

// The dW product.  Packet i + NB is asked for in the second half of stage i, behind the stage's wait, which is for packet i + 1.
// PARTS (top layer): as in dw_body
template <bool TOP, int PARTS>
struct DwOrder {
    static constexpr int STG = TOP ? 16384 + PARTS * 8192 : 32768;   // a stage of 32 samples: X | dZ, top: X | h_L
    static constexpr int NB = !TOP ? 5 : PARTS == 2 ? 3 : 4, NT = NB + 2;   // stages in LDS; of the top layer's mask words and head gradient
    static constexpr int DP = STG / 8192, D = DP + (TOP ? 2 : 0);    // loads per wavefront and stage: pieces, top: mask words, head gradient
    static constexpr int LEFT = D * (NB - 2);
};

}  // namespace ank
