// The weight-only kernel's rule from a shape to a workgroup form.  Plain C++, no HIP: a host program can walk it over shapes.
#pragma once
#include <algorithm>
#include <cstddef>

namespace rcp {

constexpr int WO_TABLE_DWORDS = 64;        // LDS look-up table of a row group
constexpr size_t WO_LDS_BYTES = 160 * 1024;  // of a compute unit

struct WoPlan {
    int ws;     // wavefronts per row group of four rows
    int slots;  // row groups per workgroup, which share one staged token
    int unr;    // 16-byte loads per lane and stage
    int chains; // running sums per lane and row
};

constexpr int wo_padded_units(int K, int span /* lanes per row group x loads per stage */)
{
    return ((K / 16 + span - 1) / span) * span;
}

// tables, the token (16 columns as 64 or 32 bytes) and two sets of four row totals per wavefront
constexpr size_t wo_lds_bytes(bool xf32, int K, int ws, int slots, int unr)
{
    return (static_cast<size_t>(slots) * WO_TABLE_DWORDS + static_cast<size_t>(wo_padded_units(K, 64 * ws * unr)) * (xf32 ? 16 : 8) +
            2 * ws * slots * 4) * 4;
}

// row groups of the compute unit that gets the most
constexpr int wo_busiest(int G, int slots, int cus)
{
    const int blocks = (G + slots - 1) / slots;
    return ((blocks + cus - 1) / cus) * slots;
}

inline WoPlan wo_plan(bool xf32, int N, int K, int cus, int forced_lanes)
{
    const int G = N / 4, U = K / 16;
    const int u1 = wo_busiest(G, 1, cus), u2 = wo_busiest(G, 2, cus), u4 = wo_busiest(G, 4, cus);
    WoPlan p{};
    // Every workgroup stages the token for itself.  While four workgroups of four wavefronts fit a compute unit's LDS beside
    // each other (up to 8192 columns in binary32, 16384 in fp16) that is cheap; two row groups of four wavefronts in one
    // workgroup then pay only where they divide evenly over the units (2 and 4 row groups a unit: 2048 x 6144 binary32
    // 4.69 -> 4.47 us, 4096 x 11008 fp16 7.22 -> 6.80, 4096 x 4096 4.28 -> 4.14; at 2.5 and 3 a unit 2560 x 8192 binary32 would
    // go 5.76 -> 6.00, 3072 x 8192 5.93 -> 6.12), and not where hardly a unit has a second one (1028 x 4096 fp16
    // 2.87 -> 3.19, 1036 x 4608 3.71 -> 3.95; level from 1044 rows on).
    const bool long_token = 4 * wo_lds_bytes(xf32, K, 4, 1, 1) > WO_LDS_BYTES;
    const bool one_each = !long_token && G < cus + cus / 64;
    if (!long_token) {
        p.ws = G <= cus * 4 ? 4 : (G <= cus * 8 ? 2 : 1);
        p.slots = p.ws == 4 ? (u1 % 2 == 0 && !one_each ? 2 : 1) : (p.ws == 2 ? 2 : 4);
    } else if (G > cus * 8) {
        // A longer token leaves the SIMDs with one or two wavefronts unless eight of them share it (32768 x 16384 bf16
        // 52.7 -> 45.4 us, 12288 x 11008 binary32 16.5 -> 15.0, 16384 x 9984 17.9 -> 16.1); single wavefronts keep their row groups
        // while four such workgroups fit and 128 lanes would pad more than 64 (16384 x 8704 binary32 15.9 against 16.7)
        const bool single = wo_padded_units(K, 64) < wo_padded_units(K, 128) && 4 * wo_lds_bytes(xf32, K, 1, 4, 1) <= WO_LDS_BYTES;
        p = single ? WoPlan{1, 4, 1, 1} : WoPlan{2, 4, 1, 1};
    } else {
        // Likewise for fewer rows, as two row groups of four wavefronts or four of two: whichever leaves the busiest unit the
        // fewer units to compute on, padding included (us in binary32, 4 x 2 / 2 x 4 wavefronts: 1280 x 14336 6.1 / 8.1,
        // 2560 x 14336 9.0 / 8.2, 5120 x 16384 12.8 / 14.4, 8192 x 14336 16.1 / 13.2; level where they are equal, and then the one with
        // fewer staged tokens for many rows: 8192 x 16384 16.5 / 15.0).  The forms of four wavefronts stage twice as many
        // tokens; they are taken where they leave an eighth less and all workgroups of the busiest unit are resident at once: one
        // row group where two would leave a unit four instead of three (2560 x 11008 bf16 6.7 against 7.1, 2304 x 22016
        // fp16 9.5 against 10.0; at 14336 columns binary32, where two are resident, 10.6 against 8.2), two of two
        // wavefronts where 256 lanes would pad (6144 x 10240 binary32 9.0 against 9.4).
        const int pad4 = wo_padded_units(K, 256), pad2 = wo_padded_units(K, 128);
        const int c42 = u2 * pad4, c24 = u4 * pad2;
        const bool two = c24 < c42 || (c24 == c42 && G > cus * 4);
        p = two ? WoPlan{2, 4, 1, 1} : WoPlan{4, 2, 1, 1};
        const int best = std::min(c42, c24);
        if (8 * u1 * pad4 <= 7 * best && u1 * wo_lds_bytes(xf32, K, 4, 1, 1) <= WO_LDS_BYTES) p = {4, 1, 1, 1};
        else if (G > cus * 4 && 8 * u2 * pad2 <= 7 * best && u2 / 2 * wo_lds_bytes(xf32, K, 2, 2, 1) <= WO_LDS_BYTES) p = {2, 2, 1, 1};
    }
    if (forced_lanes >= 64) {  // 64, 128, 256 lanes per row group, four wavefronts per workgroup
        p.ws = forced_lanes / 64;
        p.slots = 4 / p.ws;
    }
    while (p.ws > 1 && U < 64 * p.ws) {
        p.ws /= 2;
        p.slots = 4 / p.ws;
    }
    // Up to four row groups a unit a row is summed in 256 parts, whatever the form: two running sums a lane where 128 lanes share it
    // (one would be faster by 1 %, 2560 x 14336 binary32 8.17 against 8.28 us, with 1.3 times the rounding error: 1.76e-7 and
    // 1.36e-7 of the output in binary32 there, 1.33e-7 with 256 lanes)
    p.chains = p.ws == 2 && p.slots == 4 && G <= cus * 4 ? 2 : 1;
    // Loads per stage: one, which takes the fewest registers (55 to 61, eight wavefronts a SIMD; four take 83 to 88, five
    // wavefronts): 22016 x 4096 fp16 10.86 -> 10.09 us, 12288 x 4096 7.11 -> 6.53, 8192 x 16384 binary32 17.6 -> 16.4.
    // Where one row group or less falls on a compute unit (1000 x 16384 4.92 against 5.28 us) and in matrices that stream
    // for long (from 56 MB on: 80000 x 3104 24.1 against 25.6, 131072 x 4096 43.0 against 45.2, 32768 x 16384 bf16 45.2 against 47.2;
    // but 14336 x 22016 fp16 29.5 against 25.7), more loads in flight win: the largest of 4, 2, 1 that pads a lane's units by at
    // most a tenth (padding units are computed on like real ones).
    // Likewise two loads where they are all that a lane has: a whole row group of one wavefront (100000 x 1504 fp16 takes 18.1 us
    // with one, 16.9 with two, 40000 x 1504 bf16 9.0 / 9.3, 50000 x 2048 bf16 11.3 either way; with four units a lane 40000 x 4096
    // 12.8 with one, 14.0 with four), and of two wavefronts up to four row groups a unit (1028 x 2080 fp16 3.09 / 2.97, 2392 x 2080
    // bf16 4.10 / 3.96, 4096 x 2400 binary32 4.24 / 4.14, 4096 x 3904 level; 5120 x 3904 binary32 4.87 / 5.02).
    p.unr = 1;
    const int per_lane = (U + 64 * p.ws - 1) / (64 * p.ws);
    const bool both = per_lane == 2 && (p.ws == 1 || (p.ws == 2 && p.slots == 2 && G <= cus * 4));
    if (G <= cus || (one_each && p.ws == 4) || static_cast<long long>(N) * K / 4 >= (56LL << 20) || both) {
        for (int c = 2; c <= 4; c *= 2)
            if (((per_lane + c - 1) / c) * c * 10 <= per_lane * 11) p.unr = c;
    }
    return p;
}

}  // namespace rcp
