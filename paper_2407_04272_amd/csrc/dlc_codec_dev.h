// Device-side building blocks shared by the compression kernels of libdlc (gfx950 only): the LDS histogram
// layout, the Huffman codebook builder, the look-back scan over groups and the bit-stream writer.
#pragma once
#include "dlc_internal.h"

namespace dlc {

// ------------------------------------------------------------------------------------------------
// The symbol window.  Almost every element of a bell-shaped table falls into a few bins around zero, so the
// streaming kernels work on window indices: index v in [0, 254) stands for symbol win_lo + v, index 254 for an
// escape, index 255 for everything else (a symbol outside the window, a position past the end of the table).
//   - the histogram kernel counts window indices in LDS with kWinCopies copies per row (copy = lane mod
//     kWinCopies, so a wavefront's 64 updates spread over the banks whatever the symbols are) and hands the
//     indices on as one byte per element (the symbol plane); the rare index 255 is counted exactly by symbol, the
//     escapes in row 254
//   - the encode kernel looks window indices up in a 256-entry LDS table and goes back to the element itself
//     only for index 255
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kWinBins = 255;   // index of "see the element itself" (a symbol outside the window, a position past the end)
constexpr uint32_t kWinEsc = 254;    // index of an escape: its code comes from the table like any other, its record from the payload
constexpr uint32_t kWinSkip = 253;   // with row matching: an element of a row that is stored as a reference (no bits)
// window indices that stand for a symbol: [0, win_bins)
__host__ __device__ inline uint32_t win_bins(uint32_t lz) { return lz ? kWinSkip : kWinEsc; }
constexpr uint32_t kWinCopies = 16;
__host__ __device__ inline uint32_t win_lo_of(uint32_t R) { return R > kWinBins / 2u ? R - kWinBins / 2u : 0u; }
// The symbol plane: the window index of every element, one byte each, in element order; a table's part is padded to
// whole groups (and the last unit of a table is always written whole), so that every group has its 64*S bytes.
__host__ __device__ inline size_t plane_stride(const Geom& g) { return (size_t)g.G * kW * g.S; }
// LDS of the histogram kernel in words: window [kWinBins + 1][kWinCopies] | exact counts [K]
__host__ __device__ inline size_t hist_lds_bytes(uint32_t K) { return (((size_t)(kWinBins + 1) * kWinCopies + K) * 4 + 15) & ~size_t(15); }

// ------------------------------------------------------------------------------------------------
// quantise and count: one block of units of a table (used by the histogram kernel and by the kernel for small tables)
// ------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ void lds_count(uint32_t addr) {
    __hip_atomic_fetch_add(reinterpret_cast<lds_u32*>(addr), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct HistC {
    int ubias;          // window index of bin 0
    uint32_t win_lo;    // symbol of window index 0
    uint32_t lanebase;  // LDS address of this lane's copy of window row 0
    uint32_t exact;     // LDS address of the exact counts
    float Rf;
    float first, last;  // kMagic + the lowest and the highest window index a bin inside the radius can have
    float eb_sure;      // a bound a little below the table's
};

// A float of kMagicF + i, 0 <= i < 2^22, has i in its low bits, and adding kMagicF + i to a product in one fused operation
// rounds the product to a whole number (half to even).
constexpr float kMagicF = 12582912.0f;  // 1.5 * 2^23
constexpr uint32_t kMagicBits = 0x4B400000u;

template <bool LZ>
__device__ __forceinline__ HistC hist_consts(const Geom& g, const QParam& q, uint32_t lds0, uint32_t lane) {
    HistC H;
    H.win_lo = win_lo_of(g.R);
    H.ubias = (int)(g.R - H.win_lo);
    H.lanebase = lds0 + (lane & (kWinCopies - 1u)) * 4u;
    H.exact = lds0 + (kWinBins + 1u) * kWinCopies * 4u;
    H.Rf = (float)g.R;
    const int r1 = (int)g.R - 1;
    H.first = kMagicF + (float)max(0, H.ubias - r1);
    H.last = kMagicF + (float)min((int)(LZ ? kWinSkip : kWinEsc) - 1, H.ubias + r1);
    // Inside the window (|bin| <= 127) an element that is within eb_sure of a bin's centre by one fused operation is in
    // that bin and inside the bound by the quantiser's own roundings too: product and reciprocal are off by 2^-16 of a bin
    // together, the reconstruction by 2^-16 of the bound, and the margin is 2^-13.  Where a denormal or an overflowing
    // bound makes those relative errors larger, nothing is sure.
    H.eb_sure = (q.eb > 1e-30f && q.eb < 1e30f) ? q.eb * (1.0f - 0x1p-13f) : -1.0f;
    return H;
}

constexpr uint32_t kPastEnd = 0x80000001u;  // no element within the radius has this window index: a position past the end of the table
constexpr uint32_t kHistBlk = 4;  // units whose loads are issued back to back

// One block of kHistBlk units of one table; a unit is 256 consecutive elements (one 16-byte load per lane).
// `rem` = elements of the table from the block's first element on, `n_units` = units of the block that are this
// wavefront's.  FULL: all kHistBlk units are, and all their elements are inside the table (no masking at all).
// Index 254 in the plane stands for an escape.  LZ (row matching): the window is one symbol narrower, because index
// 253 stands for an element of a row that is stored as a reference (the row-matching kernels put it there
// afterwards); the symbol that would have had that index goes the way of everything outside the window.
//
// The payload's way from memory bounds it (512 MiB read and 128 MiB written by k_hist in 109 us, 6.2 TB/s), with the
// instructions an element takes close behind.  The rule is an element well inside a bin of the window: one fused operation
// rounds it to the window index (which then lies in the float's low bits: no conversion), one clamp, one fused operation
// gives its distance from the bin's centre, and the address of its count is a shift and an addition: 7 vector
// instructions.  A unit with any other element, one in thirty, goes through the quantiser's own arithmetic, 15 of them (for
// every element: k_hist 113 us).  Neither more loads in flight nor counters that no two lanes share made it shorter; a
// compute unit by itself reads about 16 bytes a cycle.
template <bool F16, bool VEC, bool FULL>
struct HistLoads {
    float x[kHistBlk][4];
    uint32_t valid[kHistBlk];
    __device__ __forceinline__ void load(const uint8_t* base, uint32_t rem, uint32_t n_units, uint32_t lane) {
        uint32_t raw[4];
#pragma unroll
        for (uint32_t u = 0; u < kHistBlk; ++u)
            valid[u] = load4<F16, VEC, FULL>(base, lane * kV + u * (kW * kV), FULL ? 0xFFFFFFFFu : (u < n_units ? rem : 0u), x[u], raw);
    }
};

// PLANE: kNoPlane, kPlane, or kPlaneThrough: past the caches, for other work-groups of the launch.  (The stores stand where they are
// made: behind a function of their own the compiler no longer shares one between the two ways through a unit, and k_hist in front of row matching,
// 96 tables of 8192 x 32, took 27.7 us instead of 25.5.)
enum PlaneStore { kNoPlane, kPlane, kPlaneThrough };
template <bool F16, bool VEC, bool FULL, bool LZ, PlaneStore PLANE = kPlane>
__device__ __forceinline__ void hist_count(const HistLoads<F16, VEC, FULL>& D, uint32_t n_units, uint32_t lane, const QParam& q,
                                           const HistC& H, uint32_t* plane) {
    constexpr uint32_t kBins = LZ ? kWinSkip : kWinEsc;  // window indices that stand for a symbol
    const float mg = kMagicF + (float)H.ubias;
    const uint32_t rows = H.lanebase - kMagicBits * (kWinCopies * 4u);  // (modulo 2^32)
#pragma unroll
    for (uint32_t u = 0; u < kHistBlk; ++u) {
        uint32_t sl[4];
        float t[4];
        bool sure = FULL || D.valid[u] == 0xFu;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float xv = D.x[u][v];
            if constexpr (F16) {  // (the reconstruction is rounded to half: the quantiser's own test, as it is)
                const float r = __builtin_rintf(xv * q.inv);
                t[v] = __builtin_amdgcn_fmed3f(r + mg, H.first, H.last);
                const float rc = t[v] - mg;
                const float xh = __half2float(half_rne(rc * q.ebx2));
                sure = sure & (rc == r) & (__builtin_fabsf(xv - xh) <= q.eb);
            } else {
                t[v] = __builtin_amdgcn_fmed3f(__builtin_fmaf(xv, q.inv, mg), H.first, H.last);
                sure = sure & (__builtin_fabsf(__builtin_fmaf(mg - t[v], q.ebx2, xv)) <= H.eb_sure);
            }
        }
        if (__builtin_expect(__ballot(!sure) == 0ull, 1)) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                sl[v] = __float_as_uint(t[v]);
                lds_count((sl[v] << 6) + rows);
            }
            static_assert(kWinCopies * 4u == 64u, "a row of the window");
            const uint32_t word = __builtin_amdgcn_perm(sl[1], sl[0], 0x0C0C0400u) | __builtin_amdgcn_perm(sl[3], sl[2], 0x04000C0Cu);
            if constexpr (PLANE == kPlane) plane[u * kW + lane] = word;
            if constexpr (PLANE == kPlaneThrough) __hip_atomic_store(&plane[u * kW + lane], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            continue;
        }
        uint32_t w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            // the quantiser (same arithmetic as quant_symbol), result as a window index
            const float xv = D.x[u][v];
            const float r = __builtin_rintf(xv * q.inv);
            float xh = r * q.ebx2;
            if constexpr (F16) xh = __half2float(half_rne(xh));
            const float d = xv - xh;
            const bool ok = (__builtin_fabsf(r) < H.Rf) & (__builtin_fabsf(d) <= q.eb);  // no short circuit: no branches
            w[v] = (uint32_t)((int)r + H.ubias);  // (bins below the window wrap to just under 2^32)
            sl[v] = w[v] < kBins ? w[v] : kWinBins;
            sl[v] = ok ? sl[v] : kWinEsc;
            if constexpr (FULL) {
                lds_count(sl[v] * (kWinCopies * 4u) + H.lanebase);
            } else {
                if ((D.valid[u] >> v) & 1u) lds_count(sl[v] * (kWinCopies * 4u) + H.lanebase);
                else { sl[v] = kWinBins; w[v] = kPastEnd; }
            }
        }
        // index 255 is rare: count those elements exactly, by symbol (escapes are counted in window row 254, which
        // the merge adds to symbol 0)
        if (__ballot(max(max(sl[0], sl[1]), max(sl[2], sl[3])) == kWinBins) != 0ull) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (sl[v] == kWinBins && w[v] != kPastEnd) lds_count(H.exact + (w[v] + H.win_lo) * 4u);
        }
        // the window indices of these four elements, for the encode kernel (a unit of this wavefront only)
        if constexpr (PLANE != kNoPlane) {
            if (FULL || u < n_units) {
                const uint32_t word = sl[0] | (sl[1] << 8) | (sl[2] << 16) | (sl[3] << 24);
                if constexpr (PLANE == kPlane) plane[u * kW + lane] = word;
                else __hip_atomic_store(&plane[u * kW + lane], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <bool F16, bool VEC, bool FULL, bool LZ, PlaneStore PLANE = kPlane>
__device__ __forceinline__ void hist_block(const uint8_t* base, uint32_t rem, uint32_t n_units, uint32_t lane, const QParam& q,
                                           const HistC& H, uint32_t* plane) {
    HistLoads<F16, VEC, FULL> D;
    D.load(base, rem, n_units, lane);
    hist_count<F16, VEC, FULL, LZ, PLANE>(D, n_units, lane, q, H, plane);
}

// The units [u0, u1) of a table (u0 a multiple of kHistBlk, and u1 if the table does not end there) by a work-group of NW wavefronts: a block of
// units at a time, the loads of the next two on their way while one is counted (memory takes 3 us to answer when all compute
// units ask, and there are few wavefronts); then the block that the table ends in.
template <bool F16, bool VEC, uint32_t NW, PlaneStore PLANE>
__device__ __forceinline__ void hist_units(const uint8_t* tab, uint8_t* plane_t, const Geom& g, uint32_t u0, uint32_t u1, uint32_t wave,
                                           uint32_t lane, const QParam& q, const HistC& H) {
    const uint32_t whole = min(u1, g.n / (kW * kV));  // units that lie inside the table
    auto first_of = [&](uint32_t u) { return tab + (size_t)u * (kW * kV) * g.es; };
    auto plane_of = [&](uint32_t u) { return reinterpret_cast<uint32_t*>(plane_t + u * (kW * kV)); };
    uint32_t u = u0 + wave * kHistBlk;
    constexpr uint32_t kStep = NW * kHistBlk;
    HistLoads<F16, VEC, true> A, B, C;
    auto have = [&](uint32_t v) { return v + kHistBlk <= whole; };  // uniform over the wavefront
    if (have(u)) A.load(first_of(u), 0u, kHistBlk, lane);
    if (have(u + kStep)) B.load(first_of(u + kStep), 0u, kHistBlk, lane);
    auto turn = [&](HistLoads<F16, VEC, true>& now, HistLoads<F16, VEC, true>& later) {
        if (!have(u)) return false;
        if (have(u + 2u * kStep)) later.load(first_of(u + 2u * kStep), 0u, kHistBlk, lane);
        hist_count<F16, VEC, true, false, PLANE>(now, kHistBlk, lane, q, H, plane_of(u));
        u += kStep;
        return true;
    };
    while (turn(A, C) && turn(B, A) && turn(C, B)) {}
    if (u < u1)
        hist_block<F16, VEC, false, false, PLANE>(first_of(u), g.n - u * (kW * kV), min(kHistBlk, u1 - u), lane, q, H, plane_of(u));
}

// a table's counts in LDS (window rows, then the exact counts), added to those in memory by NT threads: the copies of a row (skewed
// start: the threads of a wavefront read different banks) plus the exact counts
template <bool LZ, uint32_t NT>
__device__ __forceinline__ void hist_merge(const uint32_t* lh, const Geom& g, uint32_t* hist_t, uint32_t tid) {
    const uint32_t* exact = lh + (kWinBins + 1u) * kWinCopies;
    const uint32_t win_lo = win_lo_of(g.R);
    for (uint32_t k = tid; k < g.K; k += NT) {
        uint32_t s = exact[k];
        const uint32_t w = k - win_lo;
        if (w < (LZ ? kWinSkip : kWinEsc)) {
            const uint32_t* row = lh + w * kWinCopies;
            for (uint32_t c = 0; c < kWinCopies; ++c) s += row[(c + tid) & (kWinCopies - 1u)];
        }
        if (k == 0u) {  // the escapes
            const uint32_t* row = lh + kWinEsc * kWinCopies;
            for (uint32_t c = 0; c < kWinCopies; ++c) s += row[c];
        }
        if (s) atomicAdd(&hist_t[k], s);
    }
}

// ------------------------------------------------------------------------------------------------
// Huffman codebook of one table, built by one work-group (NT threads) from the table's histogram.
//   leaves ordered by (count, symbol); two queues (leaves, merged nodes in creation order; one list in their order
//   where a wavefront holds all used symbols); a tie between the queue heads takes the leaf; longest code above LMAX: lengths are cut to LMAX, the
//   Kraft sum is repaired one unit at a time (a code of length LMAX pairs up with a code taken from
//   the deepest shorter level) and the resulting lengths are handed out most frequent symbol first;
//   canonical codewords in (length, symbol) order.  One used symbol: length 0.
//   smem: codebook_smem(K) bytes, 16-byte aligned.  Ends with a barrier; results are in global memory.
// ------------------------------------------------------------------------------------------------
__host__ __device__ constexpr size_t codebook_smem(uint32_t K) { return (size_t)K * (8 + 4 + 4 + 2) + 64 * 4; }

// what another work-group of the same launch may read of a table's codebook goes past the caches
__device__ __forceinline__ void store_tmeta(TMeta* p, const TMeta& m) {
    uint64_t* q = reinterpret_cast<uint64_t*>(p);
    __hip_atomic_store(q, (uint64_t)m.n_used | (uint64_t)m.sym_lo << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, (uint64_t)m.sym_hi | (uint64_t)m.n_outliers << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool WITHIN>
__device__ __forceinline__ TMeta load_tmeta(const TMeta* p) {
    if constexpr (!WITHIN) return *p;
    const uint64_t* q = reinterpret_cast<const uint64_t*>(p);
    const uint64_t a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    TMeta m;
    m.n_used = (uint32_t)a; m.sym_lo = (uint32_t)(a >> 32); m.sym_hi = (uint32_t)b; m.n_outliers = (uint32_t)(b >> 32);
    return m;
}

struct CodebookShared {
    uint32_t first[kLmaxLimit + 2], more[kLmaxLimit + 2];  // by length: the first codeword; leaves of that length and shorter
};

__device__ __forceinline__ uint32_t lane_get(uint32_t v, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)__builtin_amdgcn_readfirstlane((int)(l & 63u)));
}
__device__ __forceinline__ uint32_t lane_put(uint32_t vec, uint32_t l, uint32_t val, uint32_t lane) {
    return lane == l ? val : vec;
}

// lane read with a wavefront-uniform lane number that the compiler can see is uniform (no broadcast of the number first)
__device__ __forceinline__ uint32_t lane_read(uint32_t v, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}

// the next lane's value; the last lane gets `last`
__device__ __forceinline__ uint32_t lane_next(uint32_t v, uint32_t last) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
}

// Lane L of clv: how many codes have length L, 1 <= L <= LM, those that were longer cut to LM.  The Kraft sum is repaired: a code of
// length LM pairs up with a code taken from the deepest shorter level, one unit at a time.
__device__ __forceinline__ uint32_t wave_limit_lengths(uint32_t clv, uint32_t LM, uint32_t lane) {
    uint32_t kraft = wave_sum(lane >= 1u && lane <= LM ? clv << (LM - lane) : 0u);  // in units of 2^-LM (K codes of length 1 at most: 2^23)
    while (kraft > 1u << LM && lane_get(clv, LM) > 0u) {
        const uint64_t shorter = __ballot(clv > 0u && lane >= 1u && lane < LM);
        clv = lane_put(clv, LM, lane_get(clv, LM) - 1u, lane);
        if (shorter) {
            const uint32_t Ld = 63u - (uint32_t)__builtin_clzll(shorter);
            clv = lane_put(clv, Ld, lane_get(clv, Ld) - 1u, lane);
            clv = lane_put(clv, Ld + 1u, lane_get(clv, Ld + 1u) + 2u, lane);
        }
        kraft -= 1u;
    }
    return clv;
}

// The whole tree of a table with at most 64 used symbols and less than 2^30 elements, built by one wavefront in registers: lane i
// holds used symbol i (symbol order) on entry.  The merge keeps leaves and merged nodes in ONE list in lane order, rising by
// weight: a step takes the two at the front off, moves the list up by two lanes and puts their sum behind everything that is not
// heavier.  That is the two-queue merge's order, ties included: a weight stands above two bits, 0 for a leaf and 1 for a merged
// node, so a leaf comes before every node of its weight, and of two nodes of one weight the older one comes first.  The list holds
// nothing else: leaves and nodes leave it in their own orders, so how many nodes every step took, which are the low two bits of the
// sum it made, says what is below what.  Nodes of one depth are steps next to one another, and so are the leaves they took: from the
// root down, a level is where the first node of the level above it starts to take.
// What bounds it is one wavefront's chains of dependent instructions (about seven cycles each): with 41 symbols 40 steps of 45 cycles
// (two queues with their heads read by computed lane numbers took 345, the numbers of what was merged carried along in a second list
// 150), the sort 1100, 13 levels 1000.  Lengths above LM are limited as described above.
// Returns the code length of the symbol the lane came in with.  2 <= n <= 64.
constexpr uint32_t kWaveElements = 1u << 30;  // tables of fewer elements
__device__ __forceinline__ uint32_t wave_huffman_lengths(uint32_t n, uint32_t LM, uint32_t cnt, uint32_t lane) {
    const uint32_t kInf = 0xFFFFFFFFu;
    // position in (count, symbol) order (lanes past n - 1, eight at a time at most, have the largest keys)
    uint32_t rank = 0;
    if (__ballot(lane < n && cnt >= 1u << 26) == 0ull) {  // the rule: count and lane are one number
        const uint32_t key = lane < n ? cnt << 6 | lane : kInf;
#pragma unroll
        for (uint32_t j0 = 0; j0 < 64u; j0 += 8u) {
            if (j0 < n) {  // uniform
#pragma unroll
                for (uint32_t u = 0; u < 8u; ++u) rank += lane_read(key, j0 + u) < key ? 1u : 0u;
            }
        }
    } else {
        const uint64_t key = (uint64_t)cnt << 32 | lane;
#pragma clang loop unroll(disable)
        for (uint32_t j = 0; j < n; ++j) rank += ((uint64_t)lane_read(cnt, j) << 32 | j) < key ? 1u : 0u;
    }
    if (lane >= n) rank = lane;  // idle lanes keep their place
    // the sorted sequence: every lane sends its count to the lane of its rank
    const uint32_t sent = (uint32_t)__builtin_amdgcn_ds_permute((int)(rank << 2), (int)cnt);
    uint32_t w = lane < n ? sent << 2 : kInf;  // (a sum of all counts is less than 2^30: kInf is heavier than any)
    uint32_t w1 = kInf, w2 = kInf;             // the list a lane further on, and two (the last lane keeps what it has)
    uint32_t sums = 0, steps = 0;              // of all steps, the latest in lane 0
    for (; steps + 1u < n; steps += 4u) {      // (steps past the last, three at most, are of no consequence)
#pragma unroll
        for (uint32_t u = 0; u < 4u; ++u) {
            w1 = lane_next(w, w1);
            w2 = lane_next(w1, w2);
            const uint32_t both = w + w1;
            uint32_t node = (both & ~3u) | 1u;
            asm("" : "+v"(node));  // (one vector instruction, not two scalar ones behind the lane read)
            const uint32_t sum = lane_read(node, 0);
            sums = (uint32_t)__builtin_amdgcn_update_dpp((int)both, (int)sums, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
            // not heavier than the sum: it moves up by two lanes; the sum's place; else by one (the median of the three)
            w = max(min(w1, sum), min(max(w1, sum), w2));
        }
    }
    const uint32_t made = (uint32_t)__shfl((int)sums, (int)((steps - 1u - lane) & 63u), 64);  // lane k: the sum of step k
    // nodes that the steps before step `lane` took; twice as many things less those are leaves
    const uint32_t took = lane + 1u < n ? made & 3u : 0u, nodes = wave_incl_scan(took) - took;
    uint32_t len = 1u, first = n - 2u;  // of the leaf at sorted position `lane`; the first node of a level (the root: alone)
    for (;;) {
        const uint32_t below = lane_read(nodes, first);
        len += lane < 2u * first - below ? 1u : 0u;
        if (first == 0u) break;  // (its level is the last, or it takes nodes before itself)
        first = below;
    }
    len = lane < n ? len : 0u;
    if (__ballot(len > LM) != 0ull) {
        const uint32_t lc = min(len, LM);
        uint32_t clv = 0;
        for (uint32_t L = 1; L <= LM; ++L) clv = lane_put(clv, L, (uint32_t)__popcll(__ballot(lane < n && lc == L)), lane);
        clv = wave_limit_lengths(clv, LM, lane);
        // lengths are handed out most frequent leaf first (the leaves are sorted by rising count)
        const uint32_t back = n - 1u - lane;
        uint32_t acc = 0, nl = 1;
        for (uint32_t L = 1; L < LM; ++L) {
            acc += lane_get(clv, L);  // leaves with a length of at most L
            nl += (back >= acc) ? 1u : 0u;
        }
        len = lane < n ? nl : 0u;
    }
    // back to symbol order: the lane that came in with a symbol reads the length at that symbol's sorted position
    return lane < n ? __shfl(len, rank, 64) : 0u;
}

// canonical codeword of every lane's symbol (the lanes are in symbol order; length 0: not used): the first code of each
// length, then the rank among the symbols of that length
__device__ __forceinline__ uint32_t wave_canonical_code(uint32_t len) {
    uint32_t code = 0, mine = 0;
#pragma unroll
    for (uint32_t L = 1; L <= (uint32_t)kLmaxLimit; ++L) {
        code <<= 1;
        const uint64_t same = __ballot(len == L);
        mine = len == L ? __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, code)) : mine;
        code += (uint32_t)__popcll(same);
    }
    return mine;
}

// The codebook of a table with at most 64 used symbols (the rule), by ONE wavefront: same inputs and outputs as
// codebook_build below, which takes every other table.  The wavefront reads the histogram 64 symbols at a time,
// gathers the used symbols into its lanes through `wsm` (LDS of this wavefront: 64 keys, then K entries of 16
// bits), builds the tree in registers, and writes the K entries of the table and the code lengths.  Returns false,
// with the histogram untouched, when the table has more than 64 used symbols.
//   K: a multiple of 64.  (Radius 8 and 16 give 16 and 32 symbols; the memory behind such a table's counts and codes is
//   the next table's: those go to codebook_build.)
//   wsm: 512 + 2 * K bytes, 8-byte aligned.
constexpr uint32_t kWaveAlphabet = 64;  // least alphabet of codebook_build_wave (every larger one is a power of two)
__host__ __device__ constexpr size_t codebook_wave_smem(uint32_t K) { return 512 + 2 * (size_t)K; }
__host__ __device__ constexpr size_t codebook_four_smem(uint32_t K) {
    return codebook_smem(K) > 4 * codebook_wave_smem(K) ? codebook_smem(K) : 4 * codebook_wave_smem(K);
}
__device__ __forceinline__ bool codebook_build_wave(const Geom& g, uint32_t* hist_t, uint32_t* hist_view_t, uint16_t* enc_t,
                                                    uint8_t* lens_t, TMeta* tmeta_t, unsigned char* wsm, uint32_t lane,
                                                    uint32_t carry) {
    const uint32_t K = g.K;
    if (g.n >= kWaveElements) return false;  // uniform
    uint64_t* key = reinterpret_cast<uint64_t*>(wsm);            // [64] count << 16 | symbol of the used symbols, symbol order
    uint16_t* ent = reinterpret_cast<uint16_t*>(wsm + 512);      // [K] len << 12 | codeword
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t n_used = 0, n_escape = 0;
    for (uint32_t kb = 0; kb < K; kb += 16u * 64u) {  // sixteen loads of 64 symbols in flight together
        // the counts were added by device-scope atomics of other work-groups, possibly on other dies
        uint32_t hv[16];
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i)
            hv[i] = kb + i * 64u < K ? __hip_atomic_load(&hist_t[kb + i * 64u + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i) {
            const uint32_t k = kb + i * 64u + lane;
            if (kb + i * 64u >= K) continue;  // uniform
            const uint32_t h = hv[i];
            // a codebook that is carried to the next call always has a code for the escape symbol
            const uint32_t c = h + ((carry != 0u && k == 0u) ? 1u : 0u);
            if (hist_t != hist_view_t) hist_view_t[k] = h;  // (the copy itself can be the source: it is left as it is)
            if (kb + i == 0u) n_escape = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
            ent[k] = 0;
            const uint64_t m = __ballot(c != 0u);
            const uint32_t at = n_used + (uint32_t)__popcll(m & below);
            if (c != 0u && at < 64u) key[at] = ((uint64_t)c << 16) | k;
            n_used += (uint32_t)__popcll(m);
        }
    }
    if (n_used > 64u) return false;  // uniform
    if (hist_t != hist_view_t)
        for (uint32_t k0 = 0; k0 < K; k0 += 64)
            __hip_atomic_store(&hist_t[k0 + lane], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_wave_barrier();
    const uint64_t kv = lane < n_used ? key[lane] : ~0ull;  // lane i: the i-th used symbol
    const uint32_t sym = (uint32_t)(kv & 0xFFFFu);
    const uint32_t lo = lane_read(sym, 0), hi = lane_read(sym, n_used ? n_used - 1u : 0u);
    if (n_used >= 2u) {
        const uint32_t len = wave_huffman_lengths(n_used, g.LMAX, (uint32_t)(kv >> 16), lane);
        const uint32_t mine_code = wave_canonical_code(len);
        if (lane < n_used) ent[sym] = (uint16_t)((len << 12) | mine_code);
    }
    __builtin_amdgcn_wave_barrier();
    for (uint32_t k0 = 0; k0 < K; k0 += 64) {
        const uint32_t e = ent[k0 + lane];
        __hip_atomic_store(&enc_t[k0 + lane], (uint16_t)e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lens_t[k0 + lane] = (uint8_t)(e >> 12);
    }
    if (lane == 0) {
        TMeta m;
        m.n_used = n_used;
        m.sym_lo = n_used ? lo : 0u;
        m.sym_hi = n_used ? hi : 0u;
        m.n_outliers = n_escape;  // symbol 0 = escape
        store_tmeta(tmeta_t, m);
    }
    return true;
}

// A work-group of four wavefronts builds the codebooks of the tables [t0, t0 + 4): a wavefront each where the table
// has at most 64 used symbols, the whole work-group one after the other for the rest.
//   smem: codebook_four_smem(K) bytes, 16-byte aligned: the work-group's area, or the wavefronts' areas where those are
//   larger (up to 64 symbols).
// hist_t is read, copied to hist_view_t (inspection) and cleared, so that the next call starts from zero counts.
// enc_t is written with device-scope stores: other work-groups of a running kernel may read it once they have
// seen the caller's completion flag.
// within: another work-group of the same launch reads the lengths, too.
template <uint32_t NT = 256>
__device__ __forceinline__ void codebook_build(const Geom& g, uint32_t* hist_t, uint32_t* hist_view_t, uint16_t* enc_t,
                                               uint8_t* lens_t, TMeta* tmeta_t, unsigned char* smem, CodebookShared& sh,
                                               uint32_t tid, uint32_t carry = 0, bool within = false) {
    const uint32_t K = g.K;
    uint64_t* key = reinterpret_cast<uint64_t*>(smem);        // [K] sort keys: count << 16 | symbol
    uint32_t* cnt = reinterpret_cast<uint32_t*>(key + K);      // [K] counts
    uint32_t* nodew = cnt + K;                                 // [K] merged-node weights, later codewords
    uint16_t* len_s = reinterpret_cast<uint16_t*>(nodew + K);  // [K] code length per symbol
    uint32_t* scratch = reinterpret_cast<uint32_t*>(len_s + K);  // [64]
    const uint32_t lane = tid & 63u, wave = tid >> 6;

    // each thread owns `per` consecutive symbols
    const uint32_t per = (K + NT - 1u) / NT;
    const uint32_t k0 = tid * per, k1 = min(K, k0 + per);
    uint32_t mine = 0;
    // the counts were added by device-scope atomics of other work-groups, possibly on other dies; a thread's loads
    // go out together (an alphabet has at most 4096 symbols)
    constexpr uint32_t kPer = (4096u + NT - 1u) / NT;
    uint32_t hv[kPer];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i)
        hv[i] = k0 + i < k1 ? __hip_atomic_load(&hist_t[k0 + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
        const uint32_t k = k0 + i;
        if (k >= k1) break;
        const uint32_t h = hv[i];
        // a codebook that is carried to the next call always has a code for the escape symbol
        cnt[k] = h + ((carry != 0u && k == 0u) ? 1u : 0u);
        if (hist_t != hist_view_t) {  // (the copy itself can be the source: it is left as it is)
            hist_view_t[k] = h;
            __hip_atomic_store(&hist_t[k], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        len_s[k] = 0;
        mine += cnt[k] != 0;
    }
    // compaction offsets of the used symbols (symbol order); the barriers inside also publish cnt[]
    uint32_t n_used;
    const uint32_t my_off = block_excl_scan<(int)(NT / 64u)>(mine, scratch, tid, &n_used);
    {
        uint32_t o = my_off;
        for (uint32_t k = k0; k < k1; ++k)
            if (cnt[k]) key[o++] = ((uint64_t)cnt[k] << 16) | k;
    }
    __syncthreads();
    // first and last used symbol: the ends of the compacted list
    const uint32_t sym_lo = n_used ? (uint32_t)(key[0] & 0xFFFFu) : 0u;
    const uint32_t sym_hi = n_used ? (uint32_t)(key[n_used - 1] & 0xFFFFu) : 0u;

    const bool by_wave = n_used <= 64u && g.n < kWaveElements;  // uniform
    if (n_used >= 2 && by_wave) {
        if (wave == 0) {
            const uint64_t kv = lane < n_used ? key[lane] : ~0ull;  // lane i: the i-th used symbol
            const uint32_t sym = (uint32_t)(kv & 0xFFFFu);
            const uint32_t len = wave_huffman_lengths(n_used, g.LMAX, (uint32_t)(kv >> 16), lane);
            const uint32_t mine_code = wave_canonical_code(len);
            if (lane < n_used) { len_s[sym] = (uint16_t)len; nodew[sym] = mine_code; }
        }
        __syncthreads();
    } else if (n_used >= 2) {
        const uint32_t n_escape = cnt[0];  // (cnt[] is scratch from here on:
        __syncthreads();                   //  once every thread has read this)
        if (n_used <= NT) {
            // rank sort, a thread per key: the keys are distinct (the symbol is part of them), so a key's place is
            // the number of smaller keys; every thread reads the same key at a time (an LDS broadcast)
            uint64_t* tmp = reinterpret_cast<uint64_t*>(cnt);  // cnt[] and nodew[] together: K words of 64 bits
            uint64_t mykey = 0;
            uint32_t rank = 0;
            if (tid < n_used) {
                mykey = key[tid];
#pragma unroll 8
                for (uint32_t j = 0; j < n_used; ++j) rank += key[j] < mykey ? 1u : 0u;
                tmp[rank] = mykey;
            }
            __syncthreads();
            if (tid < n_used) key[tid] = tmp[tid];
            __syncthreads();
        } else {
            uint32_t P = 2;
            while (P < n_used) P <<= 1;
            for (uint32_t i = n_used + tid; i < P; i += NT) key[i] = ~0ull;  // pad to a power of two
            __syncthreads();
            // bitonic sort, ascending
            for (uint32_t size = 2; size <= P; size <<= 1) {
                for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
                    for (uint32_t i = tid; i < (P >> 1); i += NT) {
                        uint32_t lo = 2 * i - (i & (stride - 1));
                        uint32_t hi = lo + stride;
                        bool up = (lo & size) == 0;
                        uint64_t a = key[lo], bb = key[hi];
                        if ((a > bb) == up) { key[lo] = bb; key[hi] = a; }
                    }
                    __syncthreads();
                }
            }
        }
        // The merge, by one wavefront: 64 leaves and 64 nodes from the heads of the two queues on are in its lanes (the next ones
        // are fetched when fewer than two are left), a step reads two of each and takes the lightest, a leaf where they are alike.
        // What a step found (heads) goes to LDS, 64 steps at a time.  (By one thread, with the queues in LDS, a step was 0.3 us of
        // dependent LDS reads, and depths, limits and codewords took as long again: 26 tables of 4096 x 64 with 83, 170 and 420
        // symbols 72, 106 and 291 us a call, now 63, 87 and 241.)
        uint32_t* const heads = cnt;  // [n_used - 1] leaf << 16 | node
        if (wave == 0) {
            const uint32_t n = n_used, kInf = 0xFFFFFFFFu;
            uint32_t leaf = 0, node = 0, leaf0 = 0, node0 = 0;  // heads, and what lane 0 holds
            auto leaves = [&] { return leaf + lane < n ? (uint32_t)(key[leaf + lane] >> 16) : kInf; };
            uint32_t L = leaves(), N = kInf, seen = 0;
            for (uint32_t k = 0; k + 1u < n; ++k) {
                if (leaf - leaf0 > 62u) { leaf0 = leaf; L = leaves(); }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (nodes that one lane has stored, read by others)
                if (node - node0 > 62u) { node0 = node; N = node + lane < k ? nodew[node + lane] : kInf; }
                const uint32_t l0 = lane_read(L, leaf - leaf0), l1 = lane_read(L, leaf - leaf0 + 1u);
                const uint32_t n0 = lane_read(N, node - node0), n1 = lane_read(N, node - node0 + 1u);
                const uint32_t took = l1 <= n0 ? 0u : (n1 < l0 ? 2u : 1u);  // nodes
                const uint32_t sum = took == 0u ? l0 + l1 : (took == 2u ? n0 + n1 : l0 + n0);
                seen = lane == (k & 63u) ? leaf << 16 | node : seen;
                if ((k & 63u) == 63u) heads[k - 63u + lane] = seen;
                if (lane == 0) nodew[k] = sum;
                N = lane == k - node0 ? sum : N;
                node += took;
                leaf += 2u - took;
            }
            const uint32_t done = (n - 1u) & ~63u;
            if (lane < n - 1u - done) heads[done + lane] = seen;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            // level by level from the root down (see wave_huffman_lengths): lane L counts the leaves of length L
            const uint32_t LM = g.LMAX;
            uint32_t clv = 0, above = n, first = n - 2u, length = 1;
            bool longer = false;
            for (;;) {
                const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)heads[first]);
                clv += lane == min(length, LM) ? above - (at >> 16) : 0u;
                longer = longer || length > LM;
                above = at >> 16;
                if (first == 0u) break;
                first = at & 0xFFFFu;
                ++length;
            }
            if (longer) clv = wave_limit_lengths(clv, LM, lane);
            const uint32_t upto = wave_incl_scan(clv);
            uint32_t code = 0, first_code = 0;
            for (uint32_t l = 1; l <= LM; ++l) {
                code <<= 1;
                first_code = lane == l ? code : first_code;
                code += lane_read(clv, l);
            }
            if (lane <= LM) { sh.more[lane] = upto; sh.first[lane] = first_code; }
        }
        __syncthreads();
        for (uint32_t i = tid; i < n_used; i += NT) {  // lengths are handed out most frequent leaf first (the leaves are sorted by rising count)
            const uint32_t rank = n_used - 1u - i;
            uint32_t l = 1;
            while (l < g.LMAX && rank >= sh.more[l]) ++l;
            len_s[(uint32_t)(key[i] & 0xFFFFu)] = (uint16_t)l;
        }
        __syncthreads();
        if (wave == 0) {  // a symbol's codeword: the first of its length and one for every smaller symbol of that length
            uint32_t next[kLmaxLimit + 1];
#pragma unroll
            for (uint32_t l = 1; l <= (uint32_t)kLmaxLimit; ++l) next[l] = l <= g.LMAX ? (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.first[l]) : 0u;
            for (uint32_t s0 = sym_lo; s0 <= sym_hi; s0 += 64u) {
                const uint32_t l_mine = s0 + lane <= sym_hi ? len_s[s0 + lane] : 0u;
                uint32_t mine_code = 0;
#pragma unroll
                for (uint32_t l = 1; l <= (uint32_t)kLmaxLimit; ++l) {
                    const uint64_t same = __ballot(l_mine == l);
                    mine_code = l_mine == l ? __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, next[l])) : mine_code;
                    next[l] += (uint32_t)__popcll(same);
                }
                if (l_mine != 0u) nodew[s0 + lane] = mine_code;
            }
        }
        if (tid == 0) cnt[0] = n_escape;  // read again at the end
        __syncthreads();
    }
    for (uint32_t k = k0; k < k1; ++k) {
        uint32_t L = len_s[k];
        __hip_atomic_store(&enc_t[k], (uint16_t)(L ? ((L << 12) | nodew[k]) : 0u), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        if (within) __hip_atomic_store(&lens_t[k], (uint8_t)L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else lens_t[k] = (uint8_t)L;
    }
    if (tid == 0) {
        TMeta m;
        // an empty histogram cannot come out of the histogram step (every table has an element); should it
        // happen anyway, the symbol range is still a valid one for the kernels that size things from it
        m.n_used = n_used; m.sym_lo = sym_lo; m.sym_hi = sym_hi; m.n_outliers = cnt[0];  // symbol 0 = escape
        store_tmeta(tmeta_t, m);
    }
    __syncthreads();
}

__device__ __forceinline__ void codebook_build_four(const Geom& g, uint32_t t0, uint32_t* hist, uint32_t* hist_view, uint16_t* enc,
                                                    uint8_t* lens, TMeta* tmeta, unsigned char* smem, CodebookShared& sh,
                                                    uint32_t* slow, uint32_t tid, uint32_t carry) {
    const uint32_t lane = tid & 63u, wave = tid >> 6, t = t0 + wave;
    if (t < g.T) {  // uniform over the wavefront
        const bool done = codebook_build_wave(g, hist + (size_t)t * g.K, hist_view + (size_t)t * g.K, enc + (size_t)t * g.K,
                                              lens + (size_t)t * g.K, tmeta + t, smem + wave * codebook_wave_smem(g.K), lane, carry);
        if (lane == 0) slow[wave] = done ? 0u : 1u;
    } else if (lane == 0) {
        slow[wave] = 0u;
    }
    __syncthreads();
    for (uint32_t w = 0; w < 4; ++w) {
        if (slow[w] == 0u) continue;  // uniform over the work-group
        const uint32_t ts = t0 + w;
        codebook_build(g, hist + (size_t)ts * g.K, hist_view + (size_t)ts * g.K, enc + (size_t)ts * g.K, lens + (size_t)ts * g.K,
                       tmeta + ts, smem, sh, tid, carry);
    }
}

// The codebook of a table whose counts lie in LDS by window index (cnt[254]: the escapes), when it has at most 64 used
// symbols, all of them inside the window; by ONE wavefront.  key: LDS for 64 keys and one that is nobody's; ent[256] (LDS): gets
// len << 12 | codeword by window index.  Returns false, with *tm untouched, when there are more than 64 used symbols.
__device__ __forceinline__ bool codebook_window_wave(const Geom& g, const uint32_t* cnt, uint64_t* key, uint16_t* ent,
                                                     TMeta* tm, uint32_t lane) {
    const uint32_t win_lo = win_lo_of(g.R);
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t n_escape = (uint32_t)__builtin_amdgcn_readfirstlane((int)cnt[kWinEsc]);
    uint32_t n_used = n_escape ? 1u : 0u;  // the escape is symbol 0: the first in symbol order
    uint32_t cv[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) cv[i] = i * 64u + lane < kWinEsc ? cnt[i * 64u + lane] : 0u;
    key[n_escape && lane == 0 ? 0u : 64u] = ((uint64_t)n_escape << 16) | kWinEsc;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        const uint64_t m = __ballot(cv[i] != 0u);
        const uint32_t at = n_used + (uint32_t)__popcll(m & below);
        key[cv[i] != 0u ? min(at, 64u) : 64u] = ((uint64_t)cv[i] << 16) | (i * 64u + lane);
        n_used += (uint32_t)__popcll(m);
    }
    if (n_used > 64u) return false;  // uniform
    reinterpret_cast<uint64_t*>(ent)[lane] = 0ull;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t kv = lane < n_used ? key[lane] : ~0ull;  // lane i: the i-th used symbol
    const uint32_t idx = (uint32_t)(kv & 0xFFFFu);
    if (n_used >= 2u) {
        const uint32_t len = wave_huffman_lengths(n_used, g.LMAX, (uint32_t)(kv >> 16), lane);
        const uint32_t code = wave_canonical_code(len);
        if (lane < n_used) ent[idx] = (uint16_t)((len << 12) | code);
    }
    const uint32_t sym = idx == kWinEsc ? 0u : win_lo + idx;
    const uint32_t lo = lane_read(sym, 0), hi = (uint32_t)__builtin_amdgcn_readlane((int)sym, (int)(n_used ? n_used - 1u : 0u));
    if (lane == 0) {
        TMeta m;
        m.n_used = n_used;
        m.sym_lo = n_used ? lo : 0u;
        m.sym_hi = n_used ? hi : 0u;
        m.n_outliers = n_escape;
        *tm = m;
    }
    return true;
}

// ------------------------------------------------------------------------------------------------
// offsets of the output: single-pass look-back scan
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kFlagAgg = 1, kFlagPrefix = 2;
constexpr uint32_t kSpinLimit = 1u << 22;

// Tells other work-groups of the launch that a table has its codebook in memory (one thread, after every wavefront that stored some
// of it has waited for its stores).
__device__ __forceinline__ void table_ready(uint32_t* ready, uint64_t epoch, uint32_t t) {
    __hip_atomic_store(&ready[t], (uint32_t)epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive prefix of `total` over the work-groups before `wg`: single-pass look-back over one record per
// work-group, 256 records per step (four per lane).  The chain of "wait for a predecessor's prefix" steps across
// the work-groups that run at the same time is what bounds a streaming kernel that places its output by such a
// scan, so the records are few and the steps wide.  Publishes this work-group's records.  Called by one whole
// wavefront.
// dom0: the first work-group of this work-group's scan domain (a destination's container: offsets start at 0 there).
__device__ __forceinline__ uint32_t wg_scan(uint64_t* state, uint64_t epoch, uint32_t wg, uint32_t total, uint32_t lane,
                                            Ctrl* ctrl, bool* dead, uint32_t dom0 = 0) {
    const uint64_t tag = epoch << 34;
    if (lane == 0)
        __hip_atomic_store(&state[wg], tag | ((uint64_t)(wg == dom0 ? kFlagPrefix : kFlagAgg) << 32) | total,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t excl = 0;
    if (wg > dom0) {
        int64_t pos = (int64_t)wg - 1;  // nearest record not yet added
        uint32_t spins = 0;
        for (;;) {
            // this lane's four records, nearest first; before the first work-group: an empty prefix
            uint32_t sum = 0;       // values up to and including the lane's first prefix record (or all four)
            bool has_p = false;     // there is a prefix record among them
            bool hole = false;      // an unpublished record comes before it
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t my = pos - (int64_t)(lane * 4u + (uint32_t)k);
                const uint64_t sv = my >= (int64_t)dom0 ? __hip_atomic_load(&state[my], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                                        : (tag | ((uint64_t)kFlagPrefix << 32));
                const uint32_t flag = (sv >> 34) == epoch ? (uint32_t)(sv >> 32) & 3u : 0u;
                if (!has_p) {
                    hole = hole || flag == 0u;
                    sum += flag != 0u ? (uint32_t)sv : 0u;
                    has_p = flag == kFlagPrefix;
                }
            }
            const uint64_t pm = __ballot(has_p);
            const uint32_t first = pm ? (uint32_t)__ffsll((unsigned long long)pm) - 1u : 64u;  // lane of the nearest prefix
            if (__ballot(hole && lane <= first) != 0ull) {  // something nearer than that prefix is not published yet
                if (++spins > kSpinLimit) {  // never expected; the bound only guarantees termination
                    if (lane == 0) { set_status(ctrl, DLC_ESTATE); atomicOr(&ctrl->abort, 1u); }
                    *dead = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
            excl += wave_sum(lane <= first ? sum : 0u);
            if (pm) break;
            pos -= 256;
        }
        if (lane == 0 && !*dead)
            __hip_atomic_store(&state[wg], tag | ((uint64_t)kFlagPrefix << 32) | (uint32_t)(excl + total),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return excl;
}

// escape records of one group, in increasing element index, behind its chunk words, for a group with more escapes
// than the encode kernel remembers on the way: a rolled loop over the group's plane words (index 254 marks an
// escape; an element of a row that is stored as a reference has index 253 and no record) and, for the raw bits,
// over its elements
template <int S, bool F16, bool VEC>
__device__ __forceinline__ void emit_escapes(uint32_t* rec, uint32_t lane, const uint8_t* gbase, const uint32_t* plane_g,
                                             uint32_t gstart, uint32_t rem) {
    uint32_t opos = 0;
    for (uint32_t j = 0; j < (uint32_t)S / kV; ++j) {
        const uint32_t off = lane * kV + j * (kW * kV);
        float x[4];
        uint32_t raw[4];
        const uint32_t valid = load4<F16, VEC>(gbase, off, rem, x, raw);
        const uint32_t m = plane_g[j * kW + lane];
        uint32_t esc = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            esc |= (((valid >> v) & 1u) && ((m >> (8 * v)) & 0xFFu) == kWinEsc) ? (1u << v) : 0u;
        if (__ballot(esc != 0u) == 0ull) continue;
        const uint32_t cnt = __popc(esc);
        const uint32_t incl = wave_incl_scan(cnt);
        uint32_t r = opos + incl - cnt;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if ((esc >> v) & 1u) {
                rec[2u * r] = gstart + off + v;
                rec[2u * r + 1] = raw[v];
                ++r;
            }
        opos += __shfl(incl, 63, 64);
    }
}

}  // namespace dlc
