// Statistics reduction for gfx950: per-table value range and exact distinct-row counts of the raw rows
// and of the rows quantised at a probe bound (the two counts of the Homogenization Index, Eq. 1).
//
// k_stats_init sets an attempt up.  k_stats_hash: two 64-bit hashes per row (raw bits; symbols at the probe bound) and the range.
// The row sets (dlc_rowmatch.hip: the rows of a table divided among work-groups by hash, open-addressing sets in
// LDS, the smallest row index of a hash owns it) give every row the owner of its hash and count the owners.
// k_stats_verify: every row that is not an owner is compared with its owner element by element, so a hash
// collision between different rows is detected (the host then repeats the reduction with another hash salt) and
// the counts are exact.
#include <algorithm>

#include "dlc_internal.h"

namespace dlc {

namespace {

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

__device__ __forceinline__ uint32_t mix32(uint32_t z) {
    z ^= z >> 16; z *= 0x85EBCA6Bu;
    z ^= z >> 13; z *= 0xC2B2AE35u;
    z ^= z >> 16;
    return z;
}

// float <-> unsigned with the same ordering
__device__ __forceinline__ uint32_t ord_enc(float f) {
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

template <bool F16>
__device__ __forceinline__ float elem_value(uint32_t raw) {
    if constexpr (F16) return __half2float(__ushort_as_half((unsigned short)raw));
    else return __uint_as_float(raw);
}

}  // namespace

namespace {

constexpr uint32_t kStPieces = 4;   // 16-byte pieces of a row that one load instruction of a wavefront takes: 64 bytes of each of 16 rows
constexpr uint32_t kStRows = 16;    // rows of a wavefront's matrix product
constexpr uint32_t kStSteps = 4;    // row sets of a wavefront whose loads the verify kernel issues back to back

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_row __attribute__((ext_vector_type(4), aligned(2)));  // a piece on an element's boundary

// The range of finite values as bit patterns.  Positive numbers rise with their patterns, negative ones fall, so the
// largest unsigned pattern is the least number if it has the sign, the least unsigned pattern the least number if none
// has, and the largest signed pattern the largest number unless all have it.  Three whole-number operations for two
// elements and no test of NaN: what is not finite shows in the two maxima afterwards.
struct StRange {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    int32_t top = (int32_t)0x80000000u;
    __device__ __forceinline__ void add(uint32_t b) { lo = min(lo, b); hi = max(hi, b); top = max(top, (int32_t)b); }
    __device__ __forceinline__ void add(const StRange& r) { lo = min(lo, r.lo); hi = max(hi, r.hi); top = max(top, r.top); }
    __device__ __forceinline__ bool finite() const { return hi < 0xFF800000u && top < 0x7F800000; }
    __device__ __forceinline__ bool none() const { return lo == 0xFFFFFFFFu; }  // (the pattern of a NaN)
    __device__ __forceinline__ uint32_t min_ord() const { return none() ? 0xFFFFFFFFu : ord_enc(__uint_as_float((hi >> 31) ? hi : lo)); }
    __device__ __forceinline__ uint32_t max_ord() const { return none() ? 0u : ord_enc(__uint_as_float((lo >> 31) ? lo : (uint32_t)top)); }
};

// element k of a piece as a binary32 number
template <bool F16>
__device__ __forceinline__ float st_piece_value(const i32x4& a, uint32_t k) {
    if constexpr (F16) return elem_value<true>(((uint32_t)a[k >> 1] >> (16u * (k & 1u))) & 0xFFFFu);
    else return __uint_as_float((uint32_t)a[k]);
}

}  // namespace

// start of an attempt: the coefficients of every byte of a row for this attempt's salt (`n_mult` words); the
// call's bounds from the host's memory; the counts of distinct rows and the collision counter cleared
__global__ __launch_bounds__(256) void k_stats_init(uint32_t* mult, uint32_t n_mult, uint32_t salt, uint32_t* unique,
                                                    uint32_t T, const QParam* host_probe, QParam* probe, Ctrl* ctrl) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n_mult) mult[i] = mix32((i + 1u) * 0x9E3779B1u + salt);
    if (i < 2u * T) unique[i] = 0u;
    if (i < T) probe[i] = host_probe[i];
    if (i == 0) ctrl->collide = 0u;
}

// pass 1: range, and two hashes of every row.  A hash is a product of a matrix of random bytes (16 functions by the bytes
// of a row) and the rows' bytes, on the matrix cores: i32_16x16x64_i8 takes 64 bytes of each of 16 rows, and its operand
// is what a 16-byte load per lane brings (lane l: row l % 16, piece l / 16), so a row's elements are not moved between
// lanes at all.  The symbols at the probe bound go the same way, as 16-bit numbers.  Two rows that differ agree in one
// function with a probability of 2^-8 at most (whatever else is in them: for one value of a differing byte's coefficient at
// most; in rows of up to 256 KiB, whose coefficients are all their own).  Four functions of a lane, each a byte further up, make
// a 32-bit number, in which they agree with 2^-25 at most (a byte that differs by 128, as the sign of an element does, leaves
// its lowest seven bits as they are), four lanes' numbers the hash.  The counts do not hang on it: rows are compared afterwards.
// Which bytes a coefficient meets is free as long as it is the same for all rows: a piece past the row's end, or the
// part of the last piece that is, is replaced by the row's last 16 bytes (elements that come twice change neither the
// range nor the bound on the probability), and a row past the batch's end by the last one.  Nothing is masked.
// NS: load instructions (steps) of one chunk; a row of more than 8 steps takes several chunks (!ONE), with the
// coefficients loaded for each.  WIDE: a row has 16 bytes or more.
// What bounds it: the payload's way from memory (512 MiB read in 80 us by a kernel that does nothing else). 128 tables of
// 8192 x 128: 97 us; the form before, a lane per row with the rows turned in LDS and 50 instructions an element (12 now),
// 193. The next rows' loads are under way while a wavefront works on the present ones (without: 159), and three wavefronts a
// SIMD with their operands in registers are faster than four (100 against 111). 16 work-groups of a table, not 32: 121.
template <bool F16, bool WIDE, uint32_t NS, bool ONE>
__global__ __launch_bounds__(256, F16 && NS >= 7u ? 2 : 3) void k_stats_hash(const void* payload, Geom g, const QParam* probe, const i32x4* __restrict__ mult,
                                                    uint64_t* rowhash, uint32_t* part_range, uint32_t waves_grid, uint32_t steps) {
    constexpr uint32_t kElems = F16 ? 8u : 4u;               // elements of a piece
    constexpr uint32_t kSets = 64u / kStRows;                // row sets of a wavefront's 64 rows
    constexpr uint32_t RS = NS > 4u ? 1u : (NS > 2u ? 2u : 4u);  // sets whose loads are issued back to back
    constexpr uint32_t kSymStep = F16 ? 1u : 2u;             // steps whose symbols fill an operand
    constexpr uint32_t kTrips = kSets / RS;                  // trips of a wavefront's 64 rows
    __shared__ uint32_t words[4][kSets][2][64];
    __shared__ i32x4 coef[ONE ? NS * 64u : 1u];
    const uint32_t t = blockIdx.y;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t wave_global = blockIdx.x * 4 + wave;
    if constexpr (ONE) {
        for (uint32_t k = threadIdx.x; k < NS * 64u; k += 256u) coef[k] = mult[min(k, steps * 64u - 1u)];
        __syncthreads();
    }
    const QParam q = probe[t];
    const float Rf = (float)g.R;
    const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
    typedef std::conditional_t<ONE, uint32_t, size_t> Off;  // (rows of one chunk are 512 bytes at most)
    const Off row_bytes = (Off)g.D * g.es;
    const uint32_t lrow = lane & (kStRows - 1u), lpiece = lane / kStRows;
    StRange total;
    struct Pieces { i32x4 v[RS][NS]; };
    Pieces a[2];  // !ONE: the first only
    auto load = [&](Pieces& a, uint32_t row0, uint32_t trip, uint32_t c) {
        const uint32_t last = g.B - 1u - row0;  // the batch's last row, counted from the first of these
        const uint8_t* base = tab + (size_t)row0 * row_bytes;
#pragma unroll
        for (uint32_t r = 0; r < RS; ++r) {
            const Off off = (Off)min((trip * RS + r) * kStRows + lrow, last) * row_bytes;
#pragma unroll
            for (uint32_t s = 0; s < NS; ++s) {
                if constexpr (WIDE) {
                    const Off at = min(((Off)(c + s) * kStPieces + lpiece) * 16u, row_bytes - 16u);
                    const u32x4_row w = *reinterpret_cast<const u32x4_row*>(base + off + at);
                    a.v[r][s] = i32x4{(int)w.x, (int)w.y, (int)w.z, (int)w.w};
                } else if constexpr (F16) {
                    const uint16_t* e = reinterpret_cast<const uint16_t*>(base + off);
#pragma unroll
                    for (uint32_t k = 0; k < 4u; ++k)
                        a.v[r][s][k] = (int)((uint32_t)e[min(2u * k, g.D - 1u)] | (uint32_t)e[min(2u * k + 1u, g.D - 1u)] << 16);
                } else {
                    const uint32_t* e = reinterpret_cast<const uint32_t*>(base + off);
#pragma unroll
                    for (uint32_t k = 0; k < 4u; ++k) a.v[r][s][k] = (int)e[min(k, g.D - 1u)];
                }
            }
        }
    };
    if constexpr (ONE) {
        if (wave_global * 64u < g.B) load(a[0], wave_global * 64u, 0u, 0u);
    }
    for (uint32_t row0 = wave_global * 64u; row0 < g.B; row0 += waves_grid * 64u) {
        i32x4 hr[RS], hq[RS];
        auto add = [&](const Pieces& a, const i32x4* m, uint32_t m_step, uint32_t trip, uint32_t c) {
#pragma unroll
            for (uint32_t r = 0; r < RS; ++r) {
                StRange part;
                i32x4 sym = {0, 0, 0, 0};
#pragma unroll
                for (uint32_t s = 0; s < NS; ++s) {
                    if (ONE || c + s < steps) {  // (uniform)
                        hr[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[s * m_step], a.v[r][s], hr[r], 0, 0, 0);
#pragma unroll
                        for (uint32_t k = 0; k < kElems; k += 2u) {
                            const float x0 = st_piece_value<F16>(a.v[r][s], k), x1 = st_piece_value<F16>(a.v[r][s], k + 1u);
                            part.add(__float_as_uint(x0));
                            part.add(__float_as_uint(x1));
                            const uint32_t c0 = quant_symbol<F16>(x0, q, Rf, (int)g.R), c1 = quant_symbol<F16>(x1, q, Rf, (int)g.R);
                            sym[(s % kSymStep) * 2u + k / 2u] = (int)(c0 | c1 << 16);
                        }
                        if constexpr (F16) hq[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[s * m_step], sym, hq[r], 0, 0, 0);
                    }
                    if constexpr (!F16) {
                        if (s % 2u == 1u || s + 1u == NS) {
                            if (ONE || c + (s & ~1u) < steps) hq[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[(s & ~1u) * m_step], sym, hq[r], 0, 0, 0);
                            sym = i32x4{0, 0, 0, 0};
                        }
                    }
                }
                if (__builtin_expect(__ballot(!part.finite()) != 0ull, 0)) {  // element by element, without what is not finite
                    part = StRange();
                    const uint8_t* base = tab + (size_t)row0 * row_bytes;
                    const Off off = (Off)min((trip * RS + r) * kStRows + lrow, g.B - 1u - row0) * row_bytes;
#pragma unroll 1
                    for (uint32_t s = 0; s < NS; ++s) {
#pragma unroll 1
                        for (uint32_t k = 0; k < kElems; ++k) {
                            // (loaded again: a register cannot be picked by a number that is not a constant)
                            const Off at = WIDE ? min(((Off)(c + s) * kStPieces + lpiece) * 16u, row_bytes - 16u) / g.es + k : min(k, g.D - 1u);
                            const uint32_t raw = F16 ? (uint32_t)reinterpret_cast<const uint16_t*>(base + off)[at] : reinterpret_cast<const uint32_t*>(base + off)[at];
                            const uint32_t b = __float_as_uint(elem_value<F16>(raw));
                            if ((b & 0x7F800000u) != 0x7F800000u) part.add(b);
                        }
                    }
                }
                total.add(part);
            }
        };
        auto hand_on = [&](uint32_t trip) {
#pragma unroll
            for (uint32_t r = 0; r < RS; ++r) {
                words[wave][trip * RS + r][0][lane] = (uint32_t)hr[r][0] + ((uint32_t)hr[r][1] << 8) + ((uint32_t)hr[r][2] << 16) + ((uint32_t)hr[r][3] << 24);
                words[wave][trip * RS + r][1][lane] = (uint32_t)hq[r][0] + ((uint32_t)hq[r][1] << 8) + ((uint32_t)hq[r][2] << 16) + ((uint32_t)hq[r][3] << 24);
            }
        };
        if constexpr (ONE) {
#pragma unroll
            for (uint32_t trip = 0; trip < kTrips; ++trip) {
                // the rows of the next trip are on their way while these are worked on (past the batch's end: the last row)
                if (trip + 1u < kTrips) load(a[(trip + 1u) & 1u], row0, trip + 1u, 0u);
                else if (row0 + waves_grid * 64u < g.B) load(a[(trip + 1u) & 1u], row0 + waves_grid * 64u, 0u, 0u);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (uint32_t r = 0; r < RS; ++r) hr[r] = hq[r] = i32x4{0, 0, 0, 0};
                add(a[trip & 1u], coef + lane, 64u, trip, 0u);
                hand_on(trip);
            }
            if constexpr (kTrips % 2u == 1u) a[0] = a[1];
        } else {
#pragma unroll 1
            for (uint32_t trip = 0; trip < kTrips; ++trip) {
                for (uint32_t r = 0; r < RS; ++r) hr[r] = hq[r] = i32x4{0, 0, 0, 0};
                for (uint32_t c = 0; c < steps; c += NS) {
                    i32x4 m[NS];
                    load(a[0], row0, trip, c);
#pragma unroll
                    for (uint32_t s = 0; s < NS; ++s) m[s] = mult[min((c + s) % kStMultSteps, steps - 1u) * 64u + lane];
                    if (c >= kStMultSteps) {  // (uniform) past the table: its coefficients again, each other by a part of its own
                        i32x4 x = mult[lane];
#pragma unroll
                        for (uint32_t k = 0; k < 4u; ++k) x[k] = (int)mix32((uint32_t)x[k] + (c / kStMultSteps) * 0x9E3779B1u);
#pragma unroll
                        for (uint32_t s = 0; s < NS; ++s) m[s] ^= x;
                    }
                    add(a[0], m, 1u, trip, c);
                }
                hand_on(trip);
            }
        }
        // the words come from other lanes of this wavefront: its LDS accesses complete in order, the compiler
        // must keep them in order too
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t row = row0 + lane;
        if (row < g.B) {
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                const uint32_t* p = words[wave][lane / kStRows][k] + lrow;
                const uint32_t w2 = p[2 * kStRows], w3 = p[3 * kStRows];
                const uint32_t lo = p[0] + (w2 << 16 | w2 >> 16), hi = p[kStRows] + (w3 << 16 | w3 >> 16);
                rowhash[((size_t)k * g.T + t) * g.B + row] = mix64(((uint64_t)hi << 32) | lo);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // the work-group's range, as order-preserving integers; k_stats_result puts a table's together (atomics of all wavefronts
    // on the tables' words, which share a few cache lines, took 50 us)
    uint32_t mn = total.min_ord(), mx = total.max_ord();
    for (int o = 32; o > 0; o >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor(mn, o, 64));
        mx = max(mx, (uint32_t)__shfl_xor(mx, o, 64));
    }
    __syncthreads();
    if (lane == 0) { words[0][0][0][wave] = mn; words[0][0][1][wave] = mx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t* a = words[0][0][0];
        const uint32_t* b = words[0][0][1];
        uint2* out = reinterpret_cast<uint2*>(part_range) + (size_t)t * gridDim.x + blockIdx.x;
        *out = make_uint2(min(min(a[0], a[1]), min(a[2], a[3])), max(max(b[0], b[1]), max(b[2], b[3])));
    }
}

namespace {

// a lane's piece of a row: NW words (16 bytes where the row length allows, else one element in one word)
template <uint32_t NW>
struct StPiece { uint32_t v[NW]; };

template <bool F16, uint32_t NW>
__device__ __forceinline__ StPiece<NW> st_load_piece(const uint8_t* tab, size_t piece) {
    StPiece<NW> r;
    if constexpr (NW == 4) {
        const uint4 x = *reinterpret_cast<const uint4*>(tab + piece * 16u);
        r.v[0] = x.x; r.v[1] = x.y; r.v[2] = x.z; r.v[3] = x.w;
    } else if constexpr (F16) {
        r.v[0] = reinterpret_cast<const uint16_t*>(tab)[piece];
    } else {
        r.v[0] = reinterpret_cast<const uint32_t*>(tab)[piece];
    }
    return r;
}

// do two words (of different bits) hold elements with different symbols?
template <bool F16, uint32_t NW>
__device__ __forceinline__ bool st_symbols_differ(uint32_t a, uint32_t b, const QParam& q, float Rf, int R) {
    if constexpr (F16 && NW == 4) {  // two elements per word
        return quant_symbol<true>(elem_value<true>(a & 0xFFFFu), q, Rf, R) != quant_symbol<true>(elem_value<true>(b & 0xFFFFu), q, Rf, R) ||
               quant_symbol<true>(elem_value<true>(a >> 16), q, Rf, R) != quant_symbol<true>(elem_value<true>(b >> 16), q, Rf, R);
    } else {
        return quant_symbol<F16>(elem_value<F16>(a), q, Rf, R) != quant_symbol<F16>(elem_value<F16>(b), q, Rf, R);
    }
}

}  // namespace

// pass 2: every row that does not own its hash must equal the owner: in its bits for the raw rows, in its symbols for
// the quantised rows (only the elements whose bits differ need the quantiser).  A row is the work of a team of
// 2^logL lanes, the smallest power of two that covers the row's pieces (64 at most: longer rows take several
// trips); a wavefront works on 64 rows per trip: those that do not own their hash are put next to one another, 64 >> logL are
// compared at a time, kStSteps times with the loads issued back to back.  own: [2][T][B], raw then quantised.
// What bounds it: two rows read for each of them (128 tables of 8192 x 128, of which 55 % repeat: 590 MB, half of it rows
// that others refer to as well) in 65 us.  With all 64 rows walked, the idle ones under a condition: 94.
template <bool F16, uint32_t NW>
__global__ __launch_bounds__(256) void k_stats_verify(const void* payload, Geom g, const QParam* probe, const uint32_t* own,
                                                      Ctrl* ctrl, TableOrder order, uint32_t logL) {
    uint32_t t, block;
    order.place(&t, &block);
    if (t >= g.T) return;  // uniform
    const uint32_t waves_grid = order.bx * 4u;
    t = g.T - 1u - t;  // (the tables that the pass before read last first: 128 tables of 8192 x 128 100 us, so 94)
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave_global = block * 4 + (threadIdx.x >> 6);
    const QParam q = probe[t];
    const float Rf = (float)g.R;
    const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
    const uint32_t W = NW == 4 ? (uint32_t)((size_t)g.D * g.es / 16u) : g.D;  // pieces per row
    const uint32_t L = 1u << logL, sub = lane & (L - 1u), team = lane >> logL, rps = 64u >> logL;
    const size_t row_bytes = (size_t)g.D * g.es;
    bool differ = false;
    for (uint32_t row0 = wave_global * 64u; row0 < g.B; row0 += waves_grid * 64u) {
        // the rows with `need` set are put next to one another and compared with the row `other` of each, all by all teams;
        // `raw`: in their bits, else in their symbols
        auto compare = [&](bool need, uint32_t other, bool raw) {
            const uint64_t mask = __ballot(need);
            const uint32_t n = (uint32_t)__popcll(mask);
            if (n == 0u) return;
            const uint32_t rank = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
            const int to = (int)((need ? rank : n + lane - rank) << 2);
            const uint32_t list_row = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)lane);
            const uint32_t list_other = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(other | (raw ? 0x80000000u : 0u)));  // (a row's index has 31 bits)
            for (uint32_t i0 = 0; i0 < n; i0 += rps * kStSteps) {
                const uint8_t* pa[kStSteps];
                const uint8_t* pb[kStSteps];
                bool in[kStSteps], bits[kStSteps];
#pragma unroll
                for (uint32_t s = 0; s < kStSteps; ++s) {
                    const uint32_t i = i0 + s * rps + team;
                    in[s] = i < n;
                    const uint32_t k = in[s] ? i : 0u;
                    const uint32_t r = (uint32_t)__shfl((int)list_row, (int)k, 64), o = (uint32_t)__shfl((int)list_other, (int)k, 64);
                    bits[s] = (o >> 31) != 0u;
                    pa[s] = tab + (size_t)(row0 + r) * row_bytes;
                    pb[s] = tab + (size_t)(o & 0x7FFFFFFFu) * row_bytes;
                }
                for (uint32_t p = sub; p < W; p += L) {
                    StPiece<NW> a[kStSteps], b[kStSteps];
#pragma unroll
                    for (uint32_t s = 0; s < kStSteps; ++s) {  // (past the list: its first row, read and not looked at)
                        a[s] = st_load_piece<F16, NW>(pa[s], p);
                        b[s] = st_load_piece<F16, NW>(pb[s], p);
                    }
#pragma unroll
                    for (uint32_t s = 0; s < kStSteps; ++s) {
                        uint32_t x = 0u;
#pragma unroll
                        for (uint32_t k = 0; k < NW; ++k) x |= a[s].v[k] ^ b[s].v[k];
                        if (x != 0u && in[s]) {
                            bool d = bits[s];
#pragma unroll
                            for (uint32_t k = 0; k < NW; ++k)
                                if (!d && a[s].v[k] != b[s].v[k]) d = st_symbols_differ<F16, NW>(a[s].v[k], b[s].v[k], q, Rf, (int)g.R);
                            differ |= d;
                        }
                    }
                }
            }
        };
        const uint32_t row = row0 + lane;
        const uint32_t own_r = row < g.B ? own[(size_t)t * g.B + row] : 0xFFFFFFFFu, own_q = row < g.B ? own[((size_t)g.T + t) * g.B + row] : 0xFFFFFFFFu;
        const bool need_r = own_r < row, need_q = own_q < row;  // (an owner is never a later row)
        compare(need_r || need_q, need_r ? own_r : own_q, need_r);
        // rows with two owners: equal in their bits to the one is equal in their symbols too
        compare(need_r && need_q && own_q != own_r, own_q, false);
    }
    if (__ballot(differ) != 0ull && lane == 0) atomicAdd(&ctrl->collide, 1u);
}

// the results, into the host's memory: the range of every table from its `parts` work-groups', a wavefront a table; its
// counts; behind them the two words of the control block that the host wants
__global__ __launch_bounds__(64) void k_stats_result(const Ctrl* ctrl, const uint32_t* part_range, uint32_t parts, const uint32_t* unique,
                                                     uint32_t T, uint32_t* out) {
    const uint32_t t = blockIdx.x, lane = threadIdx.x;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    for (uint32_t k = lane; k < parts; k += 64u) {
        const uint2 r = reinterpret_cast<const uint2*>(part_range)[(size_t)t * parts + k];
        mn = min(mn, r.x);
        mx = max(mx, r.y);
    }
    for (int o = 32; o > 0; o >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor(mn, o, 64));
        mx = max(mx, (uint32_t)__shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
        reinterpret_cast<uint2*>(out)[t] = make_uint2(mn, mx);
        reinterpret_cast<uint2*>(out)[(size_t)T + t] = reinterpret_cast<const uint2*>(unique)[t];
        if (t == 0) reinterpret_cast<uint2*>(out)[2 * (size_t)T] = make_uint2(ctrl->collide, (uint32_t)ctrl->status);
    }
}

hipError_t launch_stats(const Geom& g, const void* payload, const Ws& w, uint32_t salt, hipStream_t s) {
    const QParam* probe = w.probe;
    const uint32_t blocks_x = std::min<uint32_t>((g.B + 255u) / 256u, kStatsBlocks);  // a wavefront takes 64 rows at a time
    const uint32_t waves_grid = blocks_x * 4;
    dim3 grid(blocks_x, g.T), block(256);
    const uint32_t steps = stats_steps(g), n_mult = stats_mult_steps(g) * 256u;
    hipLaunchKernelGGL(k_stats_init, dim3((std::max(n_mult, 2u * g.T) + 255u) / 256u), block, 0, s, w.st_mult, n_mult, salt,
                       w.st_unique, g.T, w.st_pin_probe, w.probe, w.ctrl);
#define DLC_ST_HASH(FF, WIDE, NS, ONE) hipLaunchKernelGGL((k_stats_hash<FF, WIDE, NS, ONE>), grid, block, 0, s, payload, g, probe, reinterpret_cast<const i32x4*>(w.st_mult), w.rowhash, w.st_range, waves_grid, steps)
#define DLC_ST_HASH_STEPS(FF) do { \
        if (g.D * g.es < 16u) DLC_ST_HASH(FF, false, 1, true); \
        else if (steps == 1u) DLC_ST_HASH(FF, true, 1, true); \
        else if (steps == 2u) DLC_ST_HASH(FF, true, 2, true); \
        else if (steps == 3u) DLC_ST_HASH(FF, true, 3, true); \
        else if (steps == 4u) DLC_ST_HASH(FF, true, 4, true); \
        else if (steps == 5u) DLC_ST_HASH(FF, true, 5, true); \
        else if (steps == 6u) DLC_ST_HASH(FF, true, 6, true); \
        else if (steps == 7u) DLC_ST_HASH(FF, true, 7, true); \
        else if (steps == 8u) DLC_ST_HASH(FF, true, 8, true); \
        else DLC_ST_HASH(FF, true, 8, false); \
    } while (0)
    if (g.dtype == DLC_F16) DLC_ST_HASH_STEPS(true);
    else DLC_ST_HASH_STEPS(false);
#undef DLC_ST_HASH_STEPS
#undef DLC_ST_HASH
    hipError_t e = launch_row_sets(g, 2u, nullptr, w.rowhash, w.st_own, w.st_unique, w.ctrl, s);
    if (e != hipSuccess) return e;
    const bool vec = ((size_t)g.D * g.es) % 16u == 0u;
    const uint32_t pieces = vec ? (uint32_t)((size_t)g.D * g.es / 16u) : g.D;
    uint32_t logL = 0;
    while (logL < 6 && (1u << logL) < pieces) ++logL;
    // tables apart and one after the other, us: one of 65536 rows 49 and 48; 9, 12, 15, 26, 64 and 128 of 8192 x 128 8.8 and 8.4, 9.8
    // and 9.0, 9.9 and 11.2, 16.5 and 17.8, 32 and 38, 67 and 76; of few rows it is all the same or better apart (the call with five
    // of 2048 x 64 38.8 and 39.8)
    const TableOrder order(blocks_x, g.T > 12u || blocks_x <= 8u);
#define DLC_ST_VERIFY(FF, NW) hipLaunchKernelGGL((k_stats_verify<FF, NW>), dim3(order.groups(g.T)), block, 0, s, payload, g, probe, w.st_own, w.ctrl, order, logL)
    if (g.dtype == DLC_F16) { if (vec) DLC_ST_VERIFY(true, 4); else DLC_ST_VERIFY(true, 1); }
    else { if (vec) DLC_ST_VERIFY(false, 4); else DLC_ST_VERIFY(false, 1); }
#undef DLC_ST_VERIFY
    hipLaunchKernelGGL(k_stats_result, dim3(g.T), dim3(64), 0, s, w.ctrl, w.st_range, blocks_x, w.st_unique, g.T, w.st_pin);
    return hipGetLastError();
}

}  // namespace dlc
