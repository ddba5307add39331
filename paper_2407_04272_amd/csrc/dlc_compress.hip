// Compression kernels for gfx950: quantise + histogram, Huffman codebook, bit-packed encode with
// scanned offsets, finalize.
//
// Mapping used by the streaming kernels: one wavefront owns one group of 64*S symbols; lane l owns
// chunk l of the group and, at turn j, the four symbols  group_base + j*256 + 4*l .. +3  (one 16-byte
// load per lane, 1 KiB contiguous per wavefront instruction).
#include <algorithm>

#include "dlc_codec_dev.h"
#include "dlc_finalize.h"

namespace dlc {

bool launch_encode_64(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                      uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
bool launch_table_64(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                     uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
bool launch_flow_64(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                    uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
hipError_t encode_set_attributes_64();
bool launch_encode_128(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                      uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
bool launch_table_128(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                     uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
bool launch_flow_128(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                    uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
hipError_t encode_set_attributes_128();
bool launch_encode_256(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                      uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
bool launch_table_256(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                     uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
bool launch_flow_256(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                    uint64_t capacity, uint64_t* out_bytes, hipStream_t s);
hipError_t encode_set_attributes_256();
void launch_encode_carry_64(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                            uint64_t capacity, uint32_t bpt, hipStream_t s);
void launch_encode_carry_128(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                             uint64_t capacity, uint32_t bpt, hipStream_t s);
void launch_encode_carry_256(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch, uint8_t* out,
                             uint64_t capacity, uint32_t bpt, hipStream_t s);

// ------------------------------------------------------------------------------------------------
// quantiser alone (inspection entry point)
// ------------------------------------------------------------------------------------------------
template <bool F16>
__global__ __launch_bounds__(256) void k_quantize(const void* payload, Geom g, const QParam* qp, uint16_t* sym) {
    const uint32_t t = blockIdx.y;
    const QParam q = qp[t];
    const float Rf = (float)g.R;
    const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < g.n; i += gridDim.x * blockDim.x) {
        float x;
        if constexpr (F16) x = __half2float(__ushort_as_half(reinterpret_cast<const unsigned short*>(tab)[i]));
        else x = reinterpret_cast<const float*>(tab)[i];
        sym[(size_t)t * g.n + i] = (uint16_t)quant_symbol<F16>(x, q, Rf, (int)g.R);
    }
}

hipError_t launch_quantize(const Geom& g, const void* payload, const QParam* qp, uint16_t* sym, hipStream_t s) {
    dim3 grid(std::min<uint32_t>((g.n + 255) / 256, 1024), g.T);
    if (g.dtype == DLC_F16) hipLaunchKernelGGL(k_quantize<true>, grid, dim3(256), 0, s, payload, g, qp, sym);
    else hipLaunchKernelGGL(k_quantize<false>, grid, dim3(256), 0, s, payload, g, qp, sym);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// quantise + histogram
//   grid: T * bpt work-groups of 4 wavefronts; a work-group stays inside one table, counts into its LDS
//   histogram and merges that into the table's global one at the end.
// ------------------------------------------------------------------------------------------------
// The payload is cut into units of 256 elements, U per table, and every wavefront of the grid gets the same
// number of consecutive units (table after table), so that all of them finish together whatever the shape is.
// A work-group whose units touch several tables handles them one table at a time.
// SAMPLE (single-pass path with DLC_FLAG_SAMPLE_CODEBOOK): only a few groups of every table are counted, for the
// codebook; U is then the number of units of a table's sampled groups, unit u of them stands for unit
// (u / upg) * gstride * upg + u % upg of the table (upg = units of a group, gstride = groups from one sampled group
// to the next), and no plane is written.  (Building a table's codebook in the same launch was tried
// both ways: by the work-group that is the last to add its counts, the launch takes as long as the two it replaces;
// by a single work-group per table that also does all the counting, longer.)
struct SampleArgs {
    uint32_t upg, gstride;
};

template <bool F16, bool VEC, bool LZ, bool SAMPLE = false>
__global__ __launch_bounds__(256) void k_hist(const void* payload, Geom g, const QParam* qp, uint32_t* hist,
                                              uint8_t* sym_plane, uint32_t U, uint32_t units_per_wave, SampleArgs sa) {
    extern __shared__ __align__(16) uint32_t lh[];
    const uint32_t upg = sa.upg, gstride = sa.gstride;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)lh;
    const uint32_t n_words = (kWinBins + 1u) * kWinCopies + g.K;
    const uint64_t total_units = (uint64_t)g.T * U;
    // this wavefront's units [w0, w1) and the work-group's [g0, g1), as global unit numbers
    const uint64_t g0 = (uint64_t)blockIdx.x * 4u * units_per_wave;
    const uint64_t g1 = min(total_units, g0 + 4ull * units_per_wave);
    const uint64_t w0 = min(total_units, g0 + (uint64_t)wave * units_per_wave), w1 = min(total_units, w0 + units_per_wave);
    if (g0 >= g1) return;  // uniform
    const uint32_t t_first = (uint32_t)(g0 / U), t_last = (uint32_t)((g1 - 1) / U);
    for (uint32_t t = t_first; t <= t_last; ++t) {
        {
            uint4* z = reinterpret_cast<uint4*>(lh);
            for (uint32_t k = tid; k < (n_words + 3u) / 4u; k += 256) z[k] = make_uint4(0, 0, 0, 0);
        }
        __syncthreads();
        const QParam q = qp[t];
        const HistC H = hist_consts<LZ>(g, q, lds0, lane);
        const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
        // my units inside table t
        const uint64_t t0 = (uint64_t)t * U, t1 = t0 + U;
        const uint64_t a = max(w0, t0), b = min(w1, t1);
        if (a < b) {
            uint32_t u = (uint32_t)(a - t0);
            const uint32_t ue = (uint32_t)(b - t0);
            for (; u < ue; u += kHistBlk) {
                uint32_t ur = u;  // (a block of kHistBlk units never straddles two groups: upg is a multiple of it)
                if constexpr (SAMPLE) ur = (u / upg) * gstride * upg + u % upg;
                const uint32_t first = ur * (kW * kV);  // element of the table
                if constexpr (SAMPLE) {
                    if (first >= g.n) continue;  // (the last sampled group may be the table's last, ragged one)
                }
                const uint8_t* base = tab + (size_t)first * g.es;
                const uint32_t rem = g.n - first;
                const uint32_t n_units = min(kHistBlk, ue - u);
                uint32_t* plane = SAMPLE ? nullptr : reinterpret_cast<uint32_t*>(sym_plane + (size_t)t * plane_stride(g) + first);
                if (n_units == kHistBlk && rem >= kHistBlk * kW * kV) hist_block<F16, VEC, true, LZ, SAMPLE ? kNoPlane : kPlane>(base, rem, n_units, lane, q, H, plane);
                else hist_block<F16, VEC, false, LZ, SAMPLE ? kNoPlane : kPlane>(base, rem, n_units, lane, q, H, plane);
            }
        }
        __syncthreads();
        hist_merge<LZ, 256>(lh, g, hist + (size_t)t * g.K, tid);
        __syncthreads();
    }
}

// carry != 0: the codebook is for the next call (the escape symbol gets a code whether it occurred or not)
// tpw: tables per work-group, 1 or 4 (see codebook_tables_per_wg)
__global__ __launch_bounds__(256) void k_codebook(Geom g, uint32_t* hist, uint32_t* hist_view, uint16_t* enc,
                                                  uint8_t* lens, TMeta* tmeta, uint32_t carry, uint32_t tpw) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ CodebookShared sh;
    __shared__ uint32_t s_slow[4];
    if (tpw == 4u) {
        codebook_build_four(g, blockIdx.x * 4u, hist, hist_view, enc, lens, tmeta, smem, sh, s_slow, threadIdx.x, carry);
    } else {
        const uint32_t t = blockIdx.x;
        codebook_build(g, hist + (size_t)t * g.K, hist_view + (size_t)t * g.K, enc + (size_t)t * g.K,
                       lens + (size_t)t * g.K, tmeta + t, smem, sh, threadIdx.x, carry);
    }
}

// With few tables a work-group per table (all its threads read the histogram: the shortest way to one codebook); with
// many, four tables per work-group, a wavefront each (a quarter of the work-groups, and no idle wavefronts while
// one of them builds the tree).
static inline uint32_t codebook_tables_per_wg(const Geom& g) { return g.T >= 512u && g.K >= kWaveAlphabet ? 4u : 1u; }
static inline size_t codebook_lds(const Geom& g, uint32_t tpw) { return tpw == 4u ? codebook_four_smem(g.K) : codebook_smem(g.K); }

template <uint32_t NT>
__global__ __launch_bounds__(NT) void k_finalize(Geom g, FixedLayout F, const TMeta* tmeta, const uint8_t* __restrict__ lens,
                                                   const QParam* qp, Ctrl* ctrl, const uint32_t* word_start,
                                                   const uint32_t* word_end, uint8_t* __restrict__ out, uint64_t capacity,
                                                   uint64_t* out_bytes, uint32_t* esc_count, const uint8_t* rm_on,
                                                   const uint32_t* rm_ref, uint32_t* bsum) {
    // blockIdx.y: the destination whose container this work-group helps to finish
    finalize_dest<NT>(g, F, tmeta, lens, qp, ctrl, word_start, word_end, out, capacity, out_bytes, esc_count, rm_on, rm_ref, bsum,
                        blockIdx.y, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------------------------------
// single-pass path, second step: one launch, three jobs that do not wait for one another.  Where a group's words go
// is the sum of the totals of all groups before it in its container; the encode kernel has added the totals up per
// block of kSumBlock groups, so whoever needs such a sum reads the sums of the blocks before and the totals of the
// groups in between.
//   the first work-groups, one per table or per four tables: the codebook of the next call from this call's counts, into the second set of codebook arrays
//     (this call's set is still being read)
//   then nf work-groups per destination: the container's header, directory, code-length blocks, sizes (finalize_dest),
//     from the tables' word ranges, which they work out from the sums themselves
//   the rest: the groups' words from their slots to their places, kPlaceGroups groups per work-group, a group per
//     wavefront (coalesced both ways), and the group table.  Nothing is written past a container's capacity.
// ------------------------------------------------------------------------------------------------
// words of the groups [0, x) of a destination (called by a whole wavefront, same x)
__device__ __forceinline__ unsigned long long words_before(const uint32_t* bs, const uint32_t* gtot_d, uint32_t x, uint32_t lane) {
    const uint32_t blk = x / kSumBlock;
    unsigned long long acc = 0;
    for (uint32_t i = lane; i < blk; i += 64) acc += bs[i];
    for (uint32_t i = blk * kSumBlock + lane; i < x; i += 64) acc += gtot_d[i];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    return acc;
}

__global__ __launch_bounds__(256) void k_post(Geom g, FixedLayout F, const uint32_t* gtot, const uint32_t* bsum, uint32_t* bsum_next,
                                              const uint32_t* slots, uint64_t slot_words, Ctrl* ctrl, uint8_t* out,
                                              uint64_t capacity, uint32_t wpd, uint32_t nf, uint32_t* word_start,
                                              uint32_t* word_end, const TMeta* tmeta, const uint8_t* lens, const QParam* qp,
                                              uint64_t* out_bytes, uint32_t* esc_count, uint32_t* hist, uint32_t* hist_view,
                                              uint16_t* enc_next, uint8_t* lens_next, TMeta* tmeta_next, uint32_t tpw) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t gpd = g.TD * g.G;  // groups of one destination
    // work-groups that build the next call's codebooks, tpw (1 or 4) tables each; tpw == 0: none (no codebook is carried)
    const uint32_t n_cb = tpw ? (g.T + tpw - 1u) / tpw : 0u;
    if (blockIdx.x < n_cb) {  // uniform over the work-group; these come first: a codebook takes longer than a copy
        __shared__ CodebookShared sh;
        __shared__ uint32_t s_slow[4];
        if (tpw == 4u) {
            codebook_build_four(g, blockIdx.x * 4u, hist, hist_view, enc_next, lens_next, tmeta_next, smem, sh, s_slow, tid, 1u);
        } else {
            const uint32_t t = blockIdx.x;
            codebook_build(g, hist + (size_t)t * g.K, hist_view + (size_t)t * g.K, enc_next + (size_t)t * g.K,
                           lens_next + (size_t)t * g.K, tmeta_next + t, smem, sh, tid, 1u);
        }
        return;
    }
    if (blockIdx.x < n_cb + g.ND * nf) {
        const uint32_t f = blockIdx.x - n_cb, dst = f / nf, xi = f - dst * nf;
        const uint32_t* const bs = bsum + (size_t)dst * sum_blocks_per_dest(g);
        const uint32_t* const gtot_d = gtot + (size_t)dst * gpd;
        // The tables' word ranges (stored past the caches: finalize_dest reads them that way): a scan over the block
        // sums, 256 blocks a pass; the thread of a block looks after the tables that start inside it.  Every one of
        // the nf work-groups needs the last table's end, only the first of them the rest.
        __shared__ uint32_t s_scan[5];
        __shared__ unsigned long long s_sum64[4];
        const uint32_t nb = sum_blocks_per_dest(g);
        uint32_t carry = 0;
        unsigned long long all = 0;
        for (uint32_t c0 = 0; c0 < nb; c0 += 256) {  // uniform trip count
            const uint32_t blk = c0 + tid;
            const uint32_t v = blk < nb ? bs[blk] : 0u;
            unsigned long long v64 = v;
            for (int o = 32; o > 0; o >>= 1) v64 += __shfl_xor(v64, o, 64);
            if (lane == 0) s_sum64[wave] = v64;
            uint32_t tot;
            const uint32_t before = carry + block_excl_scan<4>(v, s_scan, tid, &tot);
            all += s_sum64[0] + s_sum64[1] + s_sum64[2] + s_sum64[3];
            if (xi == 0 && blk < nb) {
                const uint32_t x0 = blk * kSumBlock, x1 = min(gpd, x0 + kSumBlock);
                uint32_t w = before, i = x0;  // (one walk over the block's groups serves all the tables that start in it)
                for (uint32_t tl = (x0 + g.G - 1u) / g.G; tl < g.TD && tl * g.G < x1; ++tl) {
                    for (; i < tl * g.G; ++i) w += gtot_d[i];
                    __hip_atomic_store(&word_start[dst * g.TD + tl], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (tl > 0) __hip_atomic_store(&word_end[dst * g.TD + tl - 1u], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            carry += tot;
            __syncthreads();
        }
        if (tid == 0) {  // (clamped; past 2^32 words the format cannot say where a group starts: the call fails)
            if (all > 0xFFFFFFFFull && xi == 0) { set_status(ctrl, DLC_ECAPACITY); atomicOr(&ctrl->abort, 1u); }
            __hip_atomic_store(&word_end[dst * g.TD + g.TD - 1u], (uint32_t)min(all, 0xFFFFFFFFull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        finalize_dest<256>(g, F, tmeta, lens, qp, ctrl, word_start, word_end, out, capacity, out_bytes, esc_count,
                           (const uint8_t*)nullptr, (const uint32_t*)nullptr, bsum_next, dst, xi, nf);
        return;
    }
    const uint32_t wg = blockIdx.x - n_cb - g.ND * nf;
    const uint32_t dst = wg / wpd, k = wg - dst * wpd;  // wpd work-groups per destination
    const uint32_t g0 = k * kPlaceGroups;
    if (g0 + wave >= gpd) return;  // whole wavefront
    uint8_t* const out_d = out + (uint64_t)dst * capacity;
    const uint32_t gl = g0 + wave;  // group number inside the container
    const size_t gg = (size_t)dst * gpd + gl;
    const unsigned long long base = words_before(bsum + (size_t)dst * sum_blocks_per_dest(g), gtot + (size_t)dst * gpd, gl, lane);
    const uint32_t total = gtot[gg];
    // (word offsets are 32-bit: a container of 2^32 words or more does not fit any capacity the format can describe;
    // the finishing work-groups come to the same verdict from the same sums and report it)
    if (base + total > 0xFFFFFFFFull || F.off_payload + 4ull * (base + total) > capacity) return;  // uniform over the wavefront
    const uint32_t goff = (uint32_t)base;
    if (lane == 0) reinterpret_cast<uint32_t*>(out_d + F.off_group)[gl] = goff;
    const uint32_t* src = slots + gg * slot_words;
    uint32_t* dstw = reinterpret_cast<uint32_t*>(out_d + F.off_payload) + goff;
    uint32_t j = lane;
    for (; j + 448u < total; j += 512u) {  // eight loads in flight
        uint32_t v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v[u] = src[j + 64u * u];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) dstw[j + 64u * u] = v[u];
    }
    {  // the rest: up to eight more, all in flight too
        uint32_t v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v[u] = j + 64u * u < total ? src[j + 64u * u] : 0u;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            if (j + 64u * u < total) dstw[j + 64u * u] = v[u];
    }
}

// (with row matching: for more references than the coding launch copies, see encode_launch)
// work-groups of the finalize kernel: sixteen wavefronts each, four where a container has at most 256 tables (they start
// sooner and a scan is shorter: 5.3 us -> 4.0), but for row matching, where a work-group copies a table's references (10 us
// with sixteen, 13.6 with four)
static inline uint32_t finalize_threads(const Geom& g) { return g.TD <= 256u && !g.lz ? 256u : 1024u; }
static inline dim3 finalize_grid(const Geom& g) {
    // a wavefront per table for the code-length blocks; with row matching a work-group per table copies its references
    const uint32_t per_wg = g.lz ? 1u : finalize_threads(g) / 64u;
    return dim3(std::min<uint32_t>((std::min<uint32_t>(g.TD, 1024u) + per_wg - 1u) / per_wg, 64u), g.ND);
}

hipError_t launch_compress(const Geom& g, const void* payload, uint8_t* out, uint64_t capacity, uint64_t* out_bytes,
                           const Ws& w, uint64_t epoch, bool carry_ready, int pl, void* prof, hipStream_t s) {
    const bool f16 = g.dtype == DLC_F16;
    const FixedLayout F = fixed_layout(g);
    if (w.sample != 0) {
        // single pass without a carried codebook: the counts of a few groups of every table, their codebook (the escape
        // symbol always gets a code: an element whose symbol the sample has not seen is stored as an escape)
        uint32_t ns, gstride;
        sample_groups(g, &ns, &gstride);
        const uint32_t upg = g.S / kV;  // units of a group
        const uint32_t U = ns * upg;
        const uint64_t total_units = (uint64_t)g.T * U;
        const uint32_t units_per_wave = 4 * kHistBlk;
        const uint32_t grid_n = (uint32_t)((total_units + 4ull * units_per_wave - 1) / (4ull * units_per_wave));
        SampleArgs sa;
        sa.upg = upg; sa.gstride = gstride;
        const size_t sm = hist_lds_bytes(g.K);
        if (prof_on(pl, P_HIST)) prof_begin(prof, P_HIST, s);
#define DLC_HIST(FF, V) hipLaunchKernelGGL((k_hist<FF, V, false, true>), dim3(grid_n), dim3(256), sm, s, payload, g, w.qp, w.hist, \
                                           (uint8_t*)nullptr, U, units_per_wave, sa)
        if (f16) { if (g.vec) DLC_HIST(true, true); else DLC_HIST(true, false); }
        else { if (g.vec) DLC_HIST(false, true); else DLC_HIST(false, false); }
#undef DLC_HIST
        if (prof_on(pl, P_HIST)) prof_end(prof, P_HIST, s);
        if (prof_on(pl, P_CODEBOOK)) prof_begin(prof, P_CODEBOOK, s);
        const uint32_t tpw = codebook_tables_per_wg(g);
        hipLaunchKernelGGL(k_codebook, dim3((g.T + tpw - 1u) / tpw), dim3(256), codebook_lds(g, tpw), s, g, w.hist, w.hist_view, w.enc, w.lens,
                           w.tmeta, 1u, tpw);
        if (prof_on(pl, P_CODEBOOK)) prof_end(prof, P_CODEBOOK, s);
    }
    if (w.sample != 0 || (w.carry != 0 && carry_ready)) {
        // single pass: encode with the codebook of the previous call, then build the next one from this call's counts
        // (or, with the sample's codebook, nothing to build)
        const uint32_t bpt = (g.G + 3) / 4;
        if (prof_on(pl, P_CARRY)) prof_begin(prof, P_CARRY, s);
        switch (g.S) {
            case 64: launch_encode_carry_64(g, F, payload, w, epoch, out, capacity, bpt, s); break;
            case 128: launch_encode_carry_128(g, F, payload, w, epoch, out, capacity, bpt, s); break;
            default: launch_encode_carry_256(g, F, payload, w, epoch, out, capacity, bpt, s); break;
        }
        if (prof_on(pl, P_CARRY)) prof_end(prof, P_CARRY, s);
        {
            const uint32_t wpd = (g.TD * g.G + kPlaceGroups - 1) / kPlaceGroups, n_place = g.ND * wpd;
            const uint32_t nf = std::min<uint32_t>((std::min<uint32_t>(g.TD, 256u) + 3u) / 4u, 64u);  // a wavefront per table's code-length block
            if (prof_on(pl, P_POST)) prof_begin(prof, P_POST, s);
            const uint32_t tpw = w.sample != 0 ? 0u : codebook_tables_per_wg(g);
            hipLaunchKernelGGL(k_post, dim3((tpw ? (g.T + tpw - 1u) / tpw : 0u) + g.ND * nf + n_place), dim3(256), codebook_lds(g, tpw), s, g, F, w.gtot, w.bsum,
                               w.bsum_next, w.slots, (uint64_t)carry_slot_words(g), w.ctrl, out, capacity, wpd, nf, w.word_start,
                               w.word_end, w.tmeta, w.lens, w.qp, out_bytes, w.esc_count, w.hist, w.hist_view, w.enc_next,
                               w.lens_next, w.tmeta_next, tpw);
            if (prof_on(pl, P_POST)) prof_end(prof, P_POST, s);
        }
        return hipGetLastError();
    }
    // Larger tables go from payload to coded groups in one launch as well, a table being the work of many work-groups (k_flow): the
    // work-groups that count take 1024 shares of the payload and more, and those that code begin when the first of the counting ones
    // are done instead of after the last.  Above 311296 units of 256 elements (524288 in half precision) more are counted than are
    // ahead, and the coding of some tables has the counting of others beside it.  Fewer units than 72000 and the waits for counts and
    // codebooks inside the launch are longer than the gaps between three launches (us, three launches and one: 65536 units of 16, 64 and
    // of one table 46 and 52, 47 and 50, 52 and 51; 72000 of 64 57 and 52; 75000 of one 58 and 53, of two 54 and 52; 163840 of 64 78 and 71, 262144 of 64
    // and of one 102 and 97, 120 and 100, 307200 of 300 123 and 108, 524288 178 and 163; in half precision 65536 of 16 and 64 66 and 70, 77 and 77,
    // 75000 83 and 79, 524288 201 and 189).  From 512 tables on a work-group of the three launches builds four codebooks at a time, which
    // is the shorter way for many tables of large alphabets: tables times symbols 3 * 2^19 at most (4096 symbols: 400 tables of four
    // groups 109 and 87, 512 of three 81 and 87, 700 of two 99 and 110, 2000 of one 141 and 230; 2048: 700 of two 90 and 85, 1000 of two 95 and 110,
    // 2000 of one 131 and 165; 1024: 1000 of 17 in chunks of 64 181 and 173, 1800 296 and 301.  Where such tables use hundreds of symbols,
    // it builds their codebooks one after the other: 700 of eight groups 1337 and 882).  When every kernel is to be timed by itself the
    // launches stay apart.
    const uint64_t units = (uint64_t)g.T * ((g.n + kW * kV - 1u) / (kW * kV));
    const bool flow = !g.lz && units >= 72000u && (g.T < 512u || (uint64_t)g.T * g.K <= 3u << 19) && !prof_on(pl, P_HIST);
    // Small tables: a work-group per table.  Up to eight groups that is the
    // shorter way whatever the number of tables (one launch for three; 26 tables of eight groups: 35.6 us a call against
    // 36.3, one of one group 17.6 against 24.8).  From nine to sixteen groups, what a work-group has wavefronts for, a
    // work-group has a compute unit to itself, and it is the shorter way where there are tables enough to keep the compute units
    // busy (128 tables of sixteen groups: 65 us against 75; 64: 57 against 51; 26: 53 against 40), but not where a second
    // round of work-groups is nearly empty, and less so the longer the codes are (at ratios of 10 and 5.9: 257 tables of
    // twelve groups 110 and 197 us against 98 and 153; 300: 113 and 202 against 109 and 168; 350: 118 and 205 against 121 and
    // 184; 400: 124 and 211 against 132 and 197; 512: 142 and 229 against 159 and 344), and not in several rounds of larger tables
    // where k_flow does it (400 of sixteen groups 147 and 137, in half precision 191 and 173; of nine 94 and 96, of twelve in chunks of 64 symbols 52 and 62).  Row matching needs every row's
    // symbols before it knows the counts: it keeps the launches apart, and so do many tables
    // of a large alphabet, whose scratch memory would leave a compute unit one work-group at a time.
    const bool whole_rounds = (g.T >= 128u && g.T <= 256u) || (g.T > 352u && !(flow && g.n >= 200000u));
    const bool fused = !g.lz && (g.G <= 8u || (g.G <= 16u && whole_rounds)) && (g.T <= 256u || g.K <= 1024u);
    const uint32_t tpw = codebook_tables_per_wg(g);
    // The launch that codes the groups finishes the containers, too, where a work-group has a thread for each of a container's
    // tables (see finish_container), unless every kernel is to be timed by itself or there are very many references to copy.
    uint64_t* const fin = prof_on(pl, P_FINALIZE) ? nullptr : out_bytes;
    bool finished = false;
    if (fused) {
        if (prof_on(pl, P_TABLE)) prof_begin(prof, P_TABLE, s);
        switch (g.S) {
            case 64: finished = launch_table_64(g, F, payload, w, epoch, out, capacity, fin, s); break;
            case 128: finished = launch_table_128(g, F, payload, w, epoch, out, capacity, fin, s); break;
            default: finished = launch_table_256(g, F, payload, w, epoch, out, capacity, fin, s); break;
        }
        if (prof_on(pl, P_TABLE)) prof_end(prof, P_TABLE, s);
    } else if (flow) {
        if (prof_on(pl, P_FLOW)) prof_begin(prof, P_FLOW, s);
        switch (g.S) {
            case 64: finished = launch_flow_64(g, F, payload, w, epoch, out, capacity, fin, s); break;
            case 128: finished = launch_flow_128(g, F, payload, w, epoch, out, capacity, fin, s); break;
            default: finished = launch_flow_256(g, F, payload, w, epoch, out, capacity, fin, s); break;
        }
        if (prof_on(pl, P_FLOW)) prof_end(prof, P_FLOW, s);
    } else {
        // histogram
        {
            // equal shares of 16 units (16 KiB of fp32) per wavefront: measured best on MI355X, a little ahead of one
            // share per resident wavefront
            const uint32_t U = (g.n + kW * kV - 1) / (kW * kV);
            const uint64_t total_units = (uint64_t)g.T * U;
            // (a small payload is cut finer, so that there is a work-group for every compute unit)
            uint32_t units_per_wave = 4 * kHistBlk;
            while (units_per_wave > kHistBlk && total_units < 4ull * 256u * units_per_wave) units_per_wave -= kHistBlk;
            const uint32_t grid_n = (uint32_t)((total_units + 4ull * units_per_wave - 1) / (4ull * units_per_wave));
            const size_t sm = hist_lds_bytes(g.K);
            dim3 grid(grid_n), block(256);
            if (prof_on(pl, P_HIST)) prof_begin(prof, P_HIST, s);
#define DLC_HIST(FF, V, L) hipLaunchKernelGGL((k_hist<FF, V, L>), grid, block, sm, s, payload, g, w.qp, w.hist, w.sym_plane, U, units_per_wave, SampleArgs{})
            if (g.lz) {  // row matching wants D % 4 == 0, which makes every table start 16-byte aligned with n % 4 == 0
                if (f16) DLC_HIST(true, true, true); else DLC_HIST(false, true, true);
            } else if (f16) { if (g.vec) DLC_HIST(true, true, false); else DLC_HIST(true, false, false); }
            else { if (g.vec) DLC_HIST(false, true, false); else DLC_HIST(false, false, false); }
#undef DLC_HIST
            if (prof_on(pl, P_HIST)) prof_end(prof, P_HIST, s);
        }
        if (g.lz) {  // row matching: which rows repeat an earlier one; their elements leave the plane and the counts again
            hipError_t e = launch_row_match(g, payload, w, s);
            if (e != hipSuccess) return e;
        }
        if (prof_on(pl, P_CODEBOOK)) prof_begin(prof, P_CODEBOOK, s);
        hipLaunchKernelGGL(k_codebook, dim3((g.T + tpw - 1u) / tpw), dim3(256), codebook_lds(g, tpw), s, g, w.hist, w.hist_view, w.enc, w.lens,
                           w.tmeta, 0u, tpw);
        if (prof_on(pl, P_CODEBOOK)) prof_end(prof, P_CODEBOOK, s);
        {
            if (prof_on(pl, P_ENCODE)) prof_begin(prof, P_ENCODE, s);
            switch (g.S) {
                case 64: finished = launch_encode_64(g, F, payload, w, epoch, out, capacity, fin, s); break;
                case 128: finished = launch_encode_128(g, F, payload, w, epoch, out, capacity, fin, s); break;
                default: finished = launch_encode_256(g, F, payload, w, epoch, out, capacity, fin, s); break;
            }
            if (prof_on(pl, P_ENCODE)) prof_end(prof, P_ENCODE, s);
        }
    }
    if (!finished) {
        if (prof_on(pl, P_FINALIZE)) prof_begin(prof, P_FINALIZE, s);
#define DLC_FIN(N) hipLaunchKernelGGL(k_finalize<N>, finalize_grid(g), dim3(N), 0, s, g, F, w.tmeta, w.lens, w.qp, w.ctrl, w.word_start, \
                                      w.word_end, out, capacity, out_bytes, (uint32_t*)nullptr, g.lz ? (const uint8_t*)w.rm_on : nullptr, \
                                      (const uint32_t*)w.rm_ref, (uint32_t*)nullptr)
        if (finalize_threads(g) == 256u) DLC_FIN(256); else DLC_FIN(1024);
#undef DLC_FIN
        if (prof_on(pl, P_FINALIZE)) prof_end(prof, P_FINALIZE, s);
    }
    if (w.carry != 0)  // the codebook the next call will use: this call's counts (kept as the copy), escape symbol included
        hipLaunchKernelGGL(k_codebook, dim3((g.T + tpw - 1u) / tpw), dim3(256), codebook_lds(g, tpw), s, g, w.hist_view, w.hist_view, w.enc_next,
                           w.lens_next, w.tmeta_next, 1u, tpw);
    return hipGetLastError();
}

hipError_t compress_set_attributes() {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_codebook), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)codebook_four_smem(4096));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_post), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)codebook_four_smem(4096));
    if (e == hipSuccess) e = encode_set_attributes_64();
    if (e == hipSuccess) e = encode_set_attributes_128();
    if (e == hipSuccess) e = encode_set_attributes_256();
    return e;
}

}  // namespace dlc
