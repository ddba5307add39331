// The end of a compress call, for one container: code-length blocks behind the payload, header, directory, padding, size
// metadata; the per-call control words cleared for the next call.  Every work-group that takes part works out where the
// code-length blocks go (a scan over the tables) and writes its share of them; the first one also writes everything else.
#pragma once
#include "dlc_codec_dev.h"

namespace dlc {

__device__ __forceinline__ uint64_t a16(uint64_t x) { return (x + 15ull) & ~15ull; }

// padding between the sections of a container, and its header
template <uint32_t NT>
__device__ __forceinline__ void finish_header(const Geom& g, const FixedLayout& F, uint8_t* out, uint64_t words, uint64_t off_cb,
                                              uint64_t total, uint64_t n_esc, uint32_t tid) {
    const uint32_t T = g.TD;
    const uint64_t e0 = kHeaderBytes + (uint64_t)kDirBytes * T;
    for (uint64_t i = e0 + tid; i < F.off_group; i += NT) out[i] = 0;
    const uint64_t e1 = F.off_group + 4ull * T * g.G;
    for (uint64_t i = e1 + tid; i < F.off_chunk; i += NT) out[i] = 0;
    const uint64_t e2 = F.off_payload + 4ull * words;
    for (uint64_t i = e2 + tid; i < off_cb; i += NT) out[i] = 0;
    if (tid == 0) {
        uint32_t* h = reinterpret_cast<uint32_t*>(out);
        h[H_MAGIC] = kMagic; h[H_VERSION] = kVersion; h[H_DTYPE] = g.dtype; h[H_T] = T; h[H_B] = g.B; h[H_D] = g.D;
        h[H_R] = g.R; h[H_S] = g.S; h[H_LMAX] = g.LMAX; h[H_W] = kW; h[H_V] = kV; h[H_NG] = T * g.G;
        uint64_t* q = reinterpret_cast<uint64_t*>(out);
        q[HQ_NOUT] = n_esc; q[HQ_WORDS] = words; q[HQ_OFF_GROUP] = F.off_group; q[HQ_OFF_CHUNK] = F.off_chunk;
        q[HQ_OFF_PAYLOAD] = F.off_payload; q[HQ_OFF_CB] = off_cb;
        q[HQ_TOTAL] = total; q[HQ_TOTAL + 1] = 0; q[HQ_TOTAL + 2] = 0; q[HQ_TOTAL + 3] = 0;
    }
}

// a table's directory entry, and the bytes attributable to it
__device__ __forceinline__ void finish_table(const Geom& g, uint8_t* out, uint32_t t, const TMeta& m, uint32_t eb_bits, uint64_t block, uint32_t block_bytes,
                                             uint32_t w0, uint32_t w1, uint64_t* table_bytes) {
    uint8_t* d = out + kHeaderBytes + (uint64_t)kDirBytes * t;
    uint32_t* d32 = reinterpret_cast<uint32_t*>(d);
    d32[0] = eb_bits; d32[1] = m.n_used; d32[2] = m.sym_lo; d32[3] = m.sym_hi; d32[4] = m.n_outliers;
    d32[5] = g.G;
    uint64_t* d64 = reinterpret_cast<uint64_t*>(d + 24);
    d64[0] = block; d64[1] = 0; d64[2] = w0; d64[3] = (uint64_t)(w1 - w0);
    table_bytes[t] = 4ull * (uint64_t)(w1 - w0) + block_bytes + (uint64_t)(kW + 4u) * g.G + kDirBytes;
}

// Sizes: one destination -> out_bytes[0] is its container's size.  Several -> every destination stores its size
// behind the per-table entries, and the last one to do so adds them up into out_bytes[0] (0 if any did not fit).
// The next call starts with ticket 0 (clear_ticket: by this) and no abort (the histograms were cleared by the codebook step).  By
// one thread.
__device__ __forceinline__ void finish_sizes(const Geom& g, Ctrl* ctrl, uint64_t* out_bytes, uint32_t dst, uint64_t container_bytes, bool clear_ticket) {
    bool last = g.ND == 1;
    if (last) {
        out_bytes[0] = container_bytes;
    } else {
        unsigned long long* dest_bytes = reinterpret_cast<unsigned long long*>(out_bytes + 1 + (size_t)g.ND * g.TD);
        __hip_atomic_store(&dest_bytes[dst], (unsigned long long)container_bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = __hip_atomic_fetch_add(&ctrl->dest_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == g.ND;
        if (last) {
            unsigned long long sum = 0;
            bool all = true;
            for (uint32_t d = 0; d < g.ND; ++d) {
                const unsigned long long b = __hip_atomic_load(&dest_bytes[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                all = all && b != 0;
                sum += b;
            }
            out_bytes[0] = all ? sum : 0;
            __hip_atomic_store(&ctrl->dest_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (last) {
        if (clear_ticket) __hip_atomic_store(&ctrl->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctrl->abort, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}


// One destination's container, by work-group xi of the xn that share the work (all of NT threads); everything below is
// that container's.  The tables' word ranges may come from work-groups of the running kernel: they are read past the caches.
template <uint32_t NT>
__device__ __forceinline__ void finalize_dest(const Geom& g, const FixedLayout& F, const TMeta* tmeta, const uint8_t* __restrict__ lens,
                                              const QParam* qp, Ctrl* ctrl, const uint32_t* word_start, const uint32_t* word_end,
                                              uint8_t* __restrict__ out, uint64_t capacity, uint64_t* out_bytes, uint32_t* esc_count,
                                              const uint8_t* rm_on, const uint32_t* rm_ref, uint32_t* bsum, uint32_t dst, uint32_t xi,
                                              uint32_t xn) {
    constexpr uint32_t NW = NT / 64u;
    __shared__ uint32_t s_red[NW + 1];
    __shared__ uint32_t s_abort;
    __shared__ uint32_t s_cb[NT + 1];   // start of each table's block, relative to the pass's first block
    __shared__ uint32_t s_lo[NT], s_nl[NT];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const bool first = xi == 0;
    const uint32_t T = g.TD;
    tmeta += (size_t)dst * T;
    lens += (size_t)dst * T * g.K;
    qp += (size_t)dst * T;
    word_start += (size_t)dst * T;
    word_end += (size_t)dst * T;
    if (esc_count) esc_count += (size_t)dst * T;
    out += (uint64_t)dst * capacity;
    uint64_t* const table_bytes = out_bytes + 1 + (size_t)dst * T;
    const uint64_t words = __hip_atomic_load(&word_end[T - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t off_cb = a16(F.off_payload + 4ull * words);
    // an internal failure of the encode kernel spoils every container; one that did not fit spoils only itself, and
    // the capacity test below fails for it whenever the encode kernel's did.  (The flag is cleared by the last
    // destination to finish, so every destination's first work-group can still read it.)
    if (first && bsum) {  // single-pass path: the block sums the next call adds to start at zero (not the ones this call reads)
        const uint32_t nb = sum_blocks_per_dest(g);
        for (uint32_t i = tid; i < nb; i += NT) bsum[(size_t)dst * nb + i] = 0u;
    }
    const bool aborted = first && __hip_atomic_load(&ctrl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    uint64_t cb_carry = 0, nout_carry = 0;
    for (uint32_t base = 0; base < T; base += NT) {
        const uint32_t t = base + tid;
        TMeta m;
        uint32_t cb = 0, no = 0, nl = 0, w0 = 0, w1 = 0, eb_bits = 0;
        if (t < T) {
            m = tmeta[t];
            if (first) {  // (what the directory needs, together with the rest: one latency)
                w0 = __hip_atomic_load(&word_start[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                w1 = __hip_atomic_load(&word_end[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                eb_bits = qp[t].eb_bits;
            }
            if (first && esc_count) {  // single-pass path: the codebook is older than the payload, the escapes were counted by the encode kernel
                m.n_outliers = esc_count[t];
                esc_count[t] = 0;
            }
            if (m.sym_lo > m.sym_hi || m.sym_hi >= g.K) { m.sym_lo = 0; m.sym_hi = 0; }  // never index outside lens[]
            nl = m.sym_hi - m.sym_lo + 1u;
            cb = (nl + 3u) & ~3u;
            no = m.n_outliers;
        }
        uint32_t cb_tot, no_tot;
        const uint32_t cb_ex = block_excl_scan<(int)NW>(cb, s_red, tid, &cb_tot);
        __syncthreads();
        (void)block_excl_scan<(int)NW>(no, s_red, tid, &no_tot);
        s_cb[tid] = cb_ex;
        s_lo[tid] = m.sym_lo;
        s_nl[tid] = nl;
        if (tid == 0) {
            s_cb[NT] = cb_tot;
            // the code-length blocks are the last thing in the container: the capacity check of this pass
            s_abort = aborted || off_cb + cb_carry + cb_tot > capacity;
        }
        __syncthreads();
        if (s_abort) break;  // uniform
        const uint32_t nt = min(NT, T - base);
        // the blocks of this work-group's tables, a wavefront per table, four bytes per lane (the blocks start on
        // 4-byte boundaries and are padded to them)
        for (uint32_t lt = xi * NW + wave; lt < nt; lt += xn * NW) {
            const uint32_t n_l = s_nl[lt];
            const uint8_t* src = lens + (size_t)(base + lt) * g.K + s_lo[lt];
            uint32_t* dst = reinterpret_cast<uint32_t*>(out + off_cb + cb_carry + s_cb[lt]);
            for (uint32_t wd = lane; wd < (n_l + 3u) / 4u; wd += 64) {
                uint32_t v = 0;
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) {
                    const uint32_t i = wd * 4u + b;
                    v |= (i < n_l ? (uint32_t)src[i] : 0u) << (8u * b);
                }
                dst[wd] = v;
            }
        }
        if (first && t < T) {
            finish_table(g, out, t, m, eb_bits, off_cb + cb_carry + cb_ex, cb, w0, w1, table_bytes);
        }
        cb_carry += cb_tot;
        nout_carry += no_tot;
        __syncthreads();
    }
    // row matching: the references of the tables that use it, behind the code-length blocks, each block on a 16-byte
    // boundary (all blocks are 4*B bytes, so block k starts k * a16(4*B) after the first)
    uint64_t end_bytes = off_cb + cb_carry;  // where the container ends
    if (rm_on && !s_abort) {
        rm_on += (size_t)dst * T;
        rm_ref += (size_t)dst * T * g.B;
        const uint64_t rbase = a16(end_bytes), rsz = a16(4ull * g.B);
        uint32_t n_on = 0;  // tables with references
        for (uint32_t base = 0; base < T; base += NT) {
            uint32_t tot;
            (void)block_excl_scan<(int)NW>((base + tid < T && rm_on[base + tid]) ? 1u : 0u, s_red, tid, &tot);
            n_on += tot;
            __syncthreads();
        }
        if (n_on) end_bytes = rbase + (uint64_t)(n_on - 1u) * rsz + 4ull * g.B;
        if (end_bytes > capacity) {  // uniform
            __syncthreads();
            if (tid == 0) s_abort = 1;
            __syncthreads();
        } else if (n_on) {
            for (uint64_t i = off_cb + cb_carry + tid; first && i < rbase; i += NT) out[i] = 0;
            uint32_t on_carry = 0;
            for (uint32_t base = 0; base < T; base += NT) {
                const uint32_t t = base + tid;
                const uint32_t on = (t < T && rm_on[t]) ? 1u : 0u;
                uint32_t tot;
                const uint32_t ex = block_excl_scan<(int)NW>(on, s_red, tid, &tot);
                s_cb[tid] = on ? on_carry + ex : 0xFFFFFFFFu;  // the table's block number
                __syncthreads();
                if (first && on) {
                    uint64_t* d64 = reinterpret_cast<uint64_t*>(out + kHeaderBytes + (uint64_t)kDirBytes * t + 24);
                    d64[1] = rbase + (uint64_t)(on_carry + ex) * rsz;
                    table_bytes[t] += 4ull * g.B;
                }
                const uint32_t nt = min(NT, T - base);
                for (uint32_t lt = xi; lt < nt; lt += xn) {  // a work-group per table
                    const uint32_t k = s_cb[lt];
                    if (k == 0xFFFFFFFFu) continue;  // uniform
                    uint32_t* dstw = reinterpret_cast<uint32_t*>(out + rbase + (uint64_t)k * rsz);
                    const uint32_t* src = rm_ref + (size_t)(base + lt) * g.B;
                    for (uint32_t r = tid; r < g.B; r += NT) dstw[r] = src[r];
                    if (k + 1u < n_on)  // padding up to the next block
                        for (uint32_t r = g.B + tid; r < (uint32_t)(rsz / 4u); r += NT) dstw[r] = 0u;
                }
                on_carry += tot;
                __syncthreads();
            }
        }
    }
    if (!first) return;
    if (s_abort) {
        if (tid == 0 && !aborted) set_status(ctrl, DLC_ECAPACITY);
        for (uint32_t t = tid; t < T; t += NT) table_bytes[t] = 0;
        if (esc_count)  // whatever the passes after the failing one have not cleared
            for (uint32_t t = tid; t < T; t += NT) esc_count[t] = 0;
    } else {
        finish_header<NT>(g, F, out, words, off_cb, end_bytes, nout_carry, tid);
    }
    if (tid == 0) finish_sizes(g, ctrl, out_bytes, dst, s_abort ? 0ull : end_bytes, true);  // (0: it did not fit)
}

// ------------------------------------------------------------------------------------------------
// The same from inside the kernel that codes the groups (at most as many tables a container as a work-group has threads),
// by `xn` work-groups more for every container.  They have the last of the tickets, so everybody they wait for
// is running already.  They have the code-length blocks' words in LDS before the groups are coded: from the launch
// before, or (LATE) when the tables' work-groups say that their codebooks are there; when the last word's place is known, all
// that is left is to write.  The work-groups with a container's share 0, which write everything but the blocks' other
// words, are the last: the ticket counter is cleared when nobody can ask for one any more (TICKET false: the kernel clears it).
// (A launch of its own costs 4 us whatever it does: one table of 4096 elements 16.6 us a call, so 14.2; 26 tables of 4096 x 64
// 47.6, so 43.7; 512 MiB 202, so 197.  With row matching, where that launch copies the references as well: 3 tables of 1000 x 64
// 47.2, so 43.4, one of 65536 x 128, whose references one work-group copied, 143, so 124, 64 of 8192 x 128 170.5, so 166.4.)
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kFinishWords = 16;  // words of the code-length blocks a thread has if all symbols are used
static inline uint32_t finish_groups(const Geom& g, uint32_t nt) { return (g.TD * (g.K / 4u) + nt * kFinishWords - 1u) / (nt * kFinishWords); }

template <uint32_t NT>
struct FinLds {
    uint32_t red[NT / 64u + 1u];
    uint32_t dead;
    uint32_t cb[NT];    // start of each table's block
    uint32_t span[NT];  // lowest symbol | symbols in the block << 12
    uint32_t end[NT];   // the tables' last words
    uint32_t word[NT * kFinishWords];  // this work-group's share of the blocks
    uint32_t refs[NT];  // row matching: the tables with references
};

constexpr uint32_t kFinishRefs = 16;  // references a thread loads back to back

template <uint32_t NT, bool LATE, bool LZ = false, bool TICKET = true>
__device__ __forceinline__ void finish_container(const Geom& g, const FixedLayout& F, const TMeta* tmeta, const uint8_t* lens, const QParam* qp,
                                                 Ctrl* ctrl, const uint64_t* state, const uint32_t* ready, uint64_t epoch, uint32_t bpt, uint8_t* out, uint64_t capacity,
                                                 uint64_t* out_bytes, uint32_t f, uint32_t xn, FinLds<NT>& L, uint32_t tid,
                                                 const uint8_t* rm_on = nullptr, const uint32_t* rm_ref = nullptr) {
    const uint32_t xi = xn - 1u - f / g.ND, dst = f % g.ND, T = g.TD;  // number f of the ND * xn: the shares 0 are the last
    const bool first = xi == 0u;  // uniform
    tmeta += (size_t)dst * T;
    lens += (size_t)dst * T * g.K;
    out += (uint64_t)dst * capacity;
    state += (size_t)dst * T * bpt;
    uint64_t* const table_bytes = out_bytes + 1 + (size_t)dst * T;
    if (tid == 0) L.dead = 0u;
    auto wait = [&](auto there) {
        for (uint32_t spins = 0; !there(); ++spins) {
            if (spins > 2u * kSpinLimit) {  // never expected; the bound only guarantees termination
                set_status(ctrl, DLC_ESTATE);
                L.dead = 1u;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");  // (what the record vouches for is read after it)
    };
    auto codebook_there = [&] { return __hip_atomic_load(&ready[(size_t)dst * T + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)epoch; };
    auto prefix = [&](uint32_t wg) {  // of work-group `wg` of this container
        uint64_t sv;
        wait([&] {
            sv = __hip_atomic_load(&state[wg], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return (sv >> 34) == epoch && ((uint32_t)(sv >> 32) & 3u) == kFlagPrefix;
        });
        return (uint32_t)sv;
    };
    TMeta m;
    uint32_t nl = 0, cb = 0;
    if (tid < T) {
        if constexpr (LATE) wait(codebook_there);
        m = load_tmeta<LATE>(tmeta + tid);
        if (m.sym_lo > m.sym_hi || m.sym_hi >= g.K) { m.sym_lo = 0; m.sym_hi = 0; }  // never index outside lens[]
        nl = m.sym_hi - m.sym_lo + 1u;
        cb = (nl + 3u) & ~3u;
        L.span[tid] = m.sym_lo | (nl << 12);
    }
    __syncthreads();
    uint32_t cb_tot, n_esc;
    const uint32_t cb_ex = block_excl_scan<(int)(NT / 64u)>(cb, L.red, tid, &cb_tot);
    __syncthreads();
    (void)block_excl_scan<(int)(NT / 64u)>(tid < T ? m.n_outliers : 0u, L.red, tid, &n_esc);
    L.cb[tid] = cb_ex;
    __syncthreads();
    const uint32_t n_words = cb_tot / 4u, share = (n_words + xn - 1u) / xn, w_lo = min(n_words, xi * share), w_hi = min(n_words, w_lo + share);
    for (uint32_t i = w_lo + tid; i < w_hi; i += NT) {
        uint32_t lt = 0;  // the last block that starts at or before the word (every block has one)
#pragma unroll
        for (uint32_t h = NT / 2u; h > 0u; h >>= 1) lt += lt + h < T && L.cb[lt + h] <= 4u * i ? h : 0u;
        const uint32_t at = 4u * i - L.cb[lt], have = (L.span[lt] >> 12) - at;
        const uint8_t* src = lens + (size_t)lt * g.K + (L.span[lt] & 0xFFFu) + at;
        uint32_t c[4];
#pragma unroll
        for (uint32_t b = 0; b < 4u; ++b) {
            c[b] = 0u;
            if (b < have) c[b] = LATE ? __hip_atomic_load(src + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : src[b];
        }
        L.word[i - w_lo] = c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24);
    }
    // row matching: the references of the tables that use it, behind the code-length blocks, each table's on a 16-byte boundary: a
    // share of all of them, in place of the padding zeroes.  The first are loaded before the last word's place is known.
    uint32_t on = 0, on_ex = 0, n_on = 0, r_lo = 0, r_hi = 0, rv[LZ ? kFinishRefs : 1u];
    const uint32_t pitch = (g.B + 3u) & ~3u;  // words from one table's references to the next's
    auto load_refs = [&](uint32_t i0) {
#pragma unroll
        for (uint32_t u = 0; u < (LZ ? kFinishRefs : 0u); ++u) {
            const uint32_t i = i0 + u * NT + tid, k = i / pitch, r = i - k * pitch;
            rv[u] = i < r_hi && r < g.B ? rm_ref[((size_t)dst * T + L.refs[k]) * g.B + r] : 0u;
        }
    };
    if constexpr (LZ) {
        on = tid < T && rm_on[(size_t)dst * T + tid] ? 1u : 0u;
        __syncthreads();
        on_ex = block_excl_scan<(int)(NT / 64u)>(on, L.red, tid, &n_on);
        if (on) L.refs[on_ex] = tid;
        __syncthreads();
        const uint32_t all = n_on ? (n_on - 1u) * pitch + g.B : 0u, part = (all + xn - 1u) / xn;
        r_lo = min(all, xi * part);
        r_hi = min(all, r_lo + part);
        load_refs(r_lo);
    }
    const uint32_t eb_bits = first && tid < T ? qp[(size_t)dst * T + tid].eb_bits : 0u;
    // the words' places
    if (first) {
        if (tid < T) L.end[tid] = prefix((tid + 1u) * bpt - 1u);
    } else if (tid == 0) {
        L.end[T - 1u] = prefix(T * bpt - 1u);
    }
    __syncthreads();
    const uint64_t words = L.end[T - 1u], off_cb = a16(F.off_payload + 4ull * words);
    // (a container that did not fit spoils only itself: the test below fails for it whenever the groups' did)
    const uint64_t off_ref = a16(off_cb + cb_tot), end = n_on ? off_ref + 4ull * ((uint64_t)(n_on - 1u) * pitch + g.B) : off_cb + cb_tot;
    const bool fits = L.dead == 0u && end <= capacity;
    if (LZ && fits) {
        uint32_t* const refs = reinterpret_cast<uint32_t*>(out + off_ref);
        for (uint32_t i0 = r_lo; i0 < r_hi; i0 += NT * kFinishRefs) {
            if (i0 != r_lo) load_refs(i0);
#pragma unroll
            for (uint32_t u = 0; u < (LZ ? kFinishRefs : 0u); ++u)
                if (i0 + u * NT + tid < r_hi) refs[i0 + u * NT + tid] = rv[u];
        }
    }
    if (fits) {
        uint32_t* const blocks = reinterpret_cast<uint32_t*>(out + off_cb);
        for (uint32_t i = w_lo + tid; i < w_hi; i += NT) blocks[i] = L.word[i - w_lo];
    }
    if (!first) return;
    if (fits) {
        if (tid < T) finish_table(g, out, tid, m, eb_bits, off_cb + cb_ex, cb, tid ? L.end[tid - 1u] : 0u, L.end[tid], table_bytes);
        if constexpr (LZ) {
            if (on) {  // (by the thread that has written the entry)
                reinterpret_cast<uint64_t*>(out + kHeaderBytes + (uint64_t)kDirBytes * tid + 24)[1] = off_ref + 4ull * on_ex * pitch;
                table_bytes[tid] += 4ull * g.B;
            }
            if (n_on)
                for (uint64_t i = off_cb + cb_tot + tid; i < off_ref; i += NT) out[i] = 0;
        }
        finish_header<NT>(g, F, out, words, off_cb, end, n_esc, tid);
    } else {
        if (tid == 0 && L.dead == 0u) set_status(ctrl, DLC_ECAPACITY);
        if (tid < T) table_bytes[tid] = 0;
    }
    if (tid == 0) finish_sizes(g, ctrl, out_bytes, dst, fits ? end : 0ull, TICKET);
}

}  // namespace dlc
