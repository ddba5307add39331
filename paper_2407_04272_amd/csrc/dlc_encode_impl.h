// The encode kernels for one chunk size S (DLC_S, defined by the including source file: one file per S keeps the
// compile times apart): k_encode, which codes the symbol plane of tables of any size with codebooks that are there
// already; k_table, which does everything from the payload to the coded groups of a small table in one work-group; and
// k_flow, which does it for large payloads, many work-groups a table, in one launch as well.
#include <algorithm>

#include "dlc_codec_dev.h"
#include "dlc_finalize.h"

#define DLC_CAT2(a, b) a##b
#define DLC_CAT(a, b) DLC_CAT2(a, b)

namespace dlc {

// ------------------------------------------------------------------------------------------------
// bit-packed encode of groups, one wavefront per group, one walk.
//   walk  : lane l codes chunk l of its group.  A word of the symbol plane (four window indices) is two look-ups in a
//           table of PAIRS of symbols in LDS: one dot product of the word's bytes with (4P, 4) is the LDS address of a
//           pair's entry (joined codeword << 8 | joined length; P = how many symbols the table's used range spans).
//           The four codewords are appended to a 64-bit accumulator, and the word they complete is stored without a
//           branch to the lane's LDS column (the row of the last complete word, again and again).  Nothing has to be
//           known before: there is no first walk that adds the lengths up.
//   scan  : chunk word counts inside the wavefront, the wavefronts' totals joined per work-group, the work-groups'
//           totals across the grid by a single-pass look-back (ordered work-group ids: a work-group only ever waits for
//           work-groups that started earlier)
//   copy  : the columns to their places, a team of lanes per chunk.  A column holds `cap` words; a group with a longer
//           chunk is walked again for every further `cap` words (the words of other passes fall on rows nobody reads), from
//           the last trip on at which no column could have been full yet: the walk remembers its state there.  (From the start
//           every time: 512 MiB at a ratio of 7.2, where nearly every group has a few words too many, 243 us a call, now 216; 5.9:
//           278, now 254.  The further walks stay out of the first one's code: one loop over all of them cost the main path
//           6 us, and tables with escapes 110.)
//   escapes: their records (element index, raw bits; in increasing element index, behind the group's chunk words) are
//           written from offsets kept in LDS during the walk, up to kEncRecs per group; a group with more walks its
//           elements once more
// A table whose used symbols span more than pair_max takes the codewords one by one.  An index with no place in
// the tables (an escape, a symbol outside the window, a position past the end of the table) sends its word of the plane
// the long way, for the whole wavefront; a group of which it is known that there are none is not even tested.
// The walk takes 7 to 9 us of a work-group's 25 (128 tables of 64 groups, 16 wavefronts a compute unit); the wait for the
// scan, which all resident work-groups reach together, 7 to 9, the copy 4 to 5, the set-up 2 to 4: 62 us in two rounds.
// The kernel this replaced walked every group twice, three 16-bit look-ups an element, fully unrolled: 94 us there, and
// 40 us for a single group, most of it instruction fetches (here the loops are a few hundred instructions: 14 us with the
// counting and the codebook).
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kEncRecs = 128;   // escapes a wavefront remembers in LDS (their offsets in the group)
constexpr uint32_t kColPitch = 65;   // words from a row of the columns to the next: rows of one column lie in different banks
constexpr uint32_t kPairMax = 63;    // 4P must fit a byte

// LDS of an encoding work-group, in bytes from `at` on: window entries, escape offsets, pair table, columns
struct EncLds {
    uint32_t ent, recs, pair, stage, end;
};
__host__ __device__ inline EncLds enc_lds(uint32_t nw, uint32_t waves, uint32_t cap, uint32_t pair_max) {
    EncLds L;
    L.ent = 0;
    L.recs = 512u;
    L.pair = L.recs + nw * kEncRecs * 2u;
    L.stage = L.pair + ((pair_max * pair_max * 4u + 15u) & ~15u);
    L.end = L.stage + waves * (cap + 2u) * kColPitch * 4u;
    return L;
}

struct EmitEnv {
    const uint8_t* gbase;  // first element of the group
    uint32_t rem;          // elements of the table from there on
    uint32_t lane;
    QParam q;
    float Rf;
    int R;
    const uint16_t* enc_t;  // the table's codebook in memory
    const uint16_t* ent;    // the same by window index, in LDS
    uint32_t w01, w23, c0;  // a plane word's bytes . w01 + c0 = LDS address of its first pair's entry (w23: of its second's)
    uint32_t lo4, over4;    // (byte - lo) + over has its high bit set where the byte has no place in the pair table
    uint32_t col;           // LDS address of this lane's column
    uint32_t row_max;       // the last row (takes what is not wanted)
    uint16_t* recs;
};

constexpr uint32_t kEmitBlk = 4;  // words of the plane a trip of the walk takes; those of the next two are on their way meanwhile
constexpr uint32_t kTripBits = kEmitBlk * kV * (uint32_t)kLmaxLimit;  // a trip adds no more to a chunk

struct EmitState {
    uint64_t acc;   // the chunk's bits so far, the latest at the low end
    uint32_t nbt;   // how many (in a later pass: less the bits of the passes before, modulo 2^32)
    uint32_t nesc;  // escapes of the wavefront so far (uniform)
};

struct EmitMark {   // a walk's state before turn j (a multiple of kEmitBlk)
    uint64_t acc;
    uint32_t nbt, j;
};

__device__ __forceinline__ void emit_piece(const EmitEnv& E, EmitState& S, uint32_t code, uint32_t len) {  // len <= 32
    S.acc = (S.acc << len) | code;
    S.nbt += len;
    const uint32_t row = min(S.nbt >> 5, E.row_max);
    *reinterpret_cast<lds_u32*>(E.col + __umul24(row, kColPitch * 4u)) =
        __builtin_amdgcn_alignbit((uint32_t)(S.acc >> 32), (uint32_t)S.acc, S.nbt);  // (shift: nbt mod 32)
}

// two pairs, each (joined codeword << 8 | joined length), one after the other: at most 24 bits each
__device__ __forceinline__ void emit_two(const EmitEnv& E, EmitState& S, uint32_t e01, uint32_t e23) {
    emit_piece(E, S, e01 >> 8, e01 & 31u);
    emit_piece(E, S, e23 >> 8, e23 & 31u);
}

__device__ __forceinline__ uint32_t pair_entry(uint32_t a, uint32_t b) {  // of two (length << 12 | codeword)
    const uint32_t lb = b >> 12;
    return (((a & 0xFFFu) << lb | (b & 0xFFFu)) << 8) | ((a >> 12) + lb);
}

// (length << 12 | codeword) of the elements of a plane word that lie outside the window (bits of `out`), quantised again:
// their loads go out together, and so do the look-ups (one element after the other, each of them two round trips: 512 MiB
// with 4 % of the elements outside 1845 us a call, now 1160).  The codewords may come from this very launch: they are read
// past the caches.
template <bool F16, bool VEC>
__device__ __forceinline__ void entries_outside(const EmitEnv& E, uint32_t off, uint32_t out, uint32_t (&e)[4]) {
    float x[4];
    uint32_t raw[4], sym[4], got[4];
    (void)load4<F16, VEC>(E.gbase, off, E.rem, x, raw);
#pragma unroll
    for (int v = 0; v < 4; ++v) sym[v] = (out >> v) & 1u ? quant_symbol<F16>(x[v], E.q, E.Rf, E.R) : 0u;
#pragma unroll
    for (int v = 0; v < 4; ++v) got[v] = __hip_atomic_load(&E.enc_t[sym[v]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int v = 0; v < 4; ++v) e[v] = (out >> v) & 1u ? got[v] : e[v];
}

// a word of the plane the long way; `off`: its first element's offset in the group; rec: remember its escapes
template <bool F16, bool VEC>
__device__ __forceinline__ void emit_slow(const EmitEnv& E, EmitState& S, uint32_t m, uint32_t off, bool rec) {
    uint32_t e[4], em = 0, out = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const uint32_t b = (m >> (8 * v)) & 0xFFu;
        const bool in = off + (uint32_t)v < E.rem;  // (whatever the plane holds past the end of the table does not count)
        e[v] = in ? E.ent[b] : 0u;
        out |= (in && b == kWinBins) ? 1u << v : 0u;
        em |= (in && b == kWinEsc) ? 1u << v : 0u;
    }
    if (__ballot(out != 0u) != 0ull) entries_outside<F16, VEC>(E, off, out, e);
    // the records of these escapes, in element order (the walk meets the elements of a group in increasing index:
    // turn, lane, position)
    if (rec && __ballot(em != 0u) != 0ull) {
        const uint32_t cnt = __popc(em);
        if (S.nesc < kEncRecs) {  // uniform
            const uint32_t incl = wave_incl_scan(cnt);
            uint32_t r = S.nesc + incl - cnt;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if ((em >> v) & 1u) {
                    if (r < kEncRecs) E.recs[r] = (uint16_t)(off + (uint32_t)v);
                    ++r;
                }
            S.nesc += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        } else {  // (their group is walked once more for them: they are only counted from here on)
            S.nesc += (uint32_t)__popcll(__ballot(cnt & 1u)) + 2u * (uint32_t)__popcll(__ballot(cnt & 2u)) + 4u * (uint32_t)__popcll(__ballot(cnt & 4u));
        }
    }
    emit_two(E, S, pair_entry(e[0], e[1]), pair_entry(e[2], e[3]));
}

// the N words of one trip (at p and every kW words on).  PAIR: the pair table serves (else the codewords one by one);
// CHECK: a byte may have no place in the tables; LZ: a word may belong to a row that is stored as a reference (all
// four bytes 253: no bits)
template <bool F16, bool VEC, bool PAIR, bool CHECK, bool LZ, uint32_t N>
__device__ __forceinline__ void emit_block(const EmitEnv& E, EmitState& S, const uint32_t (&m)[N], const uint32_t* p, uint32_t off, bool rec) {
    uint32_t e01[N], e23[N];
    uint32_t w[N];
    bool bad = false;
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
        w[u] = m[u];
        const bool ref = LZ && PAIR && w[u] == 0x01010101u * kWinSkip;
        if constexpr (CHECK) {
            if constexpr (PAIR) {
                const uint32_t d = w[u] - E.lo4;
                const bool b = (((d | (d + E.over4)) & 0x80808080u) != 0u) & !ref;
                w[u] = b ? E.lo4 : w[u];  // (an address inside the table)
                bad |= b;
            } else {  // (index 254 or 255)
                const uint32_t x = ~(w[u] | 0x01010101u);
                bad |= ((x - 0x01010101u) & ~x & 0x80808080u) != 0u;
            }
        }
        if (ref) w[u] = E.lo4;
    }
    if (CHECK && __builtin_expect(__ballot(bad) != 0ull, 0)) {  // uniform over the wavefront
#pragma clang loop unroll(disable)
        for (uint32_t u = 0; u < N; ++u) emit_slow<F16, VEC>(E, S, p[u * kW], off + u * (kW * kV), rec);
        return;
    }
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
        if constexpr (PAIR) {
            e01[u] = *reinterpret_cast<lds_u32*>(__builtin_amdgcn_udot4(w[u], E.w01, E.c0, false));
            e23[u] = *reinterpret_cast<lds_u32*>(__builtin_amdgcn_udot4(w[u], E.w23, E.c0, false));
        } else {
            e01[u] = pair_entry(E.ent[w[u] & 0xFFu], E.ent[(w[u] >> 8) & 0xFFu]);
            e23[u] = pair_entry(E.ent[(w[u] >> 16) & 0xFFu], E.ent[w[u] >> 24]);
        }
    }
    uint32_t L[N], most = 0;
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
        if (LZ && PAIR && m[u] == 0x01010101u * kWinSkip) { e01[u] = 0u; e23[u] = 0u; }
        L[u] = (e01[u] + e23[u]) & 63u;  // (48 bits at most)
        most = max(most, L[u]);
    }
    if (__builtin_expect(__ballot(most > 32u) == 0ull, 1)) {  // the rule: four codewords as one piece of at most 32 bits
#pragma unroll
        for (uint32_t u = 0; u < N; ++u) emit_piece(E, S, ((e01[u] >> 8) << (e23[u] & 31u)) | (e23[u] >> 8), L[u]);
    } else {
#pragma unroll
        for (uint32_t u = 0; u < N; ++u) emit_two(E, S, e01[u], e23[u]);
    }
}

// a walk over the first `els` elements of the group, from turn `from` on (a multiple of kEmitBlk): trips of whole turns, the
// rest (at most kEmitBlk turns) a turn at a time.  Returns its state at the first trip in which a chunk could pass `limit` +
// kTripBits bits, or at the end of the trips.
template <bool F16, bool VEC, bool PAIR, bool CHECK, bool LZ>
__device__ __forceinline__ EmitMark emit_turns(const EmitEnv& E, EmitState& S, const uint32_t* plane, uint32_t els, uint32_t from, int limit, bool rec) {
    const uint32_t* p = plane + E.lane;
    const uint32_t whole = els / (kW * kV) & ~(kEmitBlk - 1u), turns = (els + kW * kV - 1u) / (kW * kV);
    EmitMark M;
    M.j = 0xFFFFFFFFu;
    if (from < whole) {
        uint32_t na[kEmitBlk], nb[kEmitBlk];  // the words of the next trip and of the one after it
        const uint32_t last = whole - kEmitBlk;
#pragma unroll
        for (uint32_t u = 0; u < kEmitBlk; ++u) na[u] = p[(from + u) * kW];
#pragma unroll
        for (uint32_t u = 0; u < kEmitBlk; ++u) nb[u] = p[(min(from + kEmitBlk, last) + u) * kW];
#pragma clang loop unroll(disable)
        for (uint32_t j = from; j < whole; j += kEmitBlk) {
            if (__ballot((int)S.nbt > limit) != 0ull) {  // uniform
                M.acc = S.acc;
                M.nbt = S.nbt;
                M.j = j;
                limit = 0x7FFFFFFF;
            }
            uint32_t m[kEmitBlk];
#pragma unroll
            for (uint32_t u = 0; u < kEmitBlk; ++u) { m[u] = na[u]; na[u] = nb[u]; }
            const uint32_t jn = min(j + 2u * kEmitBlk, last);
#pragma unroll
            for (uint32_t u = 0; u < kEmitBlk; ++u) nb[u] = p[(jn + u) * kW];
            emit_block<F16, VEC, PAIR, CHECK, LZ>(E, S, m, p + j * kW, E.lane * kV + j * (kW * kV), rec);
        }
    }
    if (M.j == 0xFFFFFFFFu) {
        M.acc = S.acc;
        M.nbt = S.nbt;
        M.j = whole;
    }
#pragma clang loop unroll(disable)
    for (uint32_t j = whole; j < turns; ++j) emit_slow<F16, VEC>(E, S, p[j * kW], E.lane * kV + j * (kW * kV), rec);
    return M;
}

// What a work-group knows when its tables are in LDS
struct GroupJob {
    uint32_t t, tl, dst;    // the table, its place in its container, the container
    uint32_t wg, dom0;      // this work-group's place in the scan, the first of its scan domain
    uint32_t grp;           // this wavefront's group (>= g.G: none; the wavefront then only takes part in the barriers)
    uint32_t lo, P;         // the used symbols span the window indices [lo, lo + P)
    bool pairs;             // the pair table is there
    bool special;           // an index without a place in the tables can occur
    uint32_t cap;           // words of a column
    uint32_t lds0;          // LDS address of the areas
    EncLds L;
};

// walk, scan, copy (see above) for the groups of a work-group of NW wavefronts
template <int S, bool F16, bool VEC, bool LZ, uint32_t NW>
__device__ __forceinline__ void encode_groups(const GroupJob& J, const void* payload, const uint8_t* sym_plane, const Geom& g,
                                              const FixedLayout& F, const QParam* qp, const uint16_t* enc, Ctrl* ctrl, uint64_t* state,
                                              uint64_t epoch, uint8_t* out, uint64_t capacity, uint32_t* word_start, uint32_t* word_end,
                                              unsigned char* smem, uint32_t tid) {
    __shared__ uint32_t s_tot[NW], s_excl, s_dead;
    const uint32_t lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t grp = J.grp, t = J.t, cap = J.cap;
    const bool active = grp < g.G;  // uniform over the wavefront
    const uint32_t gid = J.tl * g.G + (active ? grp : 0u);  // group number inside the container
    const uint32_t gstart = grp * (kW * (uint32_t)S);
    const uint8_t* const gbase = static_cast<const uint8_t*>(payload) + ((size_t)t * g.n + gstart) * g.es;
    const uint32_t* const plane = reinterpret_cast<const uint32_t*>(sym_plane + (size_t)t * plane_stride(g) + gstart);
    EmitEnv E;
    E.gbase = gbase;
    E.rem = active ? g.n - gstart : 0u;
    E.lane = lane;
    E.q = qp[t];
    E.Rf = (float)g.R;
    E.R = (int)g.R;
    E.enc_t = enc + (size_t)t * g.K;
    E.ent = reinterpret_cast<const uint16_t*>(smem + J.L.ent);
    E.w01 = (4u * J.P) | (4u << 8);
    E.w23 = E.w01 << 16;
    E.c0 = J.lds0 + J.L.pair - 4u * J.lo * (J.P + 1u);
    E.lo4 = J.lo * 0x01010101u;
    E.over4 = (128u - J.P) * 0x01010101u;
    E.row_max = cap + 1u;
    uint32_t* const rows = reinterpret_cast<uint32_t*>(smem + J.L.stage) + (active ? wave : 0u) * ((cap + 2u) * kColPitch);
    E.col = J.lds0 + (uint32_t)((unsigned char*)rows - smem) + lane * 4u;
    E.recs = reinterpret_cast<uint16_t*>(smem + J.L.recs) + wave * kEncRecs;
    const uint32_t in_group = min(E.rem, kW * (uint32_t)S);
    // a state marked below this many bits (in the trip before it, kTripBits more) has no word of the next pass behind it
    const int limit = (int)(cap * 32u - kTripBits);
    auto last_word = [&](const EmitState& St) {  // the chunk's last, partly filled word
        if (St.nbt & 31u)
            *reinterpret_cast<lds_u32*>(E.col + min((St.nbt >> 5) + 1u, E.row_max) * (kColPitch * 4u)) = (uint32_t)St.acc << (32u - (St.nbt & 31u));
    };
    EmitState St;
    St.acc = 0;
    St.nbt = 0;
    St.nesc = 0;
    EmitMark M;
    M.acc = 0;
    M.nbt = 0;
    M.j = 0;
    if (active) {
        if (J.pairs) {
            if (J.special) M = emit_turns<F16, VEC, true, true, LZ>(E, St, plane, in_group, 0u, limit, true);
            else M = emit_turns<F16, VEC, true, false, LZ>(E, St, plane, in_group, 0u, limit, true);
        } else {
            M = emit_turns<F16, VEC, false, true, LZ>(E, St, plane, in_group, 0u, limit, true);
        }
        last_word(St);
    }
    const uint32_t nw = active ? (St.nbt + 31u) >> 5 : 0u, n_esc = St.nesc;
    const uint32_t incl = wave_incl_scan(nw);
    const uint32_t lane_off = incl - nw;
    const uint32_t chunk_total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    const uint32_t total = chunk_total + 2u * n_esc;  // 0 for an idle wavefront
    if (lane == 0) s_tot[wave] = total;
    __syncthreads();
    if (wave == 0) {
        uint32_t wg_total = 0;
        for (uint32_t k = 0; k < NW; ++k) wg_total += s_tot[k];
        bool failed = false;
        const uint32_t excl = wg_scan(state, epoch, J.wg, wg_total, lane, ctrl, &failed, J.dom0);
        if (lane == 0) { s_excl = excl; s_dead = failed ? 1u : 0u; }
    }
    __syncthreads();
    if (!active) return;
    uint32_t excl = s_excl;
    for (uint32_t k = 0; k < wave; ++k) excl += s_tot[k];
    bool dead = s_dead != 0u;  // nothing may be written to the container
    if (F.off_payload + 4ull * ((uint64_t)excl + total) > capacity) {
        if (!dead && lane == 0) set_status(ctrl, DLC_ECAPACITY);
        dead = true;
    }
    if (lane == 0) {
        if (grp == 0) word_start[t] = excl;
        if (grp == g.G - 1) word_end[t] = excl + total;
    }
    if (dead) return;
    out[F.off_chunk + (uint64_t)gid * kW + lane] = (uint8_t)nw;
    if (lane == 0) reinterpret_cast<uint32_t*>(out + F.off_group)[gid] = excl;
    uint32_t* const gw = reinterpret_cast<uint32_t*>(out + F.off_payload) + excl;
    // the columns come from other lanes of this wavefront: its LDS accesses complete in order, the compiler must keep
    // them in order too
    auto in_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the columns' words to their places; they are the words from `first` on of their chunks.
    // A team of lanes copies a chunk, a word a lane: as many lanes as a chunk has words at 4 bits a symbol, a half or a quarter of
    // them where all chunks are as short (the teams' chunks lie so far apart that no two lanes meet in a bank).  (A table of 4096
    // elements, chunks of 8 words: 1.9 us with teams of 32 lanes.)
    auto copy = [&](uint32_t first) {
        in_order();
        const uint32_t n_here = nw > first ? min(nw - first, cap) : 0u;
        uint32_t log_tl = S == 256 ? 5u : (S == 128 ? 4u : 3u);  // (S / 8)
        if (S > 64 && __ballot(n_here > (uint32_t)S / 16u) == 0ull) --log_tl;
        if (S > 128 && __ballot(n_here > (uint32_t)S / 32u) == 0ull) --log_tl;
        const uint32_t TL = 1u << log_tl, team = lane >> log_tl, k0 = lane & (TL - 1u);
        const uint32_t mine = ((lane_off + first) << 8) | n_here;
        for (uint32_t k = 0; __ballot(n_here > k) != 0ull; k += TL) {  // uniform
            const uint32_t* const rl = rows + min(k + k0 + 1u, cap + 1u) * kColPitch;
#pragma clang loop unroll(disable)
            for (uint32_t i0 = 0; i0 < TL; i0 += 8u) {  // eight chunks in flight: nothing in between waits
                uint32_t oc[8], v[8];
#pragma unroll
                for (uint32_t u = 0; u < 8u; ++u) {
                    const uint32_t c = i0 + u + team * TL;
                    oc[u] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(c * 4u), (int)mine);
                    v[u] = rl[c];
                }
#pragma unroll
                for (uint32_t u = 0; u < 8u; ++u)
                    if (k + k0 < (oc[u] & 255u)) gw[(oc[u] >> 8) + k + k0] = v[u];
            }
        }
    };
    copy(0u);
    for (uint32_t first = cap; __ballot(nw > first) != 0ull; first += cap) {  // uniform; the codewords one by one from here on
        in_order();
        St.acc = M.acc;
        St.nbt = M.nbt - cap * 32u;  // (what is counted from the pass's first word on may be below zero)
        M = emit_turns<F16, VEC, false, true, LZ>(E, St, plane, in_group, M.j, limit, false);
        last_word(St);
        copy(first);
    }
    if (n_esc != 0u) {  // uniform over the wavefront
        uint32_t* rec = gw + chunk_total;
        if (n_esc <= kEncRecs) {  // the records were kept on the way
            for (uint32_t k = lane; k < n_esc; k += 64) {
                const uint32_t off = E.recs[k];
                rec[2u * k] = gstart + off;
                if constexpr (F16) rec[2u * k + 1] = reinterpret_cast<const uint16_t*>(gbase)[off];
                else rec[2u * k + 1] = reinterpret_cast<const uint32_t*>(gbase)[off];
            }
        } else {
            emit_escapes<S, F16, VEC>(rec, lane, gbase, plane, gstart, E.rem);
        }
    }
}

// the pair table of the window indices [lo, lo + P), by NT threads
__device__ __forceinline__ void build_pairs(uint32_t* pair, const uint16_t* ent, uint32_t lo, uint32_t P, uint32_t tid, uint32_t nt) {
    const uint32_t magic = (1u << 20) / P + 1u;  // i / P for i < P * P <= 63 * 63: exact
    for (uint32_t i = tid; i < P * P; i += nt) {
        const uint32_t a = (i * magic) >> 20, b = i - a * P;
        pair[i] = pair_entry(ent[lo + a], ent[lo + b]);
    }
}

// ------------------------------------------------------------------------------------------------
// groups of tables of any size, from the symbol plane, with the codebooks in memory
// ------------------------------------------------------------------------------------------------
// The `per` (NW at most) groups from J.wg % bpt * per on of table J.wg / bpt.  WITHIN: the codebook and the plane come from other work-groups of this launch
// (of the plane nothing has been read before, so there is nothing old of it in a cache; the codebook's lines hold other tables' too).
template <int S, bool F16, bool VEC, bool LZ, uint32_t NW, bool WITHIN>
__device__ __forceinline__ void encode_item(GroupJob& J, const void* payload, const uint8_t* sym_plane, const Geom& g, const FixedLayout& F,
                                            const QParam* qp, const uint16_t* enc, const TMeta* tmeta, Ctrl* ctrl, uint64_t* state, uint64_t epoch,
                                            uint8_t* out, uint64_t capacity, uint32_t bpt, uint32_t per, uint32_t* word_start, uint32_t* word_end,
                                            uint32_t cap, uint32_t pair_max, uint32_t* s_lo, uint32_t* s_hi, unsigned char* smem, uint32_t tid) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    J.t = J.wg / bpt;
    J.grp = wave < per ? (J.wg % bpt) * per + wave : g.G;
    // the destination this table belongs to: its container starts `capacity` bytes after the previous one, its
    // groups are numbered and its words are placed from 0, so the scan over work-groups starts anew at its first
    J.dst = J.t / g.TD;
    J.tl = J.t - J.dst * g.TD;
    J.dom0 = J.dst * g.TD * bpt;
    J.cap = cap;
    J.lds0 = (uint32_t)(uintptr_t)smem;
    J.L = enc_lds(NW, per, cap, pair_max);
    const uint32_t win_lo = win_lo_of(g.R);
    const uint16_t* enc_t = enc + (size_t)J.t * g.K;
    uint16_t* ent = reinterpret_cast<uint16_t*>(smem + J.L.ent);
    const TMeta tm = load_tmeta<WITHIN>(tmeta + J.t);
    for (uint32_t i = tid; i < 256u; i += 64u * NW) {
        // (index 254 is the escape, symbol 0; with row matching index 253 marks an element of a row that is stored as
        // a reference: no bits)
        const uint32_t c = win_lo + i;
        const bool sym = i < win_bins(LZ ? 1u : 0u) && c < g.K;
        uint32_t e = 0u;
        if (i == kWinEsc || sym) {
            const uint16_t* p = enc_t + (i == kWinEsc ? 0u : c);
            e = WITHIN ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
        }
        ent[i] = (uint16_t)e;
        // the span of the used symbols inside the window (a table with one used symbol has a code of length 0 for it)
        if (sym && c != 0u && (e != 0u || (tm.n_used == 1u && c == tm.sym_lo))) { atomicMin(s_lo, i); atomicMax(s_hi, i); }
    }
    __syncthreads();
    J.lo = min(*s_lo, *s_hi);
    J.P = *s_hi - J.lo + 1u;
    J.pairs = J.P <= pair_max;
    J.special = tm.n_outliers != 0u || (tm.n_used == 1u && tm.sym_lo == 0u) || (tm.sym_lo != 0u && tm.sym_lo < win_lo) ||
                tm.sym_hi >= win_lo + win_bins(LZ ? 1u : 0u);
    if (J.pairs) {
        build_pairs(reinterpret_cast<uint32_t*>(smem + J.L.pair), ent, J.lo, J.P, tid, 64u * NW);
        __syncthreads();
    }
    encode_groups<S, F16, VEC, LZ, NW>(J, payload, sym_plane, g, F, qp, enc, ctrl, state, epoch, out + (uint64_t)J.dst * capacity,
                                       capacity, word_start, word_end, smem, tid);
}

template <int S, bool F16, bool VEC, bool LZ, uint32_t NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
void k_encode(const void* payload, const uint8_t* sym_plane, Geom g, FixedLayout F, const QParam* qp, const uint16_t* enc,
              const TMeta* tmeta, const uint8_t* lens, Ctrl* ctrl, uint64_t* state, uint64_t epoch, uint8_t* out, uint64_t capacity, uint32_t bpt,
              uint32_t* word_start, uint32_t* word_end, uint64_t* out_bytes, uint32_t xn, uint32_t cap, uint32_t pair_max, const uint8_t* rm_on,
              const uint32_t* rm_ref) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_wg, s_lo, s_hi;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) { s_wg = atomicAdd(&ctrl->ticket, 1u); s_lo = 255u; s_hi = 0u; }
    __syncthreads();
    GroupJob J;
    J.wg = __builtin_amdgcn_readfirstlane(s_wg);
    if (J.wg >= g.T * bpt) {  // uniform; xn for every container
        finish_container<64u * NW, false, LZ>(g, F, tmeta, lens, qp, ctrl, state, (const uint32_t*)nullptr, epoch, bpt, out, capacity, out_bytes, J.wg - g.T * bpt, xn, *reinterpret_cast<FinLds<64u * NW>*>(smem), tid, rm_on, rm_ref);
        return;
    }
    encode_item<S, F16, VEC, LZ, NW, false>(J, payload, sym_plane, g, F, qp, enc, tmeta, ctrl, state, epoch, out, capacity, bpt, NW, word_start, word_end,
                                            cap, pair_max, &s_lo, &s_hi, smem, tid);
}

// ------------------------------------------------------------------------------------------------
// tables of more groups than one work-group takes: quantise, count, codebook, encode in one launch
//   Work-groups take tickets in the order in which they start.  Of every table there are `cpt` tickets to count a share of it (plane out, past
//   the caches; counts added to the table's), the last of which to finish builds the codebook, and `ept` to code `gpe` groups each, which
//   wait for that.  The tickets to code a table come `lag` tables after those to count it, so the codebook is there when they start;
//   whoever is waited for has an earlier ticket and waits for nobody (counting) or for still earlier ones (the scan).  With no more
//   tables than that (up to 311296 units of 256 elements, 524288 in half precision, or nearly; of 128 tables of 8192 x 128 76 are ahead) all counting
//   tickets come first, and what overlaps is the end of the counting with the codebooks and the first tables' coding, instead of two gaps.
//   What bounds it: memory (512 MiB: payload read, plane out and in, words out, 862 MB in 162 us; the last table is counted at 135), then
//   the last tables' chain of codebook 7, tables 2, walk 9, scan 4 and copy 3 us.  Three launches, each of which ends with a part of the
//   chip, take 178 us where this takes 163; 300 tables of 262144 elements 123 and 108.
// ------------------------------------------------------------------------------------------------
struct FlowPlan {
    uint32_t cpt, units;  // tickets to count a table, units each (a multiple of kHistBlk)
    uint32_t ept, gpe;    // tickets to code a table, groups each
    uint32_t lag;         // tables counted before the first is coded
    uint32_t tickets;     // in all
};
constexpr uint32_t kFlowWaves = 8;

template <int S, bool F16, bool VEC>
__global__ __launch_bounds__(64 * kFlowWaves) __attribute__((amdgpu_waves_per_eu(4)))
void k_flow(const void* payload, uint8_t* sym_plane, Geom g, FixedLayout F, const QParam* qp, uint32_t* hist, uint32_t* hist_view, uint16_t* enc,
            uint8_t* lens, TMeta* tmeta, Ctrl* ctrl, uint64_t* state, uint32_t* ready, uint32_t* arrived, uint64_t epoch, uint8_t* out, uint64_t capacity,
            FlowPlan P, uint32_t* word_start, uint32_t* word_end, uint64_t* out_bytes, uint32_t xn, uint32_t cap, uint32_t pair_max) {
    constexpr uint32_t NW = kFlowWaves, NT = 64u * NW;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ CodebookShared s_cb;
    __shared__ uint32_t s_ticket, s_lo, s_hi, s_go;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) { s_ticket = atomicAdd(&ctrl->ticket, 1u); s_lo = 255u; s_hi = 0u; }
    __syncthreads();
    const uint32_t ticket = __builtin_amdgcn_readfirstlane(s_ticket);
    if (ticket + 1u == gridDim.x && tid == 0) __hip_atomic_store(&ctrl->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // (the last of all)
    if (ticket >= P.tickets) return;  // uniform; a spare work-group
    // ticket -> what to do: the first `lag` tables' counting; a table's counting and the coding of the table `lag` before it; the last tables' coding
    uint32_t t, r;
    bool count = true;
    {
        const uint32_t head = P.lag * P.cpt, per = P.cpt + P.ept, body = (g.T - P.lag) * per;
        if (ticket < head) {
            t = ticket / P.cpt;
            r = ticket - t * P.cpt;
        } else if (ticket - head < body) {
            const uint32_t i = ticket - head, k = i / per;
            r = i - k * per;
            count = r < P.cpt;
            t = count ? P.lag + k : k;
            r = count ? r : r - P.cpt;
        } else {
            const uint32_t i = ticket - head - body;
            t = i / P.ept;
            r = i - t * P.ept;
            t += g.T - P.lag;
            count = false;
        }
    }
    if (t >= g.T) {  // uniform; xn for every container
        finish_container<NT, true, false, false>(g, F, tmeta, lens, qp, ctrl, state, ready, epoch, P.ept, out, capacity, out_bytes, ticket - g.T * (P.cpt + P.ept), xn, *reinterpret_cast<FinLds<NT>*>(smem), tid);
        return;
    }
    if (count) {
        uint32_t* const lh = reinterpret_cast<uint32_t*>(smem);
        {
            uint4* z = reinterpret_cast<uint4*>(lh);
            const uint32_t n4 = ((kWinBins + 1u) * kWinCopies + g.K + 3u) / 4u;
            for (uint32_t k = tid; k < n4; k += NT) z[k] = make_uint4(0, 0, 0, 0);
        }
        __syncthreads();
        {
            const QParam q = qp[t];
            const HistC H = hist_consts<false>(g, q, (uint32_t)(uintptr_t)smem, lane);
            const uint32_t U = (g.n + kW * kV - 1u) / (kW * kV), u0 = r * P.units;
            hist_units<F16, VEC, NW, kPlaneThrough>(static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es, sym_plane + (size_t)t * plane_stride(g), g,
                                                    u0, min(U, u0 + P.units), wave, lane, q, H);
        }
        __syncthreads();
        hist_merge<false, NT>(lh, g, hist + (size_t)t * g.K, tid);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this work-group's plane and counts are in memory
        __syncthreads();
        if (tid == 0) {
            const bool last = __hip_atomic_fetch_add(&arrived[t], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == P.cpt;
            if (last) __hip_atomic_store(&arrived[t], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_go = last ? 1u : 0u;
        }
        __syncthreads();
        if (s_go == 0u) return;  // uniform
        codebook_build<NT>(g, hist + (size_t)t * g.K, hist_view + (size_t)t * g.K, enc + (size_t)t * g.K, lens + (size_t)t * g.K, tmeta + t, smem, s_cb, tid, 0u, true);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) table_ready(ready, epoch, t);
        return;
    }
    if (tid == 0) {
        bool there = true;
        for (uint32_t spins = 0; __hip_atomic_load(&ready[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (uint32_t)epoch; ++spins) {
            if (spins > kSpinLimit) {  // never expected; the bound only guarantees termination
                set_status(ctrl, DLC_ESTATE);
                atomicOr(&ctrl->abort, 1u);
                there = false;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        s_go = there ? 1u : 0u;
    }
    __syncthreads();
    if (s_go == 0u) return;  // uniform (those behind find no record of this one and give up as well)
    GroupJob J;
    J.wg = t * P.ept + r;
    encode_item<S, F16, VEC, false, NW, true>(J, payload, sym_plane, g, F, qp, enc, tmeta, ctrl, state, epoch, out, capacity, P.ept, P.gpe, word_start, word_end,
                                              cap, pair_max, &s_lo, &s_hi, smem, tid);
}

// ------------------------------------------------------------------------------------------------
// small tables: quantise, count, codebook, encode, a work-group per table
//   The counts of a table are complete when its work-group's barrier says so, so the codebook needs no launch of its
//   own and nothing waits for another work-group before the scan.  The payload is read once; the symbol plane goes
//   through the caches.  What bounds it: with few tables the chain of latencies (loads, one wavefront's tree, the
//   walk: one table of 4096 elements 14 us, where three launches took 61), with many the counting phase (4096 tables of two
//   groups: 216 us, the three launches 283).
// ------------------------------------------------------------------------------------------------
template <int S, bool F16, bool VEC, uint32_t NW, bool FIN>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
void k_table(const void* payload, uint8_t* sym_plane, Geom g, FixedLayout F, const QParam* qp, uint32_t* hist_view, uint16_t* enc,
             uint8_t* lens, TMeta* tmeta, Ctrl* ctrl, uint64_t* state, uint32_t* ready, uint64_t epoch, uint8_t* out, uint64_t capacity,
             uint32_t* word_start, uint32_t* word_end, uint64_t* out_bytes, uint32_t xn, uint32_t cap, uint32_t pair_max) {
    constexpr uint32_t NT = 64u * NW;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ CodebookShared s_cb;
    __shared__ uint32_t s_cnt[256];
    __shared__ uint64_t s_key[65];
    __shared__ TMeta s_tm;
    __shared__ uint32_t s_wg, s_lo, s_hi, s_fast, s_out;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) { s_wg = atomicAdd(&ctrl->ticket, 1u); s_lo = 255u; s_hi = 0u; s_fast = 0u; s_out = 0u; }
    // counts: window rows and exact counts, as in the histogram kernel
    uint32_t* const lh = reinterpret_cast<uint32_t*>(smem);
    const uint32_t* const exact = lh + (kWinBins + 1u) * kWinCopies;
    {
        uint4* z = reinterpret_cast<uint4*>(lh);
        const uint32_t n4 = ((kWinBins + 1u) * kWinCopies + g.K + 3u) / 4u;
        for (uint32_t k = tid; k < n4; k += NT) z[k] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    GroupJob J;
    J.wg = __builtin_amdgcn_readfirstlane(s_wg);
    if constexpr (FIN) {
        if (J.wg >= g.T) {  // uniform; xn for every container
            finish_container<NT, true>(g, F, tmeta, lens, qp, ctrl, state, ready, epoch, 1u, out, capacity, out_bytes, J.wg - g.T, xn, *reinterpret_cast<FinLds<NT>*>(smem), tid);
            return;
        }
    }
    const uint32_t t = J.wg;  // a work-group per table, in ticket order
    J.t = t;
    J.grp = wave;
    J.dst = t / g.TD;
    J.tl = t - J.dst * g.TD;
    J.dom0 = J.dst * g.TD;
    J.cap = cap;
    J.lds0 = (uint32_t)(uintptr_t)smem;
    J.L = enc_lds(NW, min(NW, g.G), cap, pair_max);
    {
        const QParam q = qp[t];
        const HistC H = hist_consts<false>(g, q, J.lds0, lane);
        const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
        uint8_t* plane_t = sym_plane + (size_t)t * plane_stride(g);
        hist_units<F16, VEC, NW, kPlane>(tab, plane_t, g, 0u, (g.n + kW * kV - 1u) / (kW * kV), wave, lane, q, H);
    }
    __syncthreads();
    for (uint32_t r = tid; r < 256u; r += NT) {  // the copies of a row (skewed start: different banks)
        uint32_t s = 0;
        for (uint32_t c = 0; c < kWinCopies; ++c) s += lh[r * kWinCopies + ((c + r) & (kWinCopies - 1u))];
        s_cnt[r] = s;
        const uint64_t used = __ballot(r < kWinEsc && s != 0u);  // (whole wavefronts: 256 is a multiple of NT or NT of 256)
        if (used != 0ull && lane == 0) {
            atomicMin(&s_lo, r + (uint32_t)__builtin_ctzll(used));
            atomicMax(&s_hi, r + 63u - (uint32_t)__builtin_clzll(used));
        }
    }
    __syncthreads();
    const uint32_t n_other = s_cnt[kWinBins];  // elements outside the window (counted exactly, by symbol)
    uint32_t* const view_t = hist_view + (size_t)t * g.K;
    uint16_t* const enc_t = enc + (size_t)t * g.K;
    uint8_t* const lens_t = lens + (size_t)t * g.K;
    const uint32_t win_lo = win_lo_of(g.R);
    auto in_window = [&](uint32_t k, uint32_t& idx) {  // symbol -> window index
        idx = k == 0u ? kWinEsc : k - win_lo;
        return k == 0u || (k >= win_lo && idx < kWinEsc);
    };
    // A table's counts (inspection, and the codebook of the next call where it is carried), codewords and lengths by `nt` threads.
    // (No element outside the window: the exact counts are zero.)
    auto put_counts = [&](uint32_t first, uint32_t nt) {
        for (uint32_t k = first; k < g.K; k += nt) {
            uint32_t idx;
            const uint32_t s = (in_window(k, idx) ? s_cnt[idx] : 0u) + (n_other != 0u ? exact[k] : 0u);
            __hip_atomic_store(&view_t[k], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    uint16_t* const ent = reinterpret_cast<uint16_t*>(smem + J.L.ent);
    auto put_codes = [&](uint32_t first, uint32_t nt) {
        for (uint32_t k = first; k < g.K; k += nt) {
            uint32_t idx;
            const uint32_t e = in_window(k, idx) ? ent[idx] : 0u;
            enc_t[k] = (uint16_t)e;
            if constexpr (FIN) __hip_atomic_store(&lens_t[k], (uint8_t)(e >> 12), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else lens_t[k] = (uint8_t)(e >> 12);
        }
        if (first == 0u) store_tmeta(tmeta + t, s_tm);
    };
    if (n_other == 0u) {  // uniform
        if (wave == 0) {
            const bool done = codebook_window_wave(g, s_cnt, s_key, ent, &s_tm, lane);
            if (lane == 0) s_fast = done ? 1u : 0u;
        }
        __syncthreads();
    }
    // Wavefronts without a group put what nobody in the work-group reads into memory while the others code theirs (with one group of
    // 4096 elements that and the wait for it were 1.3 us of the work-group's 13)
    const bool fast = s_fast != 0u, apart = fast && g.G < NW;
    if (fast) {  // uniform
        if (!apart) {
            put_counts(tid, NT);
            put_codes(tid, NT);
        }
    } else {  // many symbols, or symbols outside the window: from the counts in memory
        put_counts(tid, NT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        codebook_build<NT>(g, view_t, view_t, enc_t, lens_t, tmeta + t, smem, s_cb, tid, 0u, FIN);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        for (uint32_t i = tid; i < 256u; i += NT) {
            const uint32_t k = i == kWinEsc ? 0u : win_lo + i;
            ent[i] = i <= kWinEsc && k < g.K ? __hip_atomic_load(&enc_t[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (uint16_t)0;
        }
        __syncthreads();
    }
    J.lo = min(s_lo, s_hi);
    J.P = s_hi - J.lo + 1u;
    J.pairs = J.P <= pair_max;
    J.special = n_other != 0u || s_cnt[kWinEsc] != 0u;
    if (J.pairs) {
        build_pairs(reinterpret_cast<uint32_t*>(smem + J.L.pair), ent, J.lo, J.P, tid, NT);
    }
    if (FIN && !apart) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the codebook is out)
    __syncthreads();
    if (!apart) {
        if (FIN && tid == 0) table_ready(ready, epoch, t);
    } else if (wave >= g.G) {
        put_counts(tid - 64u * g.G, NT - 64u * g.G);
        put_codes(tid - 64u * g.G, NT - 64u * g.G);
        if constexpr (FIN) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0 && atomicAdd(&s_out, 1u) + 1u == NW - g.G) table_ready(ready, epoch, t);  // the last of them
        }
    }
    encode_groups<S, F16, VEC, false, NW>(J, payload, sym_plane, g, F, qp, enc, ctrl, state, epoch, out + (uint64_t)J.dst * capacity,
                                          capacity, word_start, word_end, smem, tid);
}

// ---- launches ------------------------------------------------------------------------------------------------------
constexpr uint32_t kLdsMax = 160u * 1024u;        // of a compute unit
constexpr uint32_t kTableStatic = 3072u;          // LDS that k_table declares itself (rounded up)
constexpr uint32_t kEncStatic = 256u;
constexpr uint32_t kEncLdsMax = kLdsMax - kEncStatic;

// the pair table gets what is left of `budget`
static inline uint32_t pair_max_for(uint32_t budget, uint32_t nw, uint32_t waves, uint32_t cap) {
    uint32_t p = kPairMax;
    while (p > 8u && enc_lds(nw, waves, cap, p).end > budget) --p;
    return p;
}

constexpr uint32_t kFinishMost = 128;  // work-groups a container that copy its references

// out_bytes: where the sizes go if the launch is to finish the containers as well; it does if it returns true
template <uint32_t NW>
static bool DLC_CAT(encode_launch_, DLC_S)(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch,
                                           uint8_t* out, uint64_t capacity, uint64_t* out_bytes, hipStream_t s) {
    constexpr int S = DLC_S;
    const uint32_t bpt = (g.G + NW - 1u) / NW;
    uint32_t xn = finish_groups(g, 64u * NW);
    if (g.lz) xn = std::max(xn, std::min<uint32_t>(kFinishMost, (uint32_t)(((uint64_t)g.TD * g.B + 64u * NW * kFinishRefs - 1u) / (64u * NW * kFinishRefs))));
    // (With row matching up to as many references as so many work-groups load at once; more in a launch of their own: with 64
    // work-groups that go round again 64 tables of 16384 x 32 138 us instead of 134, with 128 135, 128 of 8192 x 128 279 and 275.)
    if (g.TD > 64u * NW || (g.lz && (uint64_t)g.TD * g.B > (uint64_t)kFinishMost * 64u * NW * kFinishRefs)) out_bytes = nullptr;
    dim3 grid(g.T * bpt + (out_bytes ? g.ND * xn : 0u)), block(64 * NW);
    // sixteen wavefronts a compute unit share its LDS: columns of 4 bits a symbol.  Where the grid leaves room, longer
    // columns (up to the longest code), so that no group is walked twice.
    const uint32_t per_cu = std::min(16u / NW, std::max(1u, (g.T * bpt + 255u) / 256u));
    const uint32_t budget = std::min(kLdsMax / per_cu, kEncLdsMax) - kEncStatic;
    uint32_t cap = (uint32_t)S * 12u / 32u;
    while (cap > (uint32_t)S / 8u && enc_lds(NW, NW, cap, 56u).end > budget) --cap;
    const uint32_t pair_max = pair_max_for(budget, NW, NW, cap);
    size_t sm = enc_lds(NW, NW, cap, pair_max).end;
    if (out_bytes) sm = std::max(sm, sizeof(FinLds<64u * NW>));
    const bool f16 = g.dtype == DLC_F16;
#define DLC_ENC(FF, V, LZ)                                                                                            \
    hipLaunchKernelGGL((k_encode<S, FF, V, LZ, NW>), grid, block, sm, s, payload, w.sym_plane, g, F, w.qp, w.enc, w.tmeta, w.lens, w.ctrl, \
                       w.state, epoch, out, capacity, bpt, w.word_start, w.word_end, out_bytes, xn, cap, pair_max, w.rm_on, w.rm_ref)
    if (g.lz) { if (f16) DLC_ENC(true, true, true); else DLC_ENC(false, true, true); }  // (dim % 4 == 0 there)
    else if (f16) { if (g.vec) DLC_ENC(true, true, false); else DLC_ENC(true, false, false); }
    else { if (g.vec) DLC_ENC(false, true, false); else DLC_ENC(false, false, false); }
#undef DLC_ENC
    return out_bytes != nullptr;
}

bool DLC_CAT(launch_encode_, DLC_S)(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch,
                                    uint8_t* out, uint64_t capacity, uint64_t* out_bytes, hipStream_t s) {
    // four groups a work-group where that spreads a small payload over more compute units
    if (g.G <= 4u || g.T * ((g.G + 3u) / 4u) <= 512u) return DLC_CAT(encode_launch_, DLC_S)<4u>(g, F, payload, w, epoch, out, capacity, out_bytes, s);
    return DLC_CAT(encode_launch_, DLC_S)<8u>(g, F, payload, w, epoch, out, capacity, out_bytes, s);
}

// Counting, codebooks and coding in one launch (out_bytes as above)
bool DLC_CAT(launch_flow_, DLC_S)(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch,
                                  uint8_t* out, uint64_t capacity, uint64_t* out_bytes, hipStream_t s) {
    constexpr int S = DLC_S;
    constexpr uint32_t NW = kFlowWaves;
    if (g.TD > 64u * NW) out_bytes = nullptr;
    const uint32_t xn = finish_groups(g, 64u * NW);
    FlowPlan P;
    // Shares of a table alike, 1024 in all, two rounds of the work-groups that run at a time, so that what a share costs
    // besides its loads (3 us: counters cleared, counts added) is little; but no larger than 256 KiB of fp32 (512 MiB: 2048 of them) where memory bounds the
    // counting (512 MiB by 128, 256 and 512 units 175, 171 and 177 us), 512 units where it does not (half precision 241, 208 and 188).
    const uint32_t U = (g.n + kW * kV - 1u) / (kW * kV), most = g.dtype == DLC_F16 ? 512u : 256u;
    const uint32_t want = (uint32_t)std::min<uint64_t>(most, std::max<uint64_t>(64u, (uint64_t)g.T * U / 1024u));
    const uint32_t shares = (U + want - 1u) / want;
    P.units = ((U + shares - 1u) / shares + kHistBlk - 1u) / kHistBlk * kHistBlk;
    P.cpt = (U + P.units - 1u) / P.units;
    // Eight groups a ticket, fewer where there would not be a ticket for every compute unit: groups that take long need the units more
    // than the tables in LDS cost (40 tables of 4096 x 128, 1280 groups, at 0.001 of the range 358 us with eight, 324 with five, 341 by
    // three launches; at 0.03, where a ticket takes 20 us, 12 of 16384 x 128 55.3 and 56.9, by three launches 61.2).  Not in half precision:
    // 3 tables of 60000 x 128 at 0.03 70 us with eight, 72 with five, 100 of 4000 x 48 at 0.001, eight, 454, by three launches 447.
    P.gpe = g.dtype == DLC_F16 ? NW : std::min(NW, std::max(1u, g.NG / 256u));
    P.ept = (g.G + P.gpe - 1u) / P.gpe;
    // As many shares ahead as to have a table counted when its coding starts, with all of the work-groups between at work, and a fifth
    // more: a codebook of hundreds of symbols takes 130 us, and the tickets that wait for it keep those behind them, which count,
    // from starting.  (Us at 1024, 1216 and 1600 shares: 128 tables of 8192 x 128 at bounds of 0.03, 0.002 and 0.001 of the range 162.9, 162.9
    // and 164.2, 296, 283 and 242, 806, 778 and 747, by three launches 785 at the last; 400 of them at 0.03 484, 490 and 501: more tables
    // are coded alone at the end.  In half precision, with shares twice as large, 128 of 16384 x 128 391, 396 and 394.)
    P.lag = std::min(g.T, ((g.dtype == DLC_F16 ? 1024u : 1216u) + P.cpt - 1u) / P.cpt);
    P.tickets = g.T * (P.cpt + P.ept) + (out_bytes ? g.ND * xn : 0u);
    // An eighth more work-groups than tickets: the hardware gives every XCD as many work-groups as the others, whatever theirs have to do,
    // so the XCDs whose tickets took long have as many left to start when the tickets of the others run out.  Spare ones end at
    // once.  Not where every coding ticket can have a compute unit to itself: where they go as they are dealt they nearly do.
    // (Us, without and with: 64 tables of 8192 x 128, 512 coding tickets, at bounds of 0.001, 0.003 and 0.03 of the range 558 and 480, 163 and 161, 98.4 and
    // 97.5, 64 of 16384 x 128 in half precision, 1024, at 0.001 864 and 812, at 0.03 190 and 190; one table of 500000 x 64 in half precision, 245, at 0.03
    // and 0.003 75.9 and 78.4, 168 and 173, one of 262144 x 128, 256, at 0.03 and 0.001 68.7 and 71.2, 301 and 308, 40 of 4096 x 128 327 and 325.)
    const uint32_t n_wg = P.tickets + (g.T * P.ept > 256u ? P.tickets / 8u : 0u);
    const uint32_t budget = kLdsMax / 2u - kTableStatic;
    uint32_t cap = (uint32_t)S * 12u / 32u;
    while (cap > (uint32_t)S / 8u && enc_lds(NW, P.gpe, cap, 60u).end > budget) --cap;
    const uint32_t pair_max = pair_max_for(budget, NW, P.gpe, cap);
    size_t sm = std::max((size_t)enc_lds(NW, P.gpe, cap, pair_max).end, std::max(hist_lds_bytes(g.K), codebook_smem(g.K)));
    if (out_bytes) sm = std::max(sm, sizeof(FinLds<64u * NW>));
    const bool f16 = g.dtype == DLC_F16;
#define DLC_FLOW(FF, V)                                                                                               \
    hipLaunchKernelGGL((k_flow<S, FF, V>), dim3(n_wg), dim3(64u * NW), sm, s, payload, w.sym_plane, g, F, w.qp, w.hist, w.hist_view, w.enc, w.lens, \
                       w.tmeta, w.ctrl, w.state, w.ready, w.arrived, epoch, out, capacity, P, w.word_start, w.word_end, out_bytes, xn, cap, pair_max)
    if (f16) { if (g.vec) DLC_FLOW(true, true); else DLC_FLOW(true, false); }
    else { if (g.vec) DLC_FLOW(false, true); else DLC_FLOW(false, false); }
#undef DLC_FLOW
    return out_bytes != nullptr;
}

template <uint32_t NW>
static bool DLC_CAT(table_launch_, DLC_S)(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch,
                                          uint8_t* out, uint64_t capacity, uint64_t* out_bytes, uint32_t cap, uint32_t budget, uint32_t room, hipStream_t s) {
    constexpr int S = DLC_S;
    const uint32_t xn = finish_groups(g, 64u * NW);
    // A launch that is a single round of tables (`room` work-groups run at a time; 0: it may be several): those that finish the
    // containers have to run beside them, started when the first tables are done they are late (512 tables of 256 elements 28.2
    // us, so 30.4).  Of several rounds the last is seldom full (eight containers, us, a launch of their own and in this one: 768
    // tables of four groups 84, 81, 1536 of two 114, 110, 960 of eight 176, 170, 400 of twelve 123, 118; 4096 of two 360, 354).
    // (A launch without them is an instantiation of its own: with their code in it 520 tables of six groups took 110 us, so 106.)
    if (g.TD > 64u * NW || (room != 0u && g.T + g.ND * xn > room)) out_bytes = nullptr;
    dim3 grid(g.T + (out_bytes ? g.ND * xn : 0u)), block(64 * NW);
    const uint32_t waves = std::min(NW, g.G);
    const uint32_t pair_max = pair_max_for(budget, NW, waves, cap);
    size_t sm = enc_lds(NW, waves, cap, pair_max).end;
    sm = std::max(sm, std::max(hist_lds_bytes(g.K), codebook_smem(g.K)));
    if (out_bytes) sm = std::max(sm, sizeof(FinLds<64u * NW>));
    const bool f16 = g.dtype == DLC_F16;
#define DLC_TAB2(FF, V, FIN)                                                                                          \
    hipLaunchKernelGGL((k_table<S, FF, V, NW, FIN>), grid, block, sm, s, payload, w.sym_plane, g, F, w.qp, w.hist_view, w.enc, w.lens, w.tmeta, \
                       w.ctrl, w.state, w.ready, epoch, out, capacity, w.word_start, w.word_end, out_bytes, xn, cap, pair_max)
#define DLC_TAB(FF, V) do { if (out_bytes) DLC_TAB2(FF, V, true); else DLC_TAB2(FF, V, false); } while (0)
    if (f16) { if (g.vec) DLC_TAB(true, true); else DLC_TAB(true, false); }
    else { if (g.vec) DLC_TAB(false, true); else DLC_TAB(false, false); }
#undef DLC_TAB
#undef DLC_TAB2
    return out_bytes != nullptr;
}

bool DLC_CAT(launch_table_, DLC_S)(const Geom& g, const FixedLayout& F, const void* payload, const Ws& w, uint64_t epoch,
                                   uint8_t* out, uint64_t capacity, uint64_t* out_bytes, hipStream_t s) {
    constexpr uint32_t S = DLC_S;
    if (g.T <= 256u) {
        // no more tables than compute units: a work-group has one to itself.  Sixteen wavefronts read a table of more than
        // one unit each; the columns are as long as the LDS allows (12 bits a symbol is the longest code)
        uint32_t cap = S * 12u / 32u;
        while (cap > S / 8u && enc_lds(16u, std::min(16u, g.G), cap, 56u).end > kLdsMax - kTableStatic) --cap;
        if (g.n <= 16u * kW * kV) return DLC_CAT(table_launch_, DLC_S)<4u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax - kTableStatic, 256u, s);
        return DLC_CAT(table_launch_, DLC_S)<16u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax - kTableStatic, 256u, s);
    } else if (g.T <= 512u && g.G <= 8u) {
        // two work-groups of eight wavefronts a compute unit, one round of them, with columns as long as that leaves.  (Two
        // wavefronts for tables of one or two groups: 300 tables of one group at ratios of 10 and 4.9 37 and 103 us a call, so 33
        // and 86; of four groups, four wavefronts: 50 and 117, so 51 and 112.)
        uint32_t cap = S * 12u / 32u;
        while (cap > S / 8u && enc_lds(8u, g.G, cap, 40u).end > kLdsMax / 2u - kTableStatic) --cap;
        return DLC_CAT(table_launch_, DLC_S)<8u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax / 2u - kTableStatic, 512u, s);
    } else {
        // Several rounds of work-groups, or a chip that smaller ones fill.  A compute unit holds, by registers (91 a lane: five
        // wavefronts a SIMD) or by LDS, six work-groups of two wavefronts, five of four (three with the LDS of tables of three and
        // four groups) and two of eight.  Twice as many wavefronts as a table has groups share the counting and take less time a
        // table, but more tables may then need one more round (us, with fewer and with more wavefronts: 2048 tables of one group 118,
        // 109, 1400, which six to a compute unit do in one round, 81, 91, 3072, two rounds, 144, 148; 1024 of four groups 129, 118,
        // 768 90, 104, 1400 154, 160, 2048 221, 218; of three groups 3000 255, 264).
        const uint32_t cap = S / 8u;
        if (g.G <= 2u) {
            const uint32_t rounds = (g.T + 1535u) / 1536u;
            if (rounds <= 2u && g.T > rounds * 1536u - 256u) return DLC_CAT(table_launch_, DLC_S)<2u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax / 6u - kTableStatic, 0u, s);
            return DLC_CAT(table_launch_, DLC_S)<4u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax / 6u - kTableStatic, 0u, s);
        }
        if (g.G <= 4u) {
            if (g.T <= 768u || (g.T > 1024u && (g.T <= 1536u || g.G == 3u)))
                return DLC_CAT(table_launch_, DLC_S)<4u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax / 3u - kTableStatic, 0u, s);
            return DLC_CAT(table_launch_, DLC_S)<8u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax / 3u - kTableStatic, 0u, s);
        }
        if (g.G <= 8u) return DLC_CAT(table_launch_, DLC_S)<8u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax / 2u - kTableStatic, 0u, s);
        return DLC_CAT(table_launch_, DLC_S)<16u>(g, F, payload, w, epoch, out, capacity, out_bytes, cap, kLdsMax - kTableStatic, 0u, s);
    }
}

template <uint32_t NW, bool FIN>
static hipError_t DLC_CAT(encode_attributes_, DLC_S)() {
    constexpr int S = DLC_S;
    const int bytes = (int)(kLdsMax - kTableStatic);
    const void* ks[] = {reinterpret_cast<const void*>(k_table<S, false, false, NW, FIN>), reinterpret_cast<const void*>(k_table<S, false, true, NW, FIN>),
                        reinterpret_cast<const void*>(k_table<S, true, false, NW, FIN>), reinterpret_cast<const void*>(k_table<S, true, true, NW, FIN>)};
    for (const void* k : ks) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t DLC_CAT(encode_set_attributes_, DLC_S)() {
    constexpr int S = DLC_S;
    hipError_t e = DLC_CAT(encode_attributes_, DLC_S)<2u, false>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<2u, true>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<4u, false>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<4u, true>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<8u, false>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<8u, true>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<16u, false>();
    if (e == hipSuccess) e = DLC_CAT(encode_attributes_, DLC_S)<16u, true>();
    const void* ks[] = {reinterpret_cast<const void*>(k_encode<S, false, false, false, 8u>), reinterpret_cast<const void*>(k_encode<S, false, true, false, 8u>),
                        reinterpret_cast<const void*>(k_encode<S, true, false, false, 8u>), reinterpret_cast<const void*>(k_encode<S, true, true, false, 8u>),
                        reinterpret_cast<const void*>(k_encode<S, false, true, true, 8u>), reinterpret_cast<const void*>(k_encode<S, true, true, true, 8u>),
                        reinterpret_cast<const void*>(k_encode<S, false, false, false, 4u>), reinterpret_cast<const void*>(k_encode<S, false, true, false, 4u>),
                        reinterpret_cast<const void*>(k_encode<S, true, false, false, 4u>), reinterpret_cast<const void*>(k_encode<S, true, true, false, 4u>),
                        reinterpret_cast<const void*>(k_encode<S, false, true, true, 4u>), reinterpret_cast<const void*>(k_encode<S, true, true, true, 4u>)};
    for (const void* k : ks)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kEncLdsMax);
    const void* fs[] = {reinterpret_cast<const void*>(k_flow<S, false, false>), reinterpret_cast<const void*>(k_flow<S, false, true>),
                        reinterpret_cast<const void*>(k_flow<S, true, false>), reinterpret_cast<const void*>(k_flow<S, true, true>)};
    for (const void* k : fs)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsMax - kTableStatic));
    return e;
}

}  // namespace dlc
