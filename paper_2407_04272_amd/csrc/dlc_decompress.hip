// Decompression kernels for gfx950: container validation, decode tables and chunk-parallel decode in one kernel,
// escape scatter, row copies.
#include <stddef.h>

#include <algorithm>

#include "dlc_internal.h"

namespace dlc {

__device__ __forceinline__ uint64_t d_a16(uint64_t x) { return (x + 15ull) & ~15ull; }

// What a work-group learns from the container about the table it decodes.  Every range test is written without an
// addition on the untrusted side (an offset near 2^64 must fail the test, not wrap past it).
struct DecHead {
    bool ok;
    uint32_t n_used, sym_lo, sym_hi, n_esc;
    float ebx2;
    uint64_t cb;           // byte offset of the table's code lengths
    uint64_t ref_off;      // row matching: byte offset of the table's u32 ref[B], 0 = none
    uint64_t words_total;  // payload words of the container
    uint64_t n_esc_total;  // escapes of the container
};

// Header against the context's geometry, the table's directory entry against the header.  `comp` is the start of the
// container, `comp_bytes` the room it has; `tl` the table's place in the container.  The same for every thread.
__device__ __forceinline__ DecHead dec_validate(const Geom& g, const FixedLayout& F, const uint8_t* comp,
                                                uint64_t comp_bytes, uint32_t tl) {
    DecHead H;
    H.ok = false; H.n_used = 0; H.sym_lo = 0; H.sym_hi = 0; H.n_esc = 0; H.ebx2 = 0.f; H.cb = 0; H.ref_off = 0;
    H.words_total = 0; H.n_esc_total = 0;
    if (comp_bytes < F.off_payload) return H;  // header, directory, group and chunk tables: their size is the geometry's
    // header and directory entry are read together (no test between the loads), then looked at
    const uint32_t* h = reinterpret_cast<const uint32_t*>(comp);
    const uint64_t* q = reinterpret_cast<const uint64_t*>(comp);
    const uint8_t* d = comp + kHeaderBytes + (uint64_t)kDirBytes * tl;
    const uint32_t* d32 = reinterpret_cast<const uint32_t*>(d);
    const uint64_t* d64 = reinterpret_cast<const uint64_t*>(d + 24);
    uint32_t hw[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) hw[k] = h[k];
    uint64_t hq[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) hq[k] = q[HQ_NOUT + k];
    uint32_t dw[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) dw[k] = d32[k];
    const uint64_t d_cb = d64[0], d_ref = d64[1];
    bool ok = hw[H_MAGIC] == kMagic && hw[H_VERSION] == kVersion && hw[H_DTYPE] == g.dtype && hw[H_T] == g.TD &&
              hw[H_B] == g.B && hw[H_D] == g.D && hw[H_R] == g.R && hw[H_S] == g.S && hw[H_LMAX] == g.LMAX &&
              hw[H_W] == kW && hw[H_V] == kV && hw[H_NG] == g.TD * g.G;
    H.n_esc_total = hq[HQ_NOUT - HQ_NOUT];
    H.words_total = hq[HQ_WORDS - HQ_NOUT];
    const uint64_t off_cb = hq[HQ_OFF_CB - HQ_NOUT], total = hq[HQ_TOTAL - HQ_NOUT];
    // (the code-length blocks are padded to four bytes and every table has one, so at least four bytes follow the
    // payload section: the decode kernel may read the word at the payload's end)
    ok = ok && total <= comp_bytes && hq[HQ_OFF_GROUP - HQ_NOUT] == F.off_group && hq[HQ_OFF_CHUNK - HQ_NOUT] == F.off_chunk &&
         hq[HQ_OFF_PAYLOAD - HQ_NOUT] == F.off_payload && H.words_total <= 0xFFFFFFFFull &&
         H.n_esc_total <= (uint64_t)g.n * g.TD;
    ok = ok && off_cb == d_a16(F.off_payload + 4ull * H.words_total) && total >= off_cb && total - off_cb >= 4ull;
    const float eb = __uint_as_float(dw[0]);
    H.n_used = dw[1]; H.sym_lo = dw[2]; H.sym_hi = dw[3]; H.n_esc = dw[4];
    H.cb = d_cb;
    H.ref_off = d_ref;
    H.ebx2 = eb * 2.0f;
    ok = ok && eb > 0.f && eb < __builtin_inff() && dw[5] == g.G && H.sym_lo <= H.sym_hi && H.sym_hi < g.K &&
         H.n_used >= 1 && H.n_used <= H.sym_hi - H.sym_lo + 1u && H.n_esc <= g.n;
    ok = ok && H.cb >= off_cb && H.cb <= total && (uint64_t)(H.sym_hi - H.sym_lo + 1u) <= total - H.cb;
    // row matching: references behind the code-length blocks (only a context made for it decodes them, and the
    // kernels want a lane's four elements in one row)
    if (H.ref_off != 0)
        ok = ok && g.lz != 0 && (g.D % 4u) == 0 && (H.ref_off % 4u) == 0 && H.ref_off >= off_cb && H.ref_off <= total &&
             4ull * g.B <= total - H.ref_off;
    H.ok = ok;
    return H;
}

// ------------------------------------------------------------------------------------------------
// chunk-parallel decode.  A work-group belongs to one table: it checks the container's header and the table's
// directory entry, rebuilds the canonical code from the stored lengths into an LDS decode table, and then decodes
// `iters` consecutive blocks of NW groups (NW = wavefronts of the work-group), one wavefront per group, lane l walking chunk l.  Each lane keeps
// a 64-bit window of its own bit stream, looks LMAX bits up in the decode table, and the four symbols of a turn
// leave as one 16-byte store (1 KiB contiguous per wavefront instruction).  Nothing is read from a table that fails
// validation.
//
// A lane's symbols hang on one another (the next look-up needs the length of the code before it), so the time a
// group takes is the length of that chain.  The decode table therefore answers for two codewords at a time
// (dec_entry): the bins of both, and `adv`, the bits they take.  Where the second does not fit into the LMAX bits,
// single = 1 and adv = len1: a second look-up follows, rare for the short codes of frequent symbols.
//
// With few groups the decoder is bound by the latencies of a turn (four symbols a lane), each look-up a round trip to LDS,
// so the turn is built to have little between them.  The staged words are stored with their bits reversed and the
// table is indexed by reversed strings: the stream then runs from the low end of a word to the high end, and a position
// in it is one number `p`, whose low five bits are a shift by themselves.  A turn reads the 96 bits around its place
// from LDS and shifts 64 out of them, which is all that four codewords can need: no words are carried from turn to
// turn and none is moved on under a condition.  `p` counts from 30, from the word before the chunk's first: the
// window starts two bits before the next codeword, and masked it is a table entry's byte offset as it is.  Measured against
// two words and a prefetched third in registers, moved on after every look-up, with 12-bit bins converted one by one (75
// instructions a turn, now 35): with a wavefront a group, 26 tables of 2048 x 64 36.7 us, so 31.0 (a turn of a wavefront 730
// cycles, 600), seven of 2999 x 37 38, so 28 (both are decoded in parts now, see k_decode_split); 512 MiB, where the stores bound it, 115.5, so 111.4.
//
// The bit stream words reach the lanes through LDS: the words of a group lie one after the other, so a wavefront copies
// them as they lie (256 bytes an instruction) and every lane reads its own from where its chunk starts.  A group of more
// words than the staging area (3.75 bits a symbol with two work-groups on a compute unit) goes a window at a time instead:
// the next kWin words of every chunk, a row of the staging area each, copied by a team of lanes a chunk.  (A lane copying
// its own chunk's words touched 64 lines an instruction: 512 MiB at 4.3 bits a symbol 139 us, now 125; at 6.4 bits 166, now
// 137.)  Nothing in the decode loop but a new window waits for memory: the stores just stream out.
//
// Per table the work-groups add up the escapes they have applied; the last one to finish compares the sum with the
// directory entry (counters in the workspace, zero between calls).
// ------------------------------------------------------------------------------------------------
constexpr int kWaitLoads = 0x0F70;                    // s_waitcnt vmcnt(0) and nothing else
constexpr uint32_t kRows = 30;                        // a wavefront's staging area has at least kRows words a lane (two work-groups share a CU's LDS)
constexpr uint32_t kStage = kRows * kW;
constexpr uint32_t kStageSmall = 1888;                // the same for a work-group of two wavefronts (five of those share the LDS) and with row
                                                      // matching, whose bits need LDS as well
constexpr uint32_t kWin = 29;                         // words of a chunk in a window (odd: the lanes' rows start in different banks)
constexpr uint32_t kDecWaves = 8;                     // wavefronts per work-group; 4 or 2 for tables of fewer groups (a
                                                      // destination's piece of a table can be two groups: no idle wavefronts)
constexpr uint32_t kSkipWords = 256 * kW / kV / 32;   // row matching: a bit per row of a group, rows of at least four elements

struct DecScratch {  // lives in the staging area until the decode table is complete; one[] is followed by sorted[K] and len[K]
    uint32_t ok;
    uint32_t cl[kLmaxLimit + 2], first[kLmaxLimit + 2];
    uint32_t place[kLmaxLimit + 2];  // of the first symbol of a length in the order, less the first code of that length
    uint16_t one[1 << kLmaxLimit];  // length and bin (dec_bin) of the codeword that the LMAX-bit string starts with whose first bit is bit 0 of the index
    __device__ uint16_t* sorted() { return reinterpret_cast<uint16_t*>(this + 1); }  // the symbols' bins in (length, symbol) order
    __device__ uint8_t* len(uint32_t K) { return reinterpret_cast<uint8_t*>(sorted() + K); }
};
// bytes behind the decode table: the staging areas (`stage` words) of nw wavefronts, or the scratch where that is larger
__host__ __device__ constexpr uint32_t dec_area_bytes(uint32_t nw, uint32_t stage, uint32_t K) {
    return nw * stage * 4u > (uint32_t)((sizeof(DecScratch) + 3u * K + 15u) & ~15u) ? nw * stage * 4u : (uint32_t)((sizeof(DecScratch) + 3u * K + 15u) & ~15u);
}

typedef __attribute__((address_space(3))) uint32_t lds_word_t;
typedef __attribute__((address_space(3))) uint8_t lds_byte_t;
__device__ __forceinline__ uint32_t lds_word(const lds_byte_t* base, uint32_t off) { return *reinterpret_cast<const lds_word_t*>(base + off); }
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// An entry of the decode table, for two codewords, l1 and l2 bits long, of bins b1 and b2 (bin = symbol - R).
// WIDE == false (radius up to 512): the bins as binary16 numbers 1024 + b, of which only the low eleven bits
// vary: one AND-OR makes a pair of them, a packed addition takes the 1024 off (exact: integers up to 2048) and one
// fused multiply-add each makes the product with 2 * bound, converted on the way.
//   single << 31 | adv << 27 | low bits of 1024 + b2 << 16 | l1 << 11 | low bits of 1024 + b1
// WIDE (radius 1024 and 2048): the bins as signed 12-bit numbers; l1 has three bits, so a first code of more than 8 stays alone.
//   single << 31 | adv << 27 | (l1 - 1) << 24 | b2 << 12 | b1
constexpr uint32_t kHalfLow = 0x07FF07FFu, kHalfHigh = 0x60006000u;
template <bool WIDE>
__device__ __forceinline__ uint32_t dec_bin(uint32_t sym, uint32_t R) {  // the bits of a bin, as an entry has them
    const uint32_t t = sym + 1024u - R;
    if constexpr (WIDE) return (sym - R) & 0xFFFu;
    else return t < 1024u ? 2u * t - 1024u : t;  // binary16 of t in [512, 1536): 0x6000 + 2 (t - 512), from 1024 on 0x6400 + (t - 1024)
}
template <bool WIDE>
constexpr uint32_t kBinBits = WIDE ? 12u : 11u;  // l << kBinBits | bits of the bin: what one[] holds
template <bool WIDE>  // of the codewords e1 and e2 (as in one[]); e2 counts if both fit into the LMAX bits
__device__ __forceinline__ uint32_t dec_entry(uint32_t e1, uint32_t e2, uint32_t LMAX) {
    const uint32_t l1 = e1 >> kBinBits<WIDE>, l = l1 + (e2 >> kBinBits<WIDE>);
    if constexpr (WIDE) {
        const uint32_t b1 = e1 & 0xFFFu;
        return l <= LMAX && l1 <= 8u ? (l << 27) | ((l1 - 1u) << 24) | (e2 << 12 & 0xFFF000u) | b1 : 0x80000000u | (l1 << 27) | b1;
    } else {
        return l <= LMAX ? (l << 27) | (e2 << 16 & 0x07FF0000u) | e1 : 0x80000000u | (l1 << 27) | e1;
    }
}
template <bool WIDE>
__device__ __forceinline__ uint32_t dec_len1(uint32_t e) {
    if constexpr (WIDE) return (int)e < 0 ? (e >> 27) & 15u : ((e >> 24) & 7u) + 1u;
    else return (e >> 11) & 15u;
}
template <bool WIDE>  // e with the first symbol of f as its second
__device__ __forceinline__ uint32_t dec_join(uint32_t e, uint32_t f) {
    if constexpr (WIDE) return (e & 0xFFFu) | (f << 12 & 0xFFF000u);
    else return (e & 0xFFFFu) | (f << 16 & 0x07FF0000u);
}
template <bool WIDE>  // the two reconstructions: the product of a whole number and 2 * bound, rounded once
__device__ __forceinline__ void dec_values(uint32_t e, uint32_t half_high, float ebx2, float* v) {
    if constexpr (WIDE) {
        v[0] = (float)((int)(e << 20) >> 20) * ebx2;
        v[1] = (float)((int)(e << 8) >> 20) * ebx2;
    } else {
        union { uint32_t u; half2_t h; } b;
        b.u = (e & kHalfLow) | half_high;
        b.h -= half2_t{(_Float16)1024.0f, (_Float16)1024.0f};
        v[0] = __builtin_fmaf((float)b.h.x, ebx2, 0.0f);
        v[1] = __builtin_fmaf((float)b.h.y, ebx2, 0.0f);
    }
}

// The code lengths of a table from the container, to be asked for before the groups' words.  Symbols that span at most 64: the
// length of symbol sym_lo + lane, in every wavefront.  A wider span: all lengths to LDS, counted.
template <uint32_t NT>
__device__ __forceinline__ uint32_t dec_lengths(const Geom& g, const DecHead& H, const uint8_t* comp, DecScratch& sc, uint32_t tid) {
    const uint32_t nl = H.sym_hi - H.sym_lo + 1u, lane = tid & 63u;
    if (!H.ok) return 0u;  // uniform, and so is nl
    if (nl <= 64u) return lane < nl ? comp[H.cb + lane] : 0u;
    if (tid == 0) sc.ok = H.n_used == 1u ? 0u : 1u;  // (one symbol spans one)
    if (tid < kLmaxLimit + 2) sc.cl[tid] = 0;
    __syncthreads();
    uint8_t* const sc_len = sc.len(g.K);
    for (uint32_t i = tid; i < nl; i += NT) {
        const uint32_t l = comp[H.cb + i];
        sc_len[i] = (uint8_t)l;
        if (l > g.LMAX) sc.ok = 0;
        else if (l) atomicAdd(&sc.cl[l], 1u);
    }
    return 0u;
}

// The decode table of a table's canonical code, by a work-group of NT threads.  `my_len`: what dec_lengths returned.  Where the
// symbols span at most 64, every wavefront works out counts, first codes and the symbols' order by itself, in scalar
// registers, and the work-group only meets for the look-ups (a count by LDS atomics, one wavefront's ordering and the limits
// read back from LDS, the way of a wider span: 7 barriers instead of 3, and 2500 cycles more of a work-group's 18 thousand before the first turn).
// Returns whether the code is complete and as large as the directory says (the same for every thread; ends with a barrier).
template <bool WIDE, uint32_t NT>
__device__ __forceinline__ bool dec_table(const Geom& g, const DecHead& H, uint32_t my_len, uint32_t* lut,
                                          DecScratch& sc, uint32_t tid) {
    const uint32_t lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lut_n = 1u << g.LMAX, nl = H.sym_hi - H.sym_lo + 1u;
    if (!H.ok) return false;  // uniform
    uint32_t limit[kLmaxLimit + 1];  // [l]: the first LMAX-bit string that no codeword of at most l bits starts (in scalar registers)
    bool ok;
    if (nl <= 64u) {  // uniform
        uint32_t kraft = 0, code = 0, index = 0, at = 0, place = 0;
#pragma unroll
        for (uint32_t l = 1; l <= (uint32_t)kLmaxLimit; ++l) {
            const uint64_t m = __ballot(my_len == l);
            const uint32_t c = (uint32_t)__popcll(m);
            code <<= 1;
            at = my_len == l ? index + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) : at;
            place = lane == l ? index - code : place;
            code += c;
            index += c;
            kraft += l <= g.LMAX ? c << (g.LMAX - l) : 0u;
            limit[l] = l <= g.LMAX ? code << (g.LMAX - l) : 0xFFFFFFFFu;
        }
        if (H.n_used == 1u) ok = nl == 1u && __ballot(my_len != 0u) == 0ull;
        else ok = kraft == lut_n && index == H.n_used && __ballot(my_len > g.LMAX) == 0ull;
        if (ok && wave == 0) {
            if (my_len != 0u) sc.sorted()[at] = (uint16_t)dec_bin<WIDE>(H.sym_lo + lane, g.R);
            if (lane <= (uint32_t)kLmaxLimit) sc.place[lane] = place;
        }
        __syncthreads();
    } else {
        uint8_t* const sc_len = sc.len(g.K);
        __syncthreads();
        if (wave == 0 && sc.ok != 0u) {
            // first wavefront: every lane derives the same per-length tables, then the symbols are put in
            // (length, symbol) order, 64 at a time: a symbol's place is the number of symbols of its length before it
            uint64_t kraft = 0;
            uint32_t cnt = 0, code = 0, index = 0;
            uint32_t fill[kLmaxLimit + 1];
#pragma unroll
            for (uint32_t l = 1; l <= (uint32_t)kLmaxLimit; ++l) {
                const uint32_t c = l <= g.LMAX ? sc.cl[l] : 0u;
                kraft += l <= g.LMAX ? (uint64_t)c << (g.LMAX - l) : 0ull;
                cnt += c;
                code <<= 1;
                if (lane == 0) { sc.first[l] = code; sc.place[l] = index - code; }
                fill[l] = index;
                code += c;
                index += c;
            }
            if (kraft != (1ull << g.LMAX) || cnt != H.n_used) {
                if (lane == 0) sc.ok = 0;
            } else {
                const uint64_t below = (1ull << lane) - 1ull;
                for (uint32_t base = 0; base < nl; base += 64) {
                    const uint32_t i = base + lane;
                    const uint32_t L = i < nl ? sc_len[i] : 0u;
                    if (__ballot(L != 0u) == 0ull) continue;  // (a stretch of unused symbols: the escape symbol's code can lie far below the others)
#pragma unroll
                    for (uint32_t l = 1; l <= (uint32_t)kLmaxLimit; ++l) {
                        const uint64_t m = __ballot(L == l);
                        if (L == l) sc.sorted()[fill[l] + (uint32_t)__popcll(m & below)] = (uint16_t)dec_bin<WIDE>(H.sym_lo + i, g.R);
                        fill[l] += (uint32_t)__popcll(m);
                    }
                }
            }
        }
        __syncthreads();
        ok = sc.ok != 0u;
#pragma unroll
        for (uint32_t l = 1; l <= (uint32_t)kLmaxLimit; ++l) {
            const uint32_t past = (uint32_t)__builtin_amdgcn_readfirstlane((int)(sc.first[l] + sc.cl[l]));
            limit[l] = l <= g.LMAX ? past << (g.LMAX - l) : 0xFFFFFFFFu;
        }
    }
    if (!ok) return false;  // uniform
    if (H.n_used == 1u) {  // length 0: every look-up gives one symbol and moves on by nothing
        const uint32_t e = 0x80000000u | dec_bin<WIDE>(H.sym_lo, g.R);
        for (uint32_t i = tid; i < lut_n; i += NT) lut[i] = e;
        __syncthreads();
        return true;
    }
    // the codeword that the LMAX-bit string i (its first bit the highest) starts with
    auto first_code = [&](uint32_t i) {
        uint32_t l = 1;
#pragma unroll
        for (uint32_t k = 1; k < (uint32_t)kLmaxLimit; ++k) l += i >= limit[k] ? 1u : 0u;
        return (l << kBinBits<WIDE>) | sc.sorted()[(i >> (g.LMAX - l)) + sc.place[l]];
    };
    // A thread fills eight strings that agree in all but their last three bits (an eighth of the table apart each, in the
    // order of reversed strings): all of them start with one codeword when that ends before those bits, which for the
    // short codes that cover most of the table is the rule, and for whole wavefronts at a time.
    const uint32_t eighth = lut_n >> 3;  // (lut_n >= 16: a multiple of 8)
    for (uint32_t k = tid; k < eighth; k += NT) {
        const uint32_t i0 = k * 8u, u = __builtin_bitreverse32(i0) >> (32u - g.LMAX);
        const uint32_t ea = first_code(i0);
        if (g.LMAX - (ea >> kBinBits<WIDE>) >= 3u) {
#pragma unroll
            for (uint32_t v = 0; v < 8; ++v) sc.one[u + v * eighth] = (uint16_t)ea;
        } else {
            sc.one[u] = (uint16_t)ea;
#pragma clang loop unroll(disable)
            for (uint32_t v = 1; v < 8; ++v)  // (v's bits are the string's last three, in reverse)
                sc.one[u + v * eighth] = (uint16_t)first_code(i0 | ((v & 1u) << 2 | (v & 2u) | v >> 2));
        }
    }
    __syncthreads();
#pragma clang loop unroll(disable)
    for (uint32_t i0 = tid; i0 < lut_n; i0 += NT * 4u) {  // four strings in flight per thread
        uint32_t e1[4], e2[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) e1[k] = sc.one[(i0 + k * NT) & (lut_n - 1u)];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)  // what follows the first codeword (zeros behind the LMAX bits)
            e2[k] = sc.one[((i0 + k * NT) & (lut_n - 1u)) >> (e1[k] >> kBinBits<WIDE>)];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t i = i0 + k * NT;
            if (i < lut_n) lut[i] = dec_entry<WIDE>(e1[k], e2[k], g.LMAX);
        }
    }
    __syncthreads();  // (the scratch is staging memory from here on)
    return true;
}

constexpr uint32_t kDecBit0 = 30;  // `p` at a chunk's first bit
constexpr uint32_t kSplitWaves = 8;  // wavefronts of a work-group that shares a group's chunks
struct DecTail {
    unsigned long long sum[kDecWaves];
    uint32_t bad, pad;
};

// the four elements at `el` of a group; EDGE: the table can end among them (four elements at once want no more than an
// element's alignment).  STREAM: past the caches, as an output larger than they are wants it (stores of whole kilobytes; where
// a wavefront's lanes are at different turns the caches put the lines together: 208 groups 22.5 us, now 17.6).
template <bool F16, bool VEC, bool EDGE = true, bool STREAM = false>
__device__ __forceinline__ void dec_store(uint8_t* gout, uint32_t el, uint32_t in_group, const float (&v4)[4]) {
    uint8_t* const o = gout + el * (F16 ? 2u : 4u);
    if (!EDGE || VEC || el + 3u < in_group) {
        if constexpr (F16) {
            typedef std::conditional_t<VEC, u32x2, u32x2_any> u2v;
            u2v o2;
            o2.x = (uint32_t)__half_as_ushort(half_rne(v4[0])) | ((uint32_t)__half_as_ushort(half_rne(v4[1])) << 16);
            o2.y = (uint32_t)__half_as_ushort(half_rne(v4[2])) | ((uint32_t)__half_as_ushort(half_rne(v4[3])) << 16);
            if constexpr (STREAM) __builtin_nontemporal_store(o2, reinterpret_cast<u2v*>(o));
            else *reinterpret_cast<u2v*>(o) = o2;
        } else {
            typedef std::conditional_t<VEC, u32x4, u32x4_any> u4v;
            u4v o4 = {__float_as_uint(v4[0]), __float_as_uint(v4[1]), __float_as_uint(v4[2]), __float_as_uint(v4[3])};
            if constexpr (STREAM) __builtin_nontemporal_store(o4, reinterpret_cast<u4v*>(o));
            else *reinterpret_cast<u4v*>(o) = o4;
        }
    } else {
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v)
            if (el + v < in_group) {
                if constexpr (F16) reinterpret_cast<__half*>(o)[v] = half_rne(v4[v]);
                else reinterpret_cast<float*>(o)[v] = v4[v];
            }
    }
}

// What a group's decoding starts from sits in the sections whose place the geometry fixes (the host has made sure they lie
// inside comp_bytes): its loads go out before anything else is known.  gid: the group's number inside the container.
struct GroupHead { uint32_t cw, goff, gnext; };
__device__ __forceinline__ GroupHead dec_group_head(const Geom& g, const FixedLayout& F, const uint8_t* comp, uint32_t gid, uint32_t lane) {
    const uint32_t* const goffs = reinterpret_cast<const uint32_t*>(comp + F.off_group);
    GroupHead h;
    h.cw = comp[F.off_chunk + (uint64_t)gid * kW + lane];
    h.goff = goffs[gid];
    h.gnext = gid + 1 < g.TD * g.G ? goffs[gid + 1] : 0xFFFFFFFFu;  // (the last group ends where the payload does)
    return h;
}
// A group's words (the chunks', then two per escape) checked against the container.  off: the lane's chunk starts there.
struct GroupPlace { bool ok; uint32_t n_esc, total, off; const uint32_t* words; };
__device__ __forceinline__ GroupPlace dec_group_place(const FixedLayout& F, const DecHead& H, const uint8_t* comp, const GroupHead& h) {
    GroupPlace P;
    const uint32_t incl = wave_incl_scan(h.cw);
    P.total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    const uint64_t gend = h.gnext == 0xFFFFFFFFu ? H.words_total : (uint64_t)h.gnext;
    P.ok = !(gend > H.words_total || (uint64_t)h.goff + P.total > gend || ((gend - h.goff - P.total) & 1ull));
    P.n_esc = P.ok ? (uint32_t)((gend - h.goff - P.total) >> 1) : 0u;
    P.words = reinterpret_cast<const uint32_t*>(comp + F.off_payload) + h.goff;
    P.off = incl - h.cw;
    return P;
}

// The container as a whole: its escapes are those of its tables (a container's first work-group, of NW wavefronts).
template <uint32_t NW>
__device__ __forceinline__ void dec_check_escapes(const Geom& g, const DecHead& H, const uint8_t* comp, DecTail& tail, uint32_t tid) {
    uint32_t part = 0;
    bool big = false;
    for (uint32_t k = tid; k < g.TD; k += 64u * NW) {
        const uint32_t e = reinterpret_cast<const uint32_t*>(comp + kHeaderBytes + (uint64_t)kDirBytes * k)[4];
        big = big || e > g.n;
        part += e > g.n ? 0u : e;
    }
    // (32-bit partial sums per thread cannot wrap: a thread adds at most TD / 512 counts of less than 2^31 each,
    // and TD * n < 2^32 positions in all; across threads they are added as 64-bit values)
    unsigned long long sum = part;
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if ((tid & 63u) == 0) tail.sum[tid >> 6] = sum;
    __syncthreads();
    if (tid == 0) {
        unsigned long long all = 0;
        for (uint32_t k = 0; k < NW; ++k) all += tail.sum[k];
        if (all != H.n_esc_total) tail.bad = 1u;
    }
    if (big) tail.bad = 1u;
}

// The end of a work-group, one of wpt of its table.  my_esc: the escapes its wavefront has applied.  dtab (LZ: row matching): gets
// the table's references where every work-group of the table has found its part in order, for the kernel that copies rows.
constexpr uint32_t kTableBad = 0x80000000u;  // in the count of arrivals (of less than 2^31 work-groups)
template <bool LZ>
__device__ __forceinline__ void dec_finish(const DecHead& H, bool valid, uint32_t my_esc, uint32_t wpt, Ctrl* ctrl, uint32_t* esc_seen,
                                           uint32_t* arrived, DecTable* dtab, DecTail& tail, uint32_t tid) {
    if (my_esc != 0u && (tid & 63u) == 0u) {
        __hip_atomic_fetch_add(esc_seen, my_esc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // counted before the work-group says it is done
    }
    __syncthreads();
    if (tid == 0) {
        bool corrupt = !valid || tail.bad != 0u;
        if (LZ && corrupt) {
            __hip_atomic_fetch_or(arrived, kTableBad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the same)
        }
        // the last work-group of the table: all escapes of the table have been seen
        const uint32_t before = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((LZ ? before & ~kTableBad : before) + 1u == wpt) {
            const uint32_t seen = __hip_atomic_exchange(esc_seen, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (valid && seen != H.n_esc) corrupt = true;
            if constexpr (LZ) dtab->ref_off = corrupt || (before & kTableBad) ? 0ull : H.ref_off;
        }
        if (corrupt) set_status(ctrl, DLC_ECORRUPT);
    }
}
// bytes behind the staging areas: a damaged chunk runs at most 256 codes of 12 bits past its words' start, 392 bytes; DecTail is at the end
constexpr uint32_t kDecPad = 512;
static_assert(kDecPad - sizeof(DecTail) >= 392u, "reads past the last chunk");

template <bool F16, bool VEC, bool WIDE, uint32_t NW, bool LZ>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4))) void k_decode(Geom g, FixedLayout F, const uint8_t* comp, uint64_t comp_bytes,
                                                        Ctrl* ctrl, void* outp, uint32_t wpt, uint32_t iters, uint32_t stage_words,
                                                        uint32_t* esc_seen, uint32_t* arrived, DecTable* dtab) {
    constexpr uint32_t kDecThreads = 64u * NW;
    // [1 << LMAX] decode table, NW staging arrays (the scratch before), row matching's bits, padding with DecTail.  All of the kernel's
    // LDS is in this one piece, which therefore starts at LDS address 0: a masked window is a table entry's address as it is
    extern __shared__ __align__(16) uint32_t s_lut[];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t t = blockIdx.x / wpt, b = blockIdx.x % wpt;
    const uint32_t dst = t / g.TD, tl = t - dst * g.TD;  // the container this table is in, and its place there
    comp += (uint64_t)dst * comp_bytes;
    const uint32_t lut_n = 1u << g.LMAX;
    DecScratch& sc = *reinterpret_cast<DecScratch*>(s_lut + lut_n);
    DecTail& tail = *reinterpret_cast<DecTail*>(reinterpret_cast<unsigned char*>(s_lut + lut_n) + dec_area_bytes(NW, stage_words, g.K) +
                                                (LZ ? NW * kSkipWords * 4u : 0u) + kDecPad - sizeof(DecTail));
    auto group_head = [&](uint32_t grp) { return dec_group_head(g, F, comp, tl * g.G + grp, lane); };
    const uint32_t grp_first = b * iters * NW + wave;
    GroupHead gh;
    gh.cw = 0; gh.goff = 0; gh.gnext = 0;
    if (grp_first < g.G) gh = group_head(grp_first);
    const DecHead H = dec_validate(g, F, comp, comp_bytes, tl);
    if (tid == 0) tail.bad = 0u;
    const uint32_t my_len = dec_lengths<kDecThreads>(g, H, comp, sc, tid);
    auto group_place = [&](const GroupHead& h) { return dec_group_place(F, H, comp, h); };
    uint32_t* const stage = s_lut + lut_n + wave * stage_words;
    // The first kStage words of the group as they lie, into registers.  Branch-free, all loads in flight together: an
    // index past the group's end reads its last word instead (an empty group the word at its position, which still lies
    // inside the container: code-length blocks follow the payload).
    auto word_at = [&](const GroupPlace& P, uint32_t i) {  // (a 32-bit byte offset from a uniform base: one register an address)
        return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(P.words) + i * 4u);
    };
    auto fetch_group = [&](const GroupPlace& P, uint32_t (&w)[kRows]) {
        const uint32_t last = P.total ? P.total - 1u : 0u;
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k) w[k] = word_at(P, min(k * kW + lane, last));
    };
    auto put_group = [&](const GroupPlace& P, const uint32_t (&w)[kRows]) {
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k)
            if ((NW != 2u && !LZ) || (k + 1u) * kW <= kStageSmall || k * kW + lane < stage_words) stage[k * kW + lane] = __builtin_bitreverse32(w[k]);
        for (uint32_t k = kStage + lane; k < P.total; k += kW) stage[k] = __builtin_bitreverse32(P.words[k]);
    };
    // A window: the words of every chunk from its lane's `from` on (counted inside the chunk), min(TL, kWin) a chunk, by
    // teams of TL lanes, a chunk a team; the loads [I0, I0 + w's size) of the TL that make the window.  What follows a chunk's
    // end comes from the next chunk; nothing past the group's end is read.
    auto fetch_window = [&](auto tl, auto i0, const GroupPlace& P, uint32_t from, auto& w) {
        constexpr uint32_t TL = decltype(tl)::value, I0 = decltype(i0)::value;
        uint32_t ln = lane;
        asm volatile("" : "+v"(ln));  // (worked out where it is needed: hoisted out of the loops, the lane numbers below took 46 registers)
        const uint32_t at = P.off + from, team = ln / TL, k = ln % TL, last = P.total - 1u;
#pragma unroll
        for (uint32_t i = 0; i < sizeof(w) / 4u; ++i)
            w[i] = word_at(P, min((uint32_t)__builtin_amdgcn_ds_bpermute((int)(((I0 + i) * (kW / TL) + team) * 4u), (int)at) + k, last));
    };
    auto put_window = [&](auto tl, auto i0, const auto& w) {
        constexpr uint32_t TL = decltype(tl)::value, I0 = decltype(i0)::value;
        const uint32_t team = lane / TL, k = lane % TL;
        if (k < kWin) {
#pragma unroll
            for (uint32_t i = 0; i < sizeof(w) / 4u; ++i) stage[((I0 + i) * (kW / TL) + team) * kWin + k] = __builtin_bitreverse32(w[i]);
        }
    };
    // the words come from other lanes of the wavefront.  The wait: a window's lanes that store nothing leave their loads unread,
    // and without it, which costs nothing here, the compiler waits for those inside the loop of the turns, and so for every
    // turn's store (a single group: 27.6 us -> 30)
    auto staged = [&]() {
        __builtin_amdgcn_s_waitcnt(kWaitLoads);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    using std::integral_constant;
    constexpr integral_constant<uint32_t, 0> k0{};
    constexpr integral_constant<uint32_t, 16> k16{};
    constexpr integral_constant<uint32_t, 32> k32{};
    constexpr integral_constant<uint32_t, kRows> kr{};
    // The first group's words are on their way while the decode table is made.  (The second group's too, in registers of their
    // own: slower, all work-groups then ask for everything at once.)
    uint32_t w_first[kRows] = {};
    auto fetch = [&](const GroupPlace& P) {
        if (P.total <= stage_words) fetch_group(P, w_first);
        else fetch_window(k32, k0, P, 0u, w_first);
    };
    GroupPlace gp;
    gp.ok = false; gp.n_esc = 0; gp.total = 0; gp.off = 0; gp.words = nullptr;
    if (H.ok && grp_first < g.G) {
        gp = group_place(gh);
        if (gp.ok) fetch(gp);
    }
    if (H.ok && tl == 0 && b == 0) dec_check_escapes<NW>(g, H, comp, tail, tid);
    uint32_t my_esc = 0;   // escapes this wavefront has applied (uniform)
    bool bad = false;      // something in this wavefront's groups does not add up
    // row matching: which rows of a group refer to another row, as a bit per row in LDS (at most 64*S/4 rows), and whether
    // every reference points back, at a row that is coded
    const uint32_t* const ref = LZ && H.ok && H.ref_off ? reinterpret_cast<const uint32_t*>(comp + H.ref_off) : nullptr;
    uint32_t* const skipbits = reinterpret_cast<uint32_t*>(s_lut + lut_n) + dec_area_bytes(NW, stage_words, g.K) / 4u + wave * kSkipWords;
    auto mark_rows = [&](uint32_t grp) {
        const uint32_t gstart = grp * (kW * g.S), row_lo = gstart / g.D, last_el = gstart + min(g.n - gstart, kW * g.S) - 1u;
        const uint32_t n_rows = last_el / g.D - row_lo + 1u;  // <= 64*S/4 because dim % 4 == 0 here
        for (uint32_t r0 = 0; r0 < n_rows; r0 += 128u) {  // uniform trip count; two rows of a lane in flight
            uint32_t o[2], oo[2];
#pragma unroll
            for (uint32_t k = 0; k < 2u; ++k) o[k] = ref[row_lo + min(r0 + k * 64u + lane, n_rows - 1u)];
#pragma unroll
            for (uint32_t k = 0; k < 2u; ++k) {
                const uint32_t row = row_lo + min(r0 + k * 64u + lane, n_rows - 1u);
                oo[k] = ref[min(o[k], row)];
            }
#pragma unroll
            for (uint32_t k = 0; k < 2u; ++k) {
                const uint32_t row = row_lo + min(r0 + k * 64u + lane, n_rows - 1u);
                bad |= o[k] > row || oo[k] != o[k];
                const uint64_t m = __ballot(o[k] != row);
                if (lane == 0 && r0 + k * 64u < n_rows) { skipbits[r0 / 32u + 2u * k] = (uint32_t)m; skipbits[r0 / 32u + 2u * k + 1u] = (uint32_t)(m >> 32); }
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    // Past the caches where nearly all of the output comes from here; where many rows are copies (of the last 64, a quarter or more)
    // the rows they are copied from stay in the caches for that.
    bool stream = true;
    if (LZ && ref != nullptr && grp_first < g.G) {
        const uint32_t row = g.B - 1u - min(lane, g.B - 1u), o = ref[row];
        mark_rows(grp_first);
        stream = __popcll(__ballot(o != row)) < 16;
    }
    const bool valid = dec_table<WIDE, kDecThreads>(g, H, my_len, s_lut, sc, tid);
    if (valid) {
        const float ebx2 = H.ebx2;
        const uint32_t lut_mask = (lut_n - 1u) << 2;
        uint32_t half_high = kHalfHigh;
        asm("" : "+v"(half_high));  // (a register: an AND-OR takes one other constant at most)
        uint8_t* tab = static_cast<uint8_t*>(outp) + (size_t)t * g.n * g.es;
        for (uint32_t it = 0; it < iters; ++it) {
            const uint32_t grp = grp_first + it * NW;
            if (grp >= g.G) break;  // whole wavefront
            if (it != 0) {
                gh = group_head(grp);
                gp = group_place(gh);
                if (gp.ok) fetch(gp);
                if (LZ && ref != nullptr) mark_rows(grp);
            }
            if (!gp.ok) {
                bad = true;
                continue;
            }
            const uint32_t cw = gh.cw, n_esc = gp.n_esc, total = gp.total;
            const bool linear = total <= stage_words;  // uniform
            const uint32_t st0 = (uint32_t)(uintptr_t)stage;
            if (linear) {
                put_group(gp, w_first);
            } else {
                put_window(k32, k0, w_first);
                uint32_t w[32u - kRows];
                fetch_window(k32, kr, gp, 0u, w);
                put_window(k32, kr, w);
            }
            staged();
            // a lane's place in its bit stream: bit p of the words from LDS address wa on, which is the word before its
            // chunk's word `wbase`
            uint32_t wa = st0 + (linear ? gp.off : lane * kWin) * 4u - 4u;
            asm("" : "+v"(wa));  // (one register: the compiler made two, for the words at wa and those at wa + 4)
            uint32_t wbase = 0, p = kDecBit0;
            // windows: a lane needs a new one when a turn could read past the last word, unless its chunk ends in the one it has
            uint32_t renew_at = (!linear && cw > kWin) ? (kWin - 1u) * 32u : 0xFFFFFFFFu;
            auto renew = [&]() {  // the words from the first that the next turn reads on, anew
                wbase += (p >> 5) - 1u;  // (-1 for a lane that has not taken a bit: its row then starts with the word before its chunk)
                p = (p & 31u) + 32u;
                const uint32_t left = (uint32_t)max((int32_t)(cw - wbase), 0);
                uint32_t w[16];
                if (__ballot(left > 16u) != 0ull) {
                    fetch_window(k32, k0, gp, wbase, w);
                    put_window(k32, k0, w);
                    fetch_window(k32, k16, gp, wbase, w);
                    put_window(k32, k16, w);
                } else {  // the last words of all chunks
                    fetch_window(k16, k0, gp, wbase, w);
                    put_window(k16, k0, w);
                }
                staged();
                renew_at = left > kWin ? (kWin - 1u) * 32u : 0xFFFFFFFFu;
            };
            const uint32_t gstart = grp * (kW * g.S), in_group = min(g.n - gstart, kW * g.S);  // (the table can end in this group)
            uint8_t* const gout = tab + (size_t)gstart * g.es;
            const uint32_t row_lo = gstart / g.D;
            // local / D as a multiplication (a division of its own is a third of a turn's instructions): with the reciprocal
            // rounded up it is exact while local * D < 2^32, and local < 64 * S + D
            const uint32_t row_magic = (ref != nullptr && g.D > 1u && g.D <= 32768u) ? 0xFFFFFFFFu / g.D + 1u : 0u;
            // turn j of the group; EDGE: the table ends in it, so a lane can have fewer than four elements, or none
            auto turn = [&](auto edge, auto past, uint32_t j) {
                constexpr bool EDGE = decltype(edge)::value;
                const uint32_t el = lane * kV + j * (kW * kV);  // the lane's first element, counted from the group's
                if (__ballot(p >= renew_at) != 0ull) renew();  // (whole wavefront)
                bool coded = !EDGE || el < in_group;
                if (LZ && ref != nullptr && coded) {  // a row that refers to another has no bits in the stream; it is copied afterwards
                    const uint32_t local = gstart + el - row_lo * g.D, r = row_magic ? __umulhi(local, row_magic) : local / g.D;
                    coded = ((skipbits[r >> 5] >> (r & 31u)) & 1u) == 0u;
                }
                if (!coded) return;
                const lds_byte_t* const a = reinterpret_cast<const lds_byte_t*>(wa + ((p >> 5) << 2));
                const uint32_t x0 = lds_word(a, 0u), x1 = lds_word(a, 4u), x2 = lds_word(a, 8u);
                uint32_t lo = __builtin_amdgcn_alignbit(x1, x0, p), hi = __builtin_amdgcn_alignbit(x2, x1, p);
                float v4[4];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t e = *reinterpret_cast<const lds_word_t*>(lo & lut_mask);
                    uint32_t adv = (e >> 27) & 15u;
                    const uint32_t len1 = EDGE ? dec_len1<WIDE>(e) : 0u;
                    lo = __builtin_amdgcn_alignbit(hi, lo, adv);
                    hi >>= adv;
                    if ((int)e < 0) {  // an entry that answers for one codeword only: the next one by a look-up of its own
                        const uint32_t f = *reinterpret_cast<const lds_word_t*>(lo & lut_mask), l2 = dec_len1<WIDE>(f);
                        lo = __builtin_amdgcn_alignbit(hi, lo, l2);
                        hi >>= l2;
                        adv += l2;
                        e = dec_join<WIDE>(e, f);
                    }
                    if constexpr (EDGE && !VEC) {  // a turn can reach past the table's end: such a position has no bits
                        if (el + (uint32_t)(h * 2) + 1u >= in_group) adv = el + (uint32_t)(h * 2) < in_group ? len1 : 0u;
                    }
                    p += adv;
                    dec_values<WIDE>(e, half_high, ebx2, v4 + h * 2);
                }
                dec_store<F16, VEC, EDGE, decltype(past)::value>(gout, el, in_group, v4);
            };
            const uint32_t whole = in_group / (kW * kV);
            if (!LZ || stream) {  // uniform
                for (uint32_t j = 0; j < whole; ++j) turn(std::false_type{}, std::true_type{}, j);
            } else {
                for (uint32_t j = 0; j < whole; ++j) turn(std::false_type{}, std::false_type{}, j);
            }
            if (in_group > whole * (kW * kV)) turn(std::true_type{}, std::bool_constant<!LZ>{}, whole);
            // a chunk's codewords end inside its words
            if (__ballot(32u * wbase + p - kDecBit0 > 32u * cw) != 0ull) bad = true;
            if (n_esc != 0u) {  // uniform over the wavefront: verbatim values over the decoded placeholders
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_s_waitcnt(0);  // the wavefront's own stores above are out before the overwrites below
                const uint32_t* rec = reinterpret_cast<const uint32_t*>(comp + F.off_payload) + gh.goff + total;
                bool off_range = false;
                for (uint32_t r = lane; r < n_esc; r += 64) {
                    const uint32_t at = rec[2u * r] - gstart, raw = rec[2u * r + 1];
                    if (at >= in_group) { off_range = true; continue; }
                    if constexpr (F16) reinterpret_cast<uint16_t*>(gout)[at] = (uint16_t)raw;
                    else reinterpret_cast<uint32_t*>(gout)[at] = raw;
                }
                if (__ballot(off_range) != 0ull) bad = true;
                my_esc += n_esc;
            }
        }
    }
    if (__ballot(bad) != 0ull && lane == 0) tail.bad = 1u;
    dec_finish<LZ>(H, valid, my_esc, wpt, ctrl, esc_seen + t, arrived + t, LZ ? dtab + t : nullptr, tail, tid);
}

// ------------------------------------------------------------------------------------------------
// Few groups: a work-group of NW wavefronts for each, and the chunks of the group cut into parts, a wavefront a part (lane l
// still looks after chunk l).  A group by one wavefront is a chain of 64 turns, 38 of the 57 thousand cycles of 26 tables of
// 2048 x 64, while most of the chip has nothing to do.
// Where a part's first codeword starts is not known: a part starts at a word boundary as if one started there, and a
// Huffman code falls into step by itself after a few codewords (streams of 2.2 to 4.4 bits a symbol, measured over their
// chunks: of 16 parts in 2 to 4 rounds, of 8 in 2 or 3).  Round by round every part takes its start from the end of the part
// before and goes through its bits again if that has moved; when no end moves any more every part starts where the one
// before it ends, the first at the chunk's first bit, so the parts together are the chunk.  One part is right after the first
// round and one more at least after every round, so there are no more rounds than parts, whatever the code.  Then the
// codewords counted before a part say which elements it has; of those it writes the turns that start in it.
// A chunk may have more words than its codewords need (the check is that the last one ends inside them, here as
// in k_decode), and a damaged one any bits: every loop ends at its bits' end, a codeword being a bit at least.
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kSplitTurns = 4;  // turns of a part, at least
struct SplitLds {
    uint32_t scratch, stage, ends, tail, end;  // byte offsets; the decode table comes first
};
__host__ __device__ inline SplitLds split_lds(const Geom& g, uint32_t nw) {
    SplitLds L;
    L.scratch = 4u << g.LMAX;
    L.stage = L.scratch + (((uint32_t)sizeof(DecScratch) + 3u * g.K + 15u) & ~15u) + 16u;  // (a turn reads the word before a chunk's first)
    L.ends = L.stage + kW * ((g.S * (uint32_t)kLmaxLimit + 31u) / 32u) * 4u;               // a group's words, all of them
    L.tail = L.ends + (2u * nw * kW + nw + 2u) * 4u;                                       // two sets of ends, a flag a round
    L.tail = (L.tail + 15u) & ~15u;
    L.end = L.tail + (uint32_t)sizeof(DecTail) + kDecPad;
    return L;
}

template <bool F16, bool VEC, bool WIDE>
__global__ __launch_bounds__(64 * kSplitWaves) void k_decode_split(Geom g, FixedLayout F, const uint8_t* comp, uint64_t comp_bytes, Ctrl* ctrl, void* outp,
                                                          SplitLds L, uint32_t* esc_seen, uint32_t* arrived) {
    constexpr uint32_t NW = kSplitWaves, NT = 64u * NW;
    static_assert(NW <= kDecWaves, "DecTail's sums");
    extern __shared__ __align__(16) uint32_t s_lut[];  // (all of the kernel's LDS: the table starts at LDS address 0)
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t t = blockIdx.x / g.G, grp = blockIdx.x - t * g.G;
    const uint32_t dst = t / g.TD, tl = t - dst * g.TD;
    comp += (uint64_t)dst * comp_bytes;
    unsigned char* const lds = reinterpret_cast<unsigned char*>(s_lut);
    DecScratch& sc = *reinterpret_cast<DecScratch*>(lds + L.scratch);
    uint32_t* const stage = reinterpret_cast<uint32_t*>(lds + L.stage);
    uint32_t* const ends = reinterpret_cast<uint32_t*>(lds + L.ends);
    uint32_t* const moved = ends + 2u * NW * kW;
    DecTail& tail = *reinterpret_cast<DecTail*>(lds + L.tail);
    const GroupHead gh = dec_group_head(g, F, comp, tl * g.G + grp, lane);
    const DecHead H = dec_validate(g, F, comp, comp_bytes, tl);
    if (tid == 0) tail.bad = 0u;
    if (tid < NW + 2u) moved[tid] = 0u;
    const uint32_t my_len = dec_lengths<NT>(g, H, comp, sc, tid);
    GroupPlace gp;
    gp.ok = false; gp.n_esc = 0; gp.total = 0; gp.off = 0; gp.words = nullptr;
    // A chunk may have more words than the longest codes fill; its codewords only reach the first of them, and only
    // those are staged then: cw of them, from `off` on.
    uint32_t cw = min(gh.cw, (g.S * (uint32_t)kLmaxLimit + 31u) / 32u), off = 0;
    if (H.ok) {
        gp = dec_group_place(F, H, comp, gh);
        off = gp.off;
        if (gp.ok && __ballot(cw != gh.cw) == 0ull) {
            for (uint32_t i = tid; i < gp.total; i += 2u * NT) {  // two loads in flight
                const uint32_t i2 = min(i + NT, gp.total - 1u), w0 = gp.words[i], w1 = gp.words[i2];
                stage[i] = __builtin_bitreverse32(w0);
                stage[i2] = __builtin_bitreverse32(w1);
            }
        } else if (gp.ok) {
            off = wave_incl_scan(cw) - cw;
            for (uint32_t c = wave; c < kW; c += NW) {
                const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)cw, (int)c), to = (uint32_t)__builtin_amdgcn_readlane((int)off, (int)c), at = (uint32_t)__builtin_amdgcn_readlane((int)gp.off, (int)c);
                for (uint32_t i = lane; i < n; i += kW) stage[to + i] = __builtin_bitreverse32(gp.words[at + i]);
            }
        }
    }
    if (H.ok && tl == 0 && grp == 0) dec_check_escapes<NW>(g, H, comp, tail, tid);
    const bool valid = dec_table<WIDE, NT>(g, H, my_len, s_lut, sc, tid);  // (its barriers publish the staged words, too)
    uint32_t my_esc = 0;
    bool bad = valid && !gp.ok;
    if (valid && gp.ok) {  // uniform over the work-group
        const uint32_t lut_mask = ((1u << g.LMAX) - 1u) << 2;
        uint32_t half_high = kHalfHigh;
        asm("" : "+v"(half_high));
        const uint32_t gstart = grp * (kW * g.S), in_group = min(g.n - gstart, kW * g.S);
        uint8_t* const gout = static_cast<uint8_t*>(outp) + ((size_t)t * g.n + gstart) * g.es;
        uint32_t wa = (uint32_t)(uintptr_t)(lds_byte_t*)stage + off * 4u - 4u;
        asm("" : "+v"(wa));
        struct Window { uint32_t lo, hi; };
        auto window = [&](uint32_t p) {  // the 64 bits from two before the place p (counted as in k_decode) on
            const lds_byte_t* const a = reinterpret_cast<const lds_byte_t*>(wa + ((p >> 5) << 2));
            const uint32_t x0 = lds_word(a, 0u), x1 = lds_word(a, 4u), x2 = lds_word(a, 8u);
            Window w;
            w.lo = __builtin_amdgcn_alignbit(x1, x0, p);
            w.hi = __builtin_amdgcn_alignbit(x2, x1, p);
            return w;
        };
        auto shift = [](Window& w, uint32_t by) {
            w.lo = __builtin_amdgcn_alignbit(w.hi, w.lo, by);
            w.hi >>= by;
        };
        const uint32_t turns = (in_group + kW * kV - 1u) / (kW * kV);
        const uint32_t parts = min(NW, max(1u, turns / kSplitTurns)), part = wave;
        // elements of the lane's chunk
        const uint32_t whole = in_group / (kW * kV), over = in_group - whole * (kW * kV);
        const uint32_t n_el = whole * kV + min(kV, over - min(over, lane * kV));
        const uint32_t n_turns = (n_el + kV - 1u) / kV;
        uint32_t start = 0, before = 0, count = 0;  // the part's first bit, codewords before it and in it
        if (H.n_used == 1u) {  // no bits: the turns as they come
            before = min(n_el, kV * (n_turns * part / parts));
            count = part + 1u < parts ? kV * (n_turns * (part + 1u) / parts) - before : n_el - before;
        } else {
            const uint32_t b0 = cw * part / parts * 32u, b1 = cw * (part + 1u) / parts * 32u;
            uint32_t stop = b0;
            // the part's codewords from bit `start` on: those that start before b1 (the last part's are not asked for).  Two at a
            // time while a pair cannot reach past b1, then one by one.
            auto run = [&](bool go) {
                uint32_t x = go ? start : b1, c = 0;
                while (x + g.LMAX <= b1) {
                    Window w = window(x + kDecBit0);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t e = *reinterpret_cast<const lds_word_t*>(w.lo & lut_mask), adv = (e >> 27) & 15u;
                        x += adv;
                        c += 2u + (uint32_t)((int)e >> 31);
                        shift(w, adv);
                        if (k < 3 && x + g.LMAX > b1) break;
                    }
                }
                if (x < b1) {  // (fewer than LMAX bits: one window has the codewords)
                    Window w = window(x + kDecBit0);
                    do {
                        const uint32_t l1 = dec_len1<WIDE>(*reinterpret_cast<const lds_word_t*>(w.lo & lut_mask));
                        x += l1;
                        c += 1u;
                        shift(w, l1);
                    } while (x < b1);
                }
                return (c << 16) | x;
            };
            start = b0;
            uint32_t got = part + 1u < parts ? run(true) : start;
            stop = got & 0xFFFFu;
            count = got >> 16;
            uint32_t set = 0;
            if (part < parts) ends[part * kW + lane] = got;
            __syncthreads();
            for (uint32_t round = 0; round <= parts; ++round) {  // uniform over the work-group
                const uint32_t from = part != 0u && part < parts ? ends[set * (NW * kW) + (part - 1u) * kW + lane] & 0xFFFFu : 0u;
                const bool again = part < parts && from != start;
                start = from;
                if (__ballot(again) != 0ull && part + 1u < parts) {
                    const uint32_t g2 = run(again);
                    if (again) got = g2;  // (nothing where the codeword before goes on past this part's end)
                    if (__ballot((got & 0xFFFFu) != stop) != 0ull && lane == 0) moved[round] = 1u;
                    stop = got & 0xFFFFu;
                    count = got >> 16;
                }
                set ^= 1u;
                if (part < parts) ends[set * (NW * kW) + part * kW + lane] = got;
                __syncthreads();
                if (moved[round] == 0u) break;
            }
            for (uint32_t k = 0; k + 1u < NW; ++k) before += k < min(part, parts) ? ends[set * (NW * kW) + k * kW + lane] >> 16 : 0u;
            before = min(before, n_el);
            count = part + 1u < parts ? count : n_el;
        }
        // the turns that start in this part
        const uint32_t j1 = part < parts ? min(n_turns, (before + min(count, n_el) + kV - 1u) / kV) : 0u;
        uint32_t j = (before + kV - 1u) / kV, p = start + kDecBit0;
        bool go = j < j1;
        const bool last = go && j1 == n_turns;  // this part has the chunk's last codeword
        {  // codewords of a turn that started in the part before
            Window w = window(p);
            const uint32_t skip = j * kV - before;
#pragma unroll
            for (uint32_t k = 0; k + 1u < kV; ++k) {
                const uint32_t e = *reinterpret_cast<const lds_word_t*>(w.lo & lut_mask), l1 = dec_len1<WIDE>(e);
                p += k < skip ? l1 : 0u;
                shift(w, l1);
            }
        }
        while (__ballot(go) != 0ull) {
            if (go) {
                const uint32_t el = lane * kV + j * (kW * kV);
                Window w = window(p);
                float v4[4];
#pragma unroll
                for (uint32_t h = 0; h < 2u; ++h) {
                    uint32_t e = *reinterpret_cast<const lds_word_t*>(w.lo & lut_mask);
                    uint32_t adv = (e >> 27) & 15u;
                    const uint32_t l1 = VEC ? 0u : dec_len1<WIDE>(e);
                    shift(w, adv);
                    if ((int)e < 0) {
                        const uint32_t f = *reinterpret_cast<const lds_word_t*>(w.lo & lut_mask), l2 = dec_len1<WIDE>(f);
                        shift(w, l2);
                        adv += l2;
                        e = dec_join<WIDE>(e, f);
                    }
                    if constexpr (!VEC) {  // a turn can reach past the table's end: such a position has no bits
                        if (el + h * 2u + 1u >= in_group) adv = el + h * 2u < in_group ? l1 : 0u;
                    }
                    p += adv;
                    dec_values<WIDE>(e, half_high, H.ebx2, v4 + h * 2u);
                }
                dec_store<F16, VEC>(gout, el, in_group, v4);
                ++j;
                go = j < j1;
            }
        }
        // a chunk's codewords end inside its words
        if (__ballot(last && p - kDecBit0 > 32u * gh.cw) != 0ull) bad = true;
        if (gp.n_esc != 0u) {  // uniform over the work-group: verbatim values over the decoded placeholders
            __builtin_amdgcn_s_waitcnt(kWaitLoads);  // (stores count as well: all of the work-group's are out behind the barrier,
            __syncthreads();                         // which waits for none by itself)
            bool off_range = false;
            for (uint32_t r = tid; r < gp.n_esc; r += NT) {
                const uint32_t at = gp.words[gp.total + 2u * r] - gstart, raw = gp.words[gp.total + 2u * r + 1u];
                if (at >= in_group) { off_range = true; continue; }
                if constexpr (F16) reinterpret_cast<uint16_t*>(gout)[at] = (uint16_t)raw;
                else reinterpret_cast<uint32_t*>(gout)[at] = raw;
            }
            if (__ballot(off_range) != 0ull) bad = true;
            if (wave == 0) my_esc = gp.n_esc;
        }
    }
    if (bad && lane == 0) tail.bad = 1u;
    dec_finish<false>(H, valid, my_esc, g.G, ctrl, esc_seen + t, arrived + t, nullptr, tail, tid);
}

// rows that refer to an earlier row of their table: copies of that row's reconstruction (after the decode kernel).
// A thread per 16-byte (fp32) / 8-byte (fp16) piece of a row, pieces of a row on neighbouring threads.  What bounds it: the writes
// (64 tables of 8192 x 128, 62 % of the rows, 166 MB, in 29 us: 5.7 TB/s).  They go past the caches, so that the rows they are copied
// from, which the decode kernel left there, stay: 46 us with both the other way round, when every row came from memory.
template <typename U>
__global__ __launch_bounds__(256) void k_row_copy(Geom g, const uint8_t* comp, uint64_t comp_bytes, const DecTable* dtab,
                                                  void* outp, TableOrder order) {
    uint32_t t, block;
    order.place(&t, &block);
    if (t >= g.T) return;           // uniform
    const uint32_t dst = t / g.TD;  // the container this table is in
    comp += (uint64_t)dst * comp_bytes;
    const uint64_t ref_off = dtab[t].ref_off;
    if (ref_off == 0) return;  // uniform
    const uint32_t* ref = reinterpret_cast<const uint32_t*>(comp + ref_off);
    U* tab = reinterpret_cast<U*>(static_cast<uint8_t*>(outp) + (size_t)t * g.n * g.es);
    const uint32_t upr = g.D / 4u;  // pieces per row (four elements each; dim % 4 == 0)
    const uint32_t total = g.B * upr;
    // four pieces a thread has in flight: references first, then the rows they point at (named variables, not an
    // array: the compiler moved an array of vectors into LDS)
    const uint32_t stride = order.bx * 256;
    for (uint32_t i0 = block * 256 + threadIdx.x; i0 < total; i0 += stride * 4u) {
        uint32_t row[4], o[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t i = i0 + k * stride;
            row[k] = i < total ? i / upr : 0xFFFFFFFFu;
            o[k] = i < total ? ref[row[k]] : 0xFFFFFFFFu;
        }
        auto src = [&](uint32_t k) -> size_t { return (size_t)o[k] * upr + (i0 + k * stride - row[k] * upr); };
        U v0{}, v1{}, v2{}, v3{};
        if (o[0] != row[0]) v0 = tab[src(0)];
        if (o[1] != row[1]) v1 = tab[src(1)];
        if (o[2] != row[2]) v2 = tab[src(2)];
        if (o[3] != row[3]) v3 = tab[src(3)];
        if (o[0] != row[0]) __builtin_nontemporal_store(v0, &tab[(size_t)i0]);
        if (o[1] != row[1]) __builtin_nontemporal_store(v1, &tab[(size_t)i0 + stride]);
        if (o[2] != row[2]) __builtin_nontemporal_store(v2, &tab[(size_t)i0 + 2u * stride]);
        if (o[3] != row[3]) __builtin_nontemporal_store(v3, &tab[(size_t)i0 + 3u * stride]);
    }
}

hipError_t launch_decompress(const Geom& g, const uint8_t* comp, uint64_t comp_bytes, void* out, const Ws& w, int pl,
                             void* prof, hipStream_t s) {
    const bool f16 = g.dtype == DLC_F16;
    const FixedLayout F = fixed_layout(g);
    {
        // a work-group decodes `iters` blocks of nw groups of one table, a wavefront each, and no more wavefronts than a table
        // has groups (a small grid, of row matching or of groups of few turns, takes eight all the same: they make the decode table sooner)
        const uint32_t nw = (g.G >= 6u || (uint64_t)g.T * g.G <= 512u) ? kDecWaves : (g.G >= 3u ? 4u : 2u);
        const uint32_t bpt = (g.G + nw - 1) / nw;
        auto lds_bytes = [&](uint32_t stage) { return ((size_t)4 << g.LMAX) + dec_area_bytes(nw, stage, g.K) + (g.lz ? (size_t)nw * kSkipWords * 4 : 0) + kDecPad; };
        const uint32_t stage_full = nw == 2u || g.lz ? kStageSmall : kStage;  // (of a chip that is full)
        // More blocks a work-group spread the cost of its decode table; more work-groups fill the chip and even out the compute
        // units.  Where the stores bound the whole (fp32), that is one block each, and the next work-groups fill the gaps (512
        // MiB, 1024 blocks: 111 us, with two blocks each 119; 1536 159, 180).  Where they do not (half precision), the rounds of
        // work-groups count, each as long as its blocks and its decode table, which takes 0.7 of a block: one to four blocks, as
        // that is shortest.  Us a call, one block each and this: half precision, 576 and 1024 blocks 74, 65 and 86, 69, 900 76, 76
        // (by twos 87).  (fp32 with row matching lies between the two: 560, 640, 768 and 1200 blocks, where half of the rows and
        // more are copies 95, 94, 102 and 163, by this rule 90, 88, 97 and 154; where nearly none are 103, 110, 118 and 177 against 108, 116, 124 and 187.)
        uint32_t iters = 1;
        if (f16) {
            const uint32_t per_cu = std::min<uint32_t>(16u / nw, 163840u / (uint32_t)((lds_bytes(stage_full) + 1279u) / 1280u * 1280u));
            const uint64_t room = 256ull * std::max(1u, per_cu);
            uint64_t least = ~0ull;
            for (uint32_t k = 1; k <= 4u; ++k) {
                const uint64_t rounds = ((uint64_t)g.T * ((bpt + k - 1u) / k) + room - 1u) / room, cost = rounds * (10u * k + 7u);
                if (cost < least) { least = cost; iters = k; }
            }
        } else {
            iters = (uint32_t)std::min<uint64_t>(4, std::max<uint64_t>(1, (uint64_t)g.T * bpt / 2048u));
        }
        const uint32_t wpt = (bpt + iters - 1) / iters;  // work-groups per table
        dim3 grid(g.T * wpt), block(64 * nw);
        // a grid that leaves compute units free can have larger staging areas: 6 bits a symbol
        // (LDS comes in pieces of 1280 bytes: with 1888 words a wavefront, work-groups of two take 25 of the 128, and five fit a
        // compute unit; 1184 tables of 256 elements, one round of them, 14.9 us, with 1920 words 19.4)
        const uint32_t stage = (uint64_t)g.T * wpt <= 256u ? 3072u : stage_full;
        const size_t sm = lds_bytes(stage);
        if (prof_on(pl, P_DECODE)) prof_begin(prof, P_DECODE, s);
        // Up to two groups a compute unit: a work-group each (us: one group 24, now 15; 208 groups 30.5, now 18; 512 groups of 2.2 and
        // 4.4 bits a symbol 23.8 and 29.2, now 22.7 and 23.5).  More than the chip holds at once, and a wavefront a
        // group is the shorter way (720 groups: 24 and 29 against 34 and 37).  Sixteen wavefronts, and parts half as long, are no
        // faster: they need more rounds.  Nor is it a gain where a group has 16 turns or fewer, for what is split is a chain too
        // short for the rounds (512 groups of chunks of 64, 2.2 and 6 bits a symbol: 16.1 and 22.2, a wavefront a group 13.1 and
        // 18.9; 256 tables of 4096 elements 14.0, so 13.3; of 24 and 32 turns 17.2 and 16.2, a wavefront a group 17.8 both).
        const uint32_t turns = (std::min(g.n, kW * g.S) + kW * kV - 1u) / (kW * kV);
        const bool split = !g.lz && g.NG <= 512u && turns > 16u;
        const SplitLds L = split_lds(g, kSplitWaves);
#define DLC_DEC3(FF, V, W, N, LZ) hipLaunchKernelGGL((k_decode<FF, V, W, N, LZ>), grid, block, sm, s, g, F, comp, (uint64_t)comp_bytes, w.ctrl, out, wpt, iters, stage, w.dec_esc, w.dec_arrive, w.dtab)
#define DLC_DEC2(FF, V, N, LZ) do { if (g.R > 512u) DLC_DEC3(FF, V, true, N, LZ); else DLC_DEC3(FF, V, false, N, LZ); } while (0)
#define DLC_DEC(FF, V, LZ) do { if (nw == 8u) DLC_DEC2(FF, V, 8u, LZ); else if (nw == 4u) DLC_DEC2(FF, V, 4u, LZ); else DLC_DEC2(FF, V, 2u, LZ); } while (0)
#define DLC_SPLIT2(FF, V, W) hipLaunchKernelGGL((k_decode_split<FF, V, W>), dim3(g.NG), dim3(64u * kSplitWaves), L.end, s, g, F, comp, (uint64_t)comp_bytes, w.ctrl, out, L, w.dec_esc, w.dec_arrive)
#define DLC_SPLIT(FF, V) do { if (g.R > 512u) DLC_SPLIT2(FF, V, true); else DLC_SPLIT2(FF, V, false); } while (0)
        if (split) {
            if (f16) { if (g.vec) DLC_SPLIT(true, true); else DLC_SPLIT(true, false); }
            else { if (g.vec) DLC_SPLIT(false, true); else DLC_SPLIT(false, false); }
        } else if (g.lz) { if (f16) DLC_DEC(true, true, true); else DLC_DEC(false, true, true); }  // (dim % 4 == 0 there)
        else if (f16) { if (g.vec) DLC_DEC(true, true, false); else DLC_DEC(true, false, false); }
        else { if (g.vec) DLC_DEC(false, true, false); else DLC_DEC(false, false, false); }
#undef DLC_SPLIT
#undef DLC_SPLIT2
#undef DLC_DEC
#undef DLC_DEC2
#undef DLC_DEC3
        if (g.lz) {
            // tables apart and one after the other, us a call: one of 65536 rows 56.0 and 43.3; 9, 26, 64, 65, 100 and 128 of 8192 x
            // 128 40.7 and 39.4, 48.9 and 49.8, 67.6 and 74.4, 90.8 and 95.5, 112.5 and 120.2, 125.1 and 135.2; 300 of 2048 x 128 125.6
            // and 126.0.  Tables whose work-groups an XCD runs all at once are as well there, where most of what they read was
            // written: one of 300 x 16 18.8 and 19.9, 100 of 2048 x 64 47.2 and 47.6.
            const uint32_t bx = std::min<uint32_t>((g.B * (g.D / 4u) + 255u) / 256u, 256u);
            const TableOrder order(bx, bx < 256u || g.T % 8u == 0u || g.T > 16u);
            if (f16) hipLaunchKernelGGL(k_row_copy<u32x2>, dim3(order.groups(g.T)), dim3(256), 0, s, g, comp, (uint64_t)comp_bytes, w.dtab, out, order);
            else hipLaunchKernelGGL(k_row_copy<u32x4>, dim3(order.groups(g.T)), dim3(256), 0, s, g, comp, (uint64_t)comp_bytes, w.dtab, out, order);
        }
        if (prof_on(pl, P_DECODE)) prof_end(prof, P_DECODE, s);
    }
    return hipGetLastError();
}

template <uint32_t NW>
static hipError_t decode_set_attributes() {
    const int bytes = (4 << kLmaxLimit) + (int)dec_area_bytes(NW, 3072u, 4096u) + (int)(NW * kSkipWords * 4) + (int)kDecPad;
    const void* ks[] = {reinterpret_cast<const void*>(k_decode<false, false, false, NW, false>), reinterpret_cast<const void*>(k_decode<false, false, true, NW, false>),
                        reinterpret_cast<const void*>(k_decode<false, true, false, NW, false>), reinterpret_cast<const void*>(k_decode<false, true, true, NW, false>),
                        reinterpret_cast<const void*>(k_decode<true, false, false, NW, false>), reinterpret_cast<const void*>(k_decode<true, false, true, NW, false>),
                        reinterpret_cast<const void*>(k_decode<true, true, false, NW, false>), reinterpret_cast<const void*>(k_decode<true, true, true, NW, false>),
                        reinterpret_cast<const void*>(k_decode<false, true, false, NW, true>), reinterpret_cast<const void*>(k_decode<false, true, true, NW, true>),
                        reinterpret_cast<const void*>(k_decode<true, true, false, NW, true>), reinterpret_cast<const void*>(k_decode<true, true, true, NW, true>)};
    hipError_t e = hipSuccess;
    for (const void* k : ks)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    return e;
}

static hipError_t split_set_attributes() {
    Geom g = {};
    g.LMAX = kLmaxLimit; g.K = 4096u; g.S = 256u;
    const int bytes = (int)split_lds(g, kSplitWaves).end;
    const void* ks[] = {reinterpret_cast<const void*>(k_decode_split<false, false, false>), reinterpret_cast<const void*>(k_decode_split<false, true, false>),
                        reinterpret_cast<const void*>(k_decode_split<true, false, false>), reinterpret_cast<const void*>(k_decode_split<true, true, false>),
                        reinterpret_cast<const void*>(k_decode_split<false, false, true>), reinterpret_cast<const void*>(k_decode_split<false, true, true>),
                        reinterpret_cast<const void*>(k_decode_split<true, false, true>), reinterpret_cast<const void*>(k_decode_split<true, true, true>)};
    hipError_t e = hipSuccess;
    for (const void* k : ks)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    return e;
}

hipError_t decompress_set_attributes() {
    hipError_t e = decode_set_attributes<8u>();
    if (e == hipSuccess) e = split_set_attributes();
    if (e == hipSuccess) e = decode_set_attributes<4u>();
    if (e == hipSuccess) e = decode_set_attributes<2u>();
    return e;
}

}  // namespace dlc
