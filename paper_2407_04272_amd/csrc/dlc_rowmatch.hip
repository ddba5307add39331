// Row matching for gfx950 (the vector-based LZ step of Section III-D: the fixed pattern is one embedding vector).
// For every row of a table: the first row of the batch with the same content after quantisation (all symbols
// equal and, where a symbol is the escape, the raw bits too).  Rows that have an earlier equal are not coded by
// the kernels that follow; they are stored as references.
//
// Three kernels, after the histogram kernel and on its symbol plane: a 64-bit hash per row; per table, sets of the
// rows by hash, kept in LDS (the table's rows are divided among several work-groups by their hashes, so no two
// work-groups ever meet in a set and no atomic leaves the LDS), the smallest row index of a hash owning it; then
// every other row is compared with the owner of its hash element by element.  A row whose hash meets a different
// row's (three multilinear sums modulo 2^32 with 24-bit multipliers: 2^-48 for a pair of rows at worst, far less
// for most) is looked up the long way, among the earlier rows with that hash, so the references are those of the
// definition (the first row with the content) whatever the hashes do.
#include <algorithm>

#include "dlc_internal.h"
#include "dlc_codec_dev.h"

namespace dlc {

namespace {

__device__ __forceinline__ uint64_t rm_mix64(uint64_t z) {
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

__host__ __device__ __forceinline__ uint32_t rm_mix32(uint32_t z) {
    z ^= z >> 16; z *= 0x85EBCA6Bu;
    z ^= z >> 13; z *= 0xC2B2AE35u;
    z ^= z >> 16;
    return z;
}

// what two elements must agree in to count as equal: the symbol, or for an escape the raw bits (bit 32 set)
template <bool F16>
__device__ __forceinline__ uint64_t rm_identity(const uint8_t* tab, uint32_t i, const QParam& q, float Rf, int R) {
    uint32_t raw;
    float x;
    if constexpr (F16) {
        raw = reinterpret_cast<const uint16_t*>(tab)[i];
        x = __half2float(__ushort_as_half((unsigned short)raw));
    } else {
        raw = reinterpret_cast<const uint32_t*>(tab)[i];
        x = __uint_as_float(raw);
    }
    const uint32_t c = quant_symbol<F16>(x, q, Rf, R);
    return c ? (uint64_t)c : ((1ull << 32) | raw);
}

// is one of the four bytes 254 or 255 (the plane's "escape" and "outside the window": what the element is, its raw
// bits or its symbol, is in the payload)?
__device__ __forceinline__ bool rm_has255(uint32_t w) {
    const uint32_t x = ~(w | 0x01010101u);
    return ((x - 0x01010101u) & ~x & 0x80808080u) != 0u;
}

// adds the piece's two halves to the three sums (multilinear, modulo 2^32); m: the 24-bit multipliers of the
// piece's position in the row, two per sum
__device__ __forceinline__ void rm_add_piece(uint32_t w, const uint4& m03, const uint2& m45, uint32_t a[3]) {
    const uint32_t lo = w & 0xFFFFu, hi = w >> 16;
    a[0] += __umul24(lo, m03.x) + __umul24(hi, m03.y);
    a[1] += __umul24(lo, m03.z) + __umul24(hi, m03.w);
    a[2] += __umul24(lo, m45.x) + __umul24(hi, m45.y);
}

// what an element outside the window adds to the three sums: by what it is and where it is
__device__ __forceinline__ void rm_add_other(uint64_t id, uint32_t e, uint32_t a[3]) {
    const uint32_t z = rm_mix32((uint32_t)id + 0x9E3779B9u * (e + 1u)) ^ ((id >> 32) ? 0x7F4A7C15u : 0u);
    a[0] += z;
    a[1] += rm_mix32(z);
    a[2] += rm_mix32(z ^ 0x5BD1E995u);
}

// the hash from the three sums
__device__ __forceinline__ uint64_t rm_finish(const uint32_t a[3]) {
    return rm_mix64((((uint64_t)a[1] << 32) | a[0]) + (uint64_t)a[2] * 0x9E3779B97F4A7C15ull);
}

constexpr uint32_t kRmSlab = 32;   // pieces of a row that pass 1 holds in LDS at a time
constexpr uint32_t kRmPitch = kRmSlab + 1u;

}  // namespace

// The hash and the verify kernel read the symbol plane the histogram kernel has written (one byte per element: the
// symbol's window index, 254 for an escape, 255 for a symbol outside the window), four bytes (a piece) at a time.
// An element with index 254 or 255 is looked up in the payload: the raw bits of an escape, or the symbol.

// pass 1: hash of every row, a lane per row.  A wavefront takes 64 consecutive rows: it loads their pieces as
// they lie in memory (16 bytes per lane where the row length allows), kRmSlab pieces of each row at a time, into LDS
// with an odd pitch, and every lane then walks its own row there; the multipliers of a position are the same
// for all lanes.
template <bool F16>
__global__ __launch_bounds__(256) void k_rm_hash(const void* payload, Geom g, const QParam* qp, const uint8_t* on,
                                                 uint64_t* rowhash, const uint8_t* sym_plane,
                                                 const uint32_t* __restrict__ mult, uint32_t waves_grid) {
    __shared__ uint32_t stage[4][64 * kRmPitch];
    const uint32_t t = blockIdx.y;
    if (!on[t]) return;  // uniform: the table is coded row by row as it is
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t wave_global = blockIdx.x * 4 + wave;
    const uint32_t W = g.D / 4u;
    const QParam q = qp[t];
    const float Rf = (float)g.R;
    const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
    const uint32_t* plane = reinterpret_cast<const uint32_t*>(sym_plane + (size_t)t * plane_stride(g));
    uint32_t* st = stage[wave];
    for (uint32_t row0 = wave_global * 64u; row0 < g.B; row0 += waves_grid * 64u) {
        const uint32_t nrows = min(64u, g.B - row0);
        uint32_t a[3] = {0u, 0u, 0u};
        for (uint32_t p0 = 0; p0 < W; p0 += kRmSlab) {
            const uint32_t sw = min(kRmSlab, W - p0);  // pieces of every row in this slab
            const uint32_t total = nrows * sw;         // 2048 at most
            if (sw == W && (W & 3u) == 0u) {  // whole rows, one after the other in memory, 16-byte pieces
                const uint4* src = reinterpret_cast<const uint4*>(plane + (size_t)row0 * W);
                const uint32_t n4 = total / 4u;
                const float inv = 1.0f / (float)W;
                for (uint32_t k0 = 0; k0 < n4; k0 += 64u * 8u) {
                    uint4 v[8];
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) {
                        const uint32_t i = k0 + u * 64u + lane;
                        v[u] = i < n4 ? src[i] : make_uint4(0, 0, 0, 0);
                    }
#pragma unroll
                    for (uint32_t u = 0; u < 8; ++u) {
                        const uint32_t i = k0 + u * 64u + lane;
                        if (i < n4) {
                            const uint32_t idx = i * 4u;
                            const uint32_t r = (uint32_t)(((float)idx + 0.5f) * inv);  // idx / W, exact for these sizes
                            uint32_t* d = st + idx + r * (kRmPitch - W);               // row r, piece idx - r * W
                            d[0] = v[u].x; d[1] = v[u].y; d[2] = v[u].z; d[3] = v[u].w;
                        }
                    }
                }
            } else {
                const float inv = 1.0f / (float)sw;
                for (uint32_t i = lane; i < total; i += 64u) {
                    const uint32_t r = (uint32_t)(((float)i + 0.5f) * inv), c = i - r * sw;
                    st[r * kRmPitch + c] = plane[(size_t)(row0 + r) * W + p0 + c];
                }
            }
            // the pieces come from other lanes of this wavefront: its LDS accesses complete in order, the compiler
            // must keep them in order too
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (lane < nrows) {
                const uint32_t* mine = st + lane * kRmPitch;
                for (uint32_t c0 = 0; c0 < sw; c0 += 4u) {  // (position and multipliers: the same for all lanes)
                    uint32_t w[4];
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) w[k] = c0 + k < sw ? mine[c0 + k] : 0u;
                    bool other = false;
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k) {
                        const uint32_t p = min(p0 + c0 + k, W - 1u);  // (a piece past the row's end is 0 and adds nothing)
                        const uint4 m03 = *reinterpret_cast<const uint4*>(mult + 8u * p);
                        const uint2 m45 = *reinterpret_cast<const uint2*>(mult + 8u * p + 4u);
                        rm_add_piece(w[k], m03, m45, a);
                        other = other || rm_has255(w[k]);
                    }
                    if (other) {  // rare
                        for (uint32_t k = 0; k < 4; ++k) {
                            for (uint32_t v = 0; v < 4; ++v) {
                                if (((w[k] >> (8u * v)) & 255u) < kWinEsc) continue;
                                const uint32_t e = (p0 + c0 + k) * 4u + v;
                                rm_add_other(rm_identity<F16>(tab, (row0 + lane) * g.D + e, q, Rf, (int)g.R), e, a);
                            }
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        const uint32_t row = row0 + lane;
        if (row < g.B)
            rowhash[(size_t)t * g.B + row] = rm_finish(a);
    }
}

// The same hash for rows of 256 elements and more that are whole 16-byte pieces (of four words): a row is the work of a team
// of 2^logL lanes, a piece each, as it lies in memory; where a row has 64 pieces or fewer, a lane's position in it never changes
// and the multipliers of its piece stay in registers.  Nothing goes through LDS, and the team adds its sums up (modulo 2^32).
// A lane a row leaves the chip empty where rows are few and long: a wavefront then walks 64 of them alone.  Whole calls, lane
// per row and team, us: 16 tables of 2048 rows of 1024 250 and 153, of 2048 x 2048 (26 tables) 461 and 254 (both with the
// compare kernel's finer split), 16 of 8192 x 256 144 and 125.  Rows of 128 and fewer, of which there are many, gain nothing (64
// tables of 8192 x 128: 21 us either way, of which the plane's way from memory is 12): they keep a lane each.
constexpr uint32_t kRmBlk = 4;  // pieces a lane has in flight

// the sum over the team's lanes, in all of them
__device__ __forceinline__ uint32_t rm_team_sum(uint32_t v, uint32_t logL) {
#define DLC_RM_ADD(c) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, c, 0xF, 0xF, true)
    if (logL > 0u) DLC_RM_ADD(0xB1);   // the neighbour
    if (logL > 1u) DLC_RM_ADD(0x4E);   // the other pair of four
    if (logL > 2u) DLC_RM_ADD(0x141);  // the other four of eight
    if (logL > 3u) DLC_RM_ADD(0x140);  // the other eight of sixteen
#undef DLC_RM_ADD
    if (logL > 4u) v += (uint32_t)__shfl_xor((int)v, 16, 64);
    if (logL > 5u) v += (uint32_t)__shfl_xor((int)v, 32, 64);
    return v;
}

// LONG: rows of more than 64 pieces, 64 at a time (the multipliers with them)
template <bool F16, bool LONG>
__global__ __launch_bounds__(256) void k_rm_hash_team(const void* payload, Geom g, const QParam* qp, const uint8_t* on,
                                                      uint64_t* rowhash, const uint8_t* sym_plane,
                                                      const uint32_t* __restrict__ mult, uint32_t logL) {
    const uint32_t t = blockIdx.y;
    if (!on[t]) return;  // uniform
    const uint32_t lane = threadIdx.x & 63u, L = 1u << logL, sub = lane & (L - 1u), team = lane >> logL, rps = 64u >> logL;
    const uint32_t W = g.D / 16u;
    const QParam q = qp[t];
    const float Rf = (float)g.R;
    const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
    const uint4* plane = reinterpret_cast<const uint4*>(sym_plane + (size_t)t * plane_stride(g));
    uint64_t* const out = rowhash + (size_t)t * g.B;
    uint4 m03[4];
    uint2 m45[4];
    auto load_mult = [&](uint32_t piece) {
        const uint32_t* m = mult + 32u * min(piece, W - 1u);  // (a lane past the row's end holds zeroes and adds nothing)
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            m03[k] = *reinterpret_cast<const uint4*>(m + 8u * k);
            m45[k] = *reinterpret_cast<const uint2*>(m + 8u * k + 4u);
        }
    };
    if constexpr (!LONG) load_mult(sub);
    const uint32_t step = kRmBlk * rps;  // rows a wavefront does at a time
    const uint32_t waves = gridDim.x * 4u, wave = blockIdx.x * 4u + (threadIdx.x >> 6);
    for (uint32_t row0 = wave * step; row0 < g.B; row0 += waves * step) {
        uint32_t a[kRmBlk][3];
#pragma unroll
        for (uint32_t u = 0; u < kRmBlk; ++u) a[u][0] = a[u][1] = a[u][2] = 0u;
        for (uint32_t p0 = 0; p0 < (LONG ? W : 1u); p0 += 64u) {
            const uint32_t p = p0 + sub;
            uint4 v[kRmBlk];
#pragma unroll
            for (uint32_t u = 0; u < kRmBlk; ++u) {
                const uint32_t row = row0 + u * rps + team;
                v[u] = row < g.B && p < W ? plane[(size_t)row * W + p] : make_uint4(0u, 0u, 0u, 0u);
            }
            if constexpr (LONG) load_mult(p);
#pragma unroll
            for (uint32_t u = 0; u < kRmBlk; ++u) {
                const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                bool other = false;
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    rm_add_piece(w[k], m03[k], m45[k], a[u]);
                    other = other || rm_has255(w[k]);
                }
                if (other) {  // rare
                    const uint32_t row = row0 + u * rps + team;
                    for (uint32_t k = 0; k < 4; ++k) {
                        for (uint32_t b = 0; b < 4; ++b) {
                            if (((w[k] >> (8u * b)) & 255u) < kWinEsc) continue;
                            const uint32_t e = (p * 4u + k) * 4u + b;
                            rm_add_other(rm_identity<F16>(tab, row * g.D + e, q, Rf, (int)g.R), e, a[u]);
                        }
                    }
                }
            }
        }
        uint32_t mine[3] = {0u, 0u, 0u};
#pragma unroll
        for (uint32_t u = 0; u < kRmBlk; ++u) {
#pragma unroll
            for (uint32_t i = 0; i < 3; ++i) {
                a[u][i] = rm_team_sum(a[u][i], logL);
                if (sub == u) mine[i] = a[u][i];
            }
        }
        const uint32_t row = row0 + sub * rps + team;  // (a team has kRmBlk lanes or more)
        if (sub < kRmBlk && row < g.B) out[row] = rm_finish(mine);
    }
}

// the sets: work-group (part, t, set) takes the rows of table t whose hashes' top bits say `part`, puts them into an
// open-addressing set in LDS, where the smallest row index of a hash stays, and then looks every one of its rows up again:
// own[row] = the smallest row index with the row's hash.
// TAG (batches of kRmTagRows at most): a slot holds the hash's upper 48 bits and the row's index, so that neither way
// leaves the LDS and the smaller index wins by a minimum of whole slots; the place in the set comes from the lower bits, so
// rows whose hashes differ meet in one slot only if 48 bits agree and the others lead to neighbouring places (2^-58 for a
// pair; those who use the owners compare the rows, and treat such a pair as one whose hashes agree).  Otherwise a slot holds
// an index alone, and the hash of the row that sits there is read from memory.  128 tables of 8192 rows, two sets:
// 25 us, 45 before (a dependent read of memory for every row on each way); one set of 64 tables 14, before 32.  Of that the
// strides of every hash's own made 3 (with the next place for all, the longest of 64 lanes' searches is what counts).
// A table's work-groups differ in y alone: they read the same hashes, and for multiples of eight tables through the same L2.
// n_slots (a power of two) is the batch size or more whenever that fits the LDS, so the set cannot fill up; for larger
// batches a work-group's share of the rows is half the slots or less, and where a set does fill up all the same (hashes that
// crowd into one share), the rows that found no slot are their own owners (coded rows, for row matching), and ctrl, if given,
// gets an error (the statistics want exact counts).  rowhash and own: [sets][T][B]; on (optional): tables to skip; unique
// (optional): [T][sets] counts of the rows that own their hash.
constexpr uint32_t kRmTagRows = 65536;
template <bool TAG>
__global__ __launch_bounds__(1024) void k_rm_sets(Geom g, const uint8_t* on, const uint64_t* rowhash, uint32_t* own,
                                                  uint32_t n_slots, uint32_t parts, uint32_t* unique, Ctrl* ctrl) {
    typedef std::conditional_t<TAG, unsigned long long, uint32_t> Slot;
    extern __shared__ __align__(16) uint32_t slot_words[];
    __shared__ uint32_t s_owners;
    const uint32_t part = blockIdx.y, t = blockIdx.x, set = blockIdx.z, tid = threadIdx.x;
    if (on && !on[t]) return;  // uniform
    constexpr Slot kEmpty = (Slot)~0ull;  // (as a row's slot: the batch's last possible row, which no later row looks for)
    constexpr uint32_t kBatch = 4;  // hashes a thread loads back to back
    constexpr uint64_t kTag = ~(uint64_t)(kRmTagRows - 1u);
    const uint64_t* rh = rowhash + ((size_t)set * g.T + t) * g.B;
    uint32_t* own_t = own + ((size_t)set * g.T + t) * g.B;
    uint64_t h[kBatch];
    auto load = [&](uint32_t r0) {
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) h[k] = r0 + k * 1024u < g.B ? rh[r0 + k * 1024u] : 0ull;
    };
    load(tid);
    Slot* slot = reinterpret_cast<Slot*>(slot_words);
    volatile Slot* vslot = slot;
    for (uint32_t k = tid; k < n_slots * (uint32_t)sizeof(Slot) / 16u; k += 1024)
        reinterpret_cast<uint4*>(slot_words)[k] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (tid == 0) s_owners = 0u;
    __syncthreads();
    auto mine = [&](uint32_t row, uint64_t hash) { return row < g.B && ((uint32_t)(hash >> 52) & (parts - 1u)) == part; };
    auto place = [&](uint64_t hash) { return (uint32_t)(TAG ? hash : hash >> 20) & (n_slots - 1u); };
    auto stride = [&](uint64_t hash) { return (uint32_t)(hash >> 32) | 1u; };  // (odd: all places in turn)
    auto same = [&](Slot cur, uint64_t hash) {  // is the row in this slot one with this hash?
        if constexpr (TAG) return ((cur ^ hash) & kTag) == 0ull;
        else return rh[cur] == hash;
    };
    for (uint32_t r0 = tid; r0 < g.B; r0 += 1024u * kBatch) {
        if (r0 != tid) load(r0);
        // the first place of every row: the reads of a batch together, then the exchanges; what is left goes on by itself
        Slot me[kBatch], cur[kBatch];
        bool left[kBatch];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            const uint32_t row = r0 + k * 1024u;
            left[k] = mine(row, h[k]);
            me[k] = TAG ? (Slot)((h[k] & kTag) | row) : (Slot)row;
            cur[k] = vslot[place(h[k])];
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            if (left[k] && cur[k] == kEmpty) {
                cur[k] = atomicCAS(&slot[place(h[k])], kEmpty, me[k]);
                left[k] = cur[k] != kEmpty;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            if (!left[k]) continue;
            uint32_t pos = place(h[k]);
            Slot c = cur[k];
            bool placed = false;
            for (uint32_t probe_n = 0; probe_n < n_slots; ++probe_n) {
                if (c == kEmpty) {
                    c = atomicCAS(&slot[pos], kEmpty, me[k]);
                    if (c == kEmpty) { placed = true; break; }
                }
                if (same(c, h[k])) {
                    if (me[k] < c) atomicMin(&slot[pos], me[k]);
                    placed = true;
                    break;
                }
                pos = (pos + stride(h[k])) & (n_slots - 1u);
                c = vslot[pos];
            }
            if (!placed && ctrl) set_status(ctrl, DLC_ESTATE);
        }
    }
    __syncthreads();
    uint32_t owners = 0;
    for (uint32_t r0 = tid; r0 < g.B; r0 += 1024u * kBatch) {
        if (g.B > 1024u * kBatch) load(r0);  // (else they are still there)
        Slot cur[kBatch];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) cur[k] = vslot[place(h[k])];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            const uint32_t row = r0 + k * 1024u;
            if (!mine(row, h[k])) continue;
            uint32_t o = row;
            uint32_t pos = place(h[k]);
            Slot c = cur[k];
            for (uint32_t probe_n = 0; probe_n < n_slots && c != kEmpty; ++probe_n) {
                if (same(c, h[k])) {
                    o = (uint32_t)c & (TAG ? kRmTagRows - 1u : 0xFFFFFFFFu);
                    break;
                }
                pos = (pos + stride(h[k])) & (n_slots - 1u);
                c = vslot[pos];
            }
            own_t[row] = o;
            owners += o == row ? 1u : 0u;
        }
    }
    if (unique) {  // uniform
        owners = wave_sum(owners);
        if ((tid & 63u) == 0u && owners) atomicAdd(&s_owners, owners);
        __syncthreads();
        if (tid == 0 && s_owners) atomicAdd(&unique[(size_t)t * gridDim.z + set], s_owners);
    }
}

// pass 2: ref[row] = the owner of the row's hash if the two rows are equal element by element, else the row itself.
// The elements of a row that refers to another leave the table's counts again (the histogram kernel has counted
// every row) and get index 253 in the plane, which the encode kernel's table maps to no bits at all.  Only rows
// that nobody compares with are changed: an owner is never such a row.
// A lane holds a piece of PW words of the plane (16 bytes where the row length allows, else 4); a row is the work
// of a team of 2^logL lanes, the smallest power of two that covers the row's pieces (64 at most: longer rows take
// several trips); a wavefront works on 64 rows per trip: those with an earlier owner are put next to one another, 64 >> logL
// at a time are compared.  64 tables of 8192 x 128: 24 us; all 64 rows walked, the idle ones under a condition, 26, four sets
// of them in flight at half the wavefronts 34.  (rows: 64, or fewer where that leaves too few wavefronts, see launch_row_match)
template <uint32_t PW>
struct RmPiece { uint32_t v[PW]; };

template <uint32_t PW>
__device__ __forceinline__ RmPiece<PW> rm_load_piece(const uint32_t* plane, size_t piece) {
    RmPiece<PW> r;
    if constexpr (PW == 4) {
        const uint4 q = *reinterpret_cast<const uint4*>(plane + piece * 4u);
        r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
    } else {
        r.v[0] = plane[piece];
    }
    return r;
}

template <bool F16, uint32_t PW>
__global__ __launch_bounds__(256) void k_rm_owner(const void* payload, Geom g, const QParam* qp, const uint8_t* on,
                                                  const uint32_t* rowown, const uint64_t* rowhash, uint32_t* ref, uint8_t* sym_plane,
                                                  uint32_t* hist, TableOrder order, uint32_t logL, uint32_t rows) {
    extern __shared__ __align__(16) uint32_t lh[];  // what to take off the counts: window [kWinBins + 1][kWinCopies] | exact [K]
    uint32_t t, block;
    order.place(&t, &block);
    if (t >= g.T) return;  // uniform
    const uint32_t waves_grid = order.bx * 4u;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave_global = block * 4 + (tid >> 6);
    uint32_t* ref_t = ref + (size_t)t * g.B;
    if (!on[t]) {  // uniform: every row is a coded row
        for (uint32_t row = wave_global * 64 + lane; row < g.B; row += waves_grid * 64) ref_t[row] = row;
        return;
    }
    const uint32_t n_words = (kWinBins + 1u) * kWinCopies + g.K;
    {
        uint4* z = reinterpret_cast<uint4*>(lh);
        for (uint32_t k = tid; k < (n_words + 3u) / 4u; k += 256) z[k] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    uint32_t* win = lh + (lane & (kWinCopies - 1u));
    uint32_t* exact = lh + (kWinBins + 1u) * kWinCopies;
    const uint32_t L = 1u << logL, sub = lane & (L - 1u), team = lane >> logL, rps = 64u >> logL, W = g.D / (4u * PW);
    const uint64_t teammask = (L == 64u ? ~0ull : ((1ull << L) - 1ull)) << (team * L);
    const QParam q = qp[t];
    const float Rf = (float)g.R;
    const uint8_t* tab = static_cast<const uint8_t*>(payload) + (size_t)t * g.n * g.es;
    uint32_t* plane = reinterpret_cast<uint32_t*>(sym_plane + (size_t)t * plane_stride(g));
    for (uint32_t row0 = wave_global * rows; row0 < g.B; row0 += waves_grid * rows) {
        // the rows that have an earlier owner are put next to one another, rps of them are compared at a time
        const uint32_t row_mine = row0 + lane;
        const uint32_t end = min(g.B, row0 + rows);
        const uint32_t own_mine = row_mine < end ? rowown[(size_t)t * g.B + row_mine] : 0xFFFFFFFFu;
        const bool need_mine = own_mine < row_mine;  // (an owner is never a later row)
        if (row_mine < end && !need_mine) ref_t[row_mine] = row_mine;
        const uint64_t mask = __ballot(need_mine);
        const uint32_t n = (uint32_t)__popcll(mask), rank = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        const int to = (int)((need_mine ? rank : n + lane - rank) << 2);
        const uint32_t list_row = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)row_mine);
        const uint32_t list_own = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)own_mine);
        for (uint32_t i0 = 0; i0 < n; i0 += rps) {
            const bool need = i0 + team < n;
            const uint32_t row = (uint32_t)__shfl((int)list_row, (int)(need ? i0 + team : 0u), 64);
            uint32_t own = (uint32_t)__shfl((int)list_own, (int)(need ? i0 + team : 0u), 64);
            bool differ = false;
            RmPiece<PW> w;  // the row's piece of the last trip (the only one unless a row has more than 64 pieces)
#pragma unroll
            for (uint32_t k = 0; k < PW; ++k) w.v[k] = 0u;
            for (uint32_t p = sub; p < W; p += L) {
                if (need) {
                    w = rm_load_piece<PW>(plane, (size_t)row * W + p);
                    const RmPiece<PW> b = rm_load_piece<PW>(plane, (size_t)own * W + p);
                    uint32_t x = 0u;
                    bool other = false;
#pragma unroll
                    for (uint32_t k = 0; k < PW; ++k) {
                        x |= w.v[k] ^ b.v[k];
                        other = other || rm_has255(w.v[k]);
                    }
                    if (x != 0u) differ = true;
                    else if (other) {  // rare: the elements outside the window, by what they are
                        for (uint32_t k = 0; k < PW; ++k) {
                            for (uint32_t v = 0; v < 4; ++v) {
                                if (((w.v[k] >> (8u * v)) & 255u) < kWinEsc) continue;
                                const uint32_t e = (p * PW + k) * 4u + v;
                                if (rm_identity<F16>(tab, row * g.D + e, q, Rf, (int)g.R) != rm_identity<F16>(tab, own * g.D + e, q, Rf, (int)g.R))
                                    differ = true;
                            }
                        }
                    }
                }
            }
            bool same = need && (__ballot(differ) & teammask) == 0ull;  // the same for all lanes of a team
            // A row that is not its hash's owner's equal: two different rows with one hash.  The first earlier row
            // with the row's content, if there is one, has that hash too: the whole wavefront looks through the
            // earlier rows with it, one such row at a time (never expected; slow and plain).
            uint64_t coll = __ballot(need && !same && sub == 0u);
            while (coll != 0ull) {  // uniform over the wavefront
                const uint32_t leader = (uint32_t)__ffsll((unsigned long long)coll) - 1u;
                coll &= coll - 1ull;
                const uint32_t crow = lane_read(row, leader);
                const uint64_t h = rowhash[(size_t)t * g.B + crow];
                uint32_t found = crow;
                for (uint32_t j0 = 0; j0 < crow && found == crow; j0 += 64u) {
                    const uint32_t j = j0 + lane;
                    uint64_t m = __ballot(j < crow && rowhash[(size_t)t * g.B + j] == h);
                    while (m != 0ull && found == crow) {
                        const uint32_t jj = j0 + (uint32_t)__ffsll((unsigned long long)m) - 1u;
                        m &= m - 1ull;
                        bool d = false;
                        for (uint32_t e = lane; e < g.D; e += 64u)
                            d = d || rm_identity<F16>(tab, crow * g.D + e, q, Rf, (int)g.R) != rm_identity<F16>(tab, jj * g.D + e, q, Rf, (int)g.R);
                        if (__ballot(d) == 0ull) found = jj;
                    }
                }
                if (found != crow && team == (leader >> logL)) {
                    own = found;
                    same = true;
                }
            }
            if (sub == 0u && need) ref_t[row] = same ? own : row;
            if (!same) continue;
            for (uint32_t p = sub; p < W; p += L) {
                const RmPiece<PW> wv = W <= L ? w : rm_load_piece<PW>(plane, (size_t)row * W + p);
#pragma unroll
                for (uint32_t k = 0; k < PW; ++k) {
                    if (!rm_has255(wv.v[k])) {
#pragma unroll
                        for (uint32_t v = 0; v < 4; ++v) atomicSub(&win[((wv.v[k] >> (8u * v)) & 255u) * kWinCopies], 1u);
                    } else {
                        for (uint32_t v = 0; v < 4; ++v) {
                            const uint32_t idx = (wv.v[k] >> (8u * v)) & 255u;
                            if (idx < kWinEsc) {
                                atomicSub(&win[idx * kWinCopies], 1u);
                            } else {
                                const uint64_t id = rm_identity<F16>(tab, row * g.D + (p * PW + k) * 4u + v, q, Rf, (int)g.R);
                                atomicSub(&exact[(id >> 32) ? 0u : (uint32_t)id], 1u);
                            }
                        }
                    }
                }
                if constexpr (PW == 4) *reinterpret_cast<uint4*>(plane + ((size_t)row * W + p) * 4u) = make_uint4(0xFDFDFDFDu, 0xFDFDFDFDu, 0xFDFDFDFDu, 0xFDFDFDFDu);
                else plane[(size_t)row * W + p] = 0xFDFDFDFDu;
            }
        }
    }
    __syncthreads();
    // merge (the sums are negative numbers modulo 2^32, and so is what the global counts get added)
    const uint32_t win_lo = win_lo_of(g.R);
    for (uint32_t k = tid; k < g.K; k += 256) {
        uint32_t s = exact[k];
        const uint32_t wi = k - win_lo;
        if (wi < kWinSkip) {
            const uint32_t* row = lh + wi * kWinCopies;
            for (uint32_t c = 0; c < kWinCopies; ++c) s += row[(c + tid) & (kWinCopies - 1u)];
        }
        if (s) atomicAdd(&hist[(size_t)t * g.K + k], s);
    }
}

void row_match_multipliers(uint32_t* mult, uint32_t n_pieces) {
    for (uint32_t p = 0; p < n_pieces; ++p)
        for (uint32_t i = 0; i < 8; ++i) mult[8 * p + i] = i < 6 ? (rm_mix32(p * 6u + i + 1u) & 0xFFFFFFu) : 0u;
}

hipError_t launch_row_sets(const Geom& g, uint32_t n_sets, const uint8_t* on, const uint64_t* rowhash, uint32_t* own,
                           uint32_t* unique, Ctrl* ctrl, hipStream_t s) {
    // slots for the whole batch, 16384 at most; a work-group a compute unit (32 per table and set at most: each reads all the
    // table's hashes; 64 tables of 8192: 14 us, with two work-groups a compute unit 20; 9, 26 and 65 tables of 16384, whose
    // sets fill a compute unit's LDS, with the next more: 31, 35 and 41 us, so 19, 21 and 28), and more where a batch is large:
    // a work-group's share of the rows is half its slots or less (up to 32 M rows)
    uint32_t n_slots = 64;
    while (n_slots < g.B && n_slots < 16384u) n_slots <<= 1;
    uint32_t parts = 1;
    while (parts < 32u && 2u * parts * g.T * n_sets <= 256u) parts <<= 1;
    while (parts < 4096u && (uint64_t)parts * n_slots < 2ull * g.B) parts <<= 1;
    if (g.B <= kRmTagRows)
        hipLaunchKernelGGL(k_rm_sets<true>, dim3(g.T, parts, n_sets), dim3(1024), n_slots * 8u, s, g, on, rowhash, own, n_slots, parts,
                           unique, ctrl);
    else
        hipLaunchKernelGGL(k_rm_sets<false>, dim3(g.T, parts, n_sets), dim3(1024), n_slots * 4u, s, g, on, rowhash, own, n_slots, parts,
                           unique, ctrl);
    return hipGetLastError();
}

// work-groups of four wavefronts a table, `rows` rows at a time each: 32 at most where there are tables enough, else as many as
// a thousand work-groups need (whole calls, us, with 32 for all and with this: one table of 65536 x 128 221 and 143, of 300000 x
// 64 682 and 447)
static uint32_t row_blocks(const Geom& g, uint32_t rows) {
    return std::min<uint32_t>((g.B + 4u * rows - 1u) / (4u * rows), std::max<uint32_t>(32u, 1024u / g.T));
}

hipError_t launch_row_match(const Geom& g, const void* payload, const Ws& w, hipStream_t s) {
    const uint32_t pw = g.D % 16u == 0u ? 4u : 1u;  // words of the plane per lane in pass 2
    uint32_t logL = 0;
    while (logL < 6 && (1u << logL) < g.D / (4u * pw)) ++logL;
    const size_t sm = hist_lds_bytes(g.K);
    const dim3 block(256);
    if (pw == 4u && g.D >= 256u) {
        const uint32_t trips = (uint32_t)((((uint64_t)g.B << logL) + 64u * kRmBlk - 1u) / (64u * kRmBlk));  // of a wavefront
        const dim3 grid((trips + 7u) / 8u, g.T);  // two each
#define DLC_RM_HASH(FF, LL) hipLaunchKernelGGL((k_rm_hash_team<FF, LL>), grid, block, 0, s, payload, g, w.qp, w.rm_on, w.rm_hash, w.sym_plane, w.rm_mult, logL)
        if (g.D > 1024u) { if (g.dtype == DLC_F16) DLC_RM_HASH(true, true); else DLC_RM_HASH(false, true); }
        else { if (g.dtype == DLC_F16) DLC_RM_HASH(true, false); else DLC_RM_HASH(false, false); }
#undef DLC_RM_HASH
    } else {
        const dim3 grid(row_blocks(g, 64u), g.T);
        const uint32_t waves_grid = grid.x * 4u;
        if (g.dtype == DLC_F16)
            hipLaunchKernelGGL(k_rm_hash<true>, grid, block, 0, s, payload, g, w.qp, w.rm_on, w.rm_hash, w.sym_plane, w.rm_mult, waves_grid);
        else
            hipLaunchKernelGGL(k_rm_hash<false>, grid, block, 0, s, payload, g, w.qp, w.rm_on, w.rm_hash, w.sym_plane, w.rm_mult, waves_grid);
    }
    {
        hipError_t e = launch_row_sets(g, 1u, w.rm_on, w.rm_hash, w.rm_own, nullptr, nullptr, s);
        if (e != hipSuccess) return e;
    }
    // A wavefront takes 64 rows at a time, fewer (but a row a team) where there would be less than eight wavefronts a compute unit,
    // or sixteen where a row takes a wavefront's time.  Whole calls, us, at 64 rows and at this rule's: one table of 8192 x 128 64
    // and 60, 9 of them 83 and 80, 26 of 512 x 64 48.4 and 46.4, 4 of 1024 x 512 75 and 56, 16 of 2048 x 1024 153 and 116; four
    // thousand wavefronts for short rows too: one of 65536 x 128 149 instead of 143.
    uint32_t rows = 64u;
    const uint32_t lim = g.D >= 256u ? 4096u : 2048u;
    while (rows > 8u && rows > (64u >> logL) && (uint64_t)g.T * g.B < (uint64_t)lim * rows) rows /= 2u;
    // tables apart and one after the other, us: one of 65536 rows 74 and 69; 9, 26, 44, 64 and 128 of 8192 x 128 14.1 and 13.4, 17.1
    // and 16.3, 20.3 both, 24.4 and 25.0, 41.1 and 43.4
    const TableOrder order(row_blocks(g, rows), g.T >= 48u);
#define DLC_RM_OWNER(FF, PP) hipLaunchKernelGGL((k_rm_owner<FF, PP>), dim3(order.groups(g.T)), block, sm, s, payload, g, w.qp, w.rm_on, w.rm_own, w.rm_hash, w.rm_ref, w.sym_plane, w.hist, order, logL, rows)
    if (g.dtype == DLC_F16) { if (pw == 4u) DLC_RM_OWNER(true, 4); else DLC_RM_OWNER(true, 1); }
    else { if (pw == 4u) DLC_RM_OWNER(false, 4); else DLC_RM_OWNER(false, 1); }
#undef DLC_RM_OWNER
    return hipGetLastError();
}

hipError_t row_match_set_attributes() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_rm_sets<true>), hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 8);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k_rm_sets<false>), hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 4);
}

}  // namespace dlc
