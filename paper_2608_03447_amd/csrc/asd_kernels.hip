// gfx950 kernels of the ASD verifier.
//
// Stage 1 (asd_row_kernel): one workgroup per (row, vocabulary split) tile
// streams the tile's logits once from HBM with 16-byte non-temporal loads and
// keeps, per lane, the greatest logit seen so far (Eq. 1).  Logits are compared
// as order-preserving integer keys, so the whole reduction is integer max work
// with no rounding.  The tile that owns the draft token's column also gathers
// z(x) (Eq. 3).  With one tile per row the tile writes the row's record:
// argmax, mismatch bit d (Eq. 5) and regret r = fl32(z(y*) - z(x)).  With
// several tiles per row each tile writes a partial; no workgroup waits for or
// signals another.  Block 0 also writes the packed row offsets of the requests.
//
// Stage 2 (asd_scan_kernel): one wavefront per request runs Algorithm 1 with
// lanes = block positions.  Each lane forms its row's record (or combines the
// row's split partials), then the wavefront ballots the mismatches and walks
// only those, in position order: the B = 0 dispatch stops at the first one
// (Eq. 2); otherwise a mismatch is accepted while the gate r <= g q (Eqs. 7,
// 11), the budget fl32(s + C) <= B (Eq. 9) and the cap N <= M (Eq. 10) hold,
// and the first that fails ends the longest feasible prefix (Eq. 12).  Exact
// matches in between are feasible by Eq. 14's first term.  The running sum C
// is accumulated in position order, one binary32 addition per accepted
// mismatch, exactly as the sequential definition does.  Then the ledger update
// (Eq. 13) and the recovery or bonus token.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <mutex>

#include "asd_plan.h"

// Workspace of asd_verify_static, for callers that cannot allocate: one fixed
// array per device, held until the process ends.  In host code its name is
// only a stand-in for the symbol, not a device address; host code uses the
// address static_scratch_address returns for the current device.
static __device__ __align__(256) unsigned char scratch[asd::kStaticScratchBytes];

namespace asd {

hipError_t static_scratch_address(void** ptr) {
    static std::mutex m;
    static std::map<int, void*> by_device;   // each device holds its own copy
    int device = 0;
    hipError_t err = hipGetDevice(&device);
    if (err != hipSuccess) return err;
    std::lock_guard<std::mutex> lock(m);
    auto it = by_device.find(device);
    if (it == by_device.end()) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return err;
        if (p == nullptr) return hipErrorInvalidSymbol;
        it = by_device.emplace(device, p).first;
    }
    *ptr = it->second;
    return hipSuccess;
}

// Sticky error word of this device: the kernels OR in kErr* bits when they meet
// data that the verifier reads in a defined but unusual way.
__device__ uint32_t asd_error_word;

hipError_t error_word_address(uint32_t** ptr) {
    return hipGetSymbolAddress((void**)ptr, HIP_SYMBOL(asd_error_word));
}

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// 16-byte vectors per lane per group in the streaming loop.
constexpr int kUnroll = 4;
constexpr int kGroupVecs = kRowThreads * kUnroll;
constexpr int kWaves = kRowThreads / 64;

// ------------------------------------------------------------ integer keys
//
// key(x) is an integer that orders logits the way the argmax must: numeric
// order with -0 == +0, and every NaN, of either sign and any payload, above
// +inf and equal to every other NaN (so a row's first NaN is its argmax).  For
// a number's sign-magnitude pattern: key = magnitude when the sign is clear,
// key = -magnitude when it is set; every NaN has the key kNan, one above +inf's.

// Smallest key of each dtype (below every key a real logit can have), the key
// of +inf, the key of every NaN, and the greatest pattern that is not a NaN
// with the sign bit set (-inf's).
template <int EB> struct KeyTraits;
template <> struct KeyTraits<2> {
    static constexpr uint32_t kNonePacked = 0x80008000u;   // bf16 keys lie in [-0x7f80, 0x7f81]
    static constexpr int32_t kInf = 0x7f80;
    static constexpr int32_t kNan = 0x7f81;
    static constexpr uint32_t kNegInfPattern = 0xff80u;
};
template <> struct KeyTraits<4> {
    static constexpr int32_t kNone = (int32_t)0x80000000;   // f32 keys >= -0x7f800000
    static constexpr int32_t kInf = 0x7f800000;
    static constexpr int32_t kNan = 0x7f800001;
    static constexpr uint32_t kNegInfPattern = 0xff800000u;
};

// The key of every binary32 pattern (used where one pass must rank anything).
__device__ __forceinline__ int32_t f32_key(uint32_t u) {
    const uint32_t mag = u & 0x7fffffffu;
    const int32_t key = (int32_t)u < 0 ? -(int32_t)mag : (int32_t)mag;
    return mag > 0x7f800000u ? KeyTraits<4>::kNan : key;
}

// Three ways to rank logits, cheapest first.
//  kKeysRaw:   the raw bit patterns read as signed integers.  For every pattern
//              with the sign bit clear that is neither +0 nor a NaN this equals
//              the key, and every pattern with the sign bit set reads as
//              negative.  So among elements that include a number in [1, +inf]
//              and no NaN, the raw maximum is the exact maximum, found with one
//              integer max per element.
//  kKeysExact: sign-magnitude keys, exact for every number.
//  kKeysNan:   min(magnitude, kNan): every NaN gets kNan and every number a
//              smaller key, so in a tile known to hold a NaN the greatest key
//              is kNan and its first element is the tile's first NaN.
// With raw and sign-magnitude keys a NaN's key is not kNan.  Those passes keep
// the greatest pattern read as unsigned, which exceeds -inf's exactly when a
// NaN with the sign bit set is present; a NaN with it clear shows as a greatest
// key above +inf's.  Either sends the tile to a NaN pass.
constexpr int kKeysRaw = 0, kKeysExact = 1, kKeysNan = 2;
constexpr int32_t kRawExactFrom = 1;

// Two bf16 sign-magnitude keys at once, one per 16-bit half.
__device__ __forceinline__ uint32_t bf16x2_keys(uint32_t w) {
    const u16x2 v = __builtin_bit_cast(u16x2, w);
    const u16x2 neg = (u16x2)(unsigned short)0x8000 - v;       // -magnitude, mod 2^16
    const u16x2 sign = __builtin_bit_cast(u16x2, __builtin_bit_cast(s16x2, v) >> (s16x2)15);
    return __builtin_bit_cast(uint32_t, (neg & sign) | (v & ~sign));
}

__device__ __forceinline__ uint32_t pkmax16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, a),
                                                                  __builtin_bit_cast(s16x2, b)));
}

__device__ __forceinline__ uint32_t pkmaxu16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}

__device__ __forceinline__ uint32_t pkminu16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}

template <int EB, int kMode>
__device__ __forceinline__ uint32_t dword_keys(uint32_t w) {
    if constexpr (kMode == kKeysRaw) {
        return w;
    } else if constexpr (kMode == kKeysExact) {
        if constexpr (EB == 2) return bf16x2_keys(w);
        else return (int32_t)w < 0 ? 0x80000000u - w : w;
    } else {
        if constexpr (EB == 2) return pkminu16(w & 0x7fff7fffu, (uint32_t)KeyTraits<2>::kNan * 0x10001u);
        else return min(w & 0x7fffffffu, (uint32_t)KeyTraits<4>::kNan);
    }
}

// Max key over the 16-byte vectors of one group.  With raw and sign-magnitude
// keys `umax` also takes the greatest pattern read as unsigned (per 16-bit half
// for bf16).
template <int EB, int kMode>
__device__ __forceinline__ int32_t group_max_key(const u32x4 (&raw)[kUnroll], uint32_t& umax) {
    if constexpr (EB == 2) {
        uint32_t acc = KeyTraits<2>::kNonePacked;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t k0 = dword_keys<2, kMode>(raw[u].x), k1 = dword_keys<2, kMode>(raw[u].y);
            const uint32_t k2 = dword_keys<2, kMode>(raw[u].z), k3 = dword_keys<2, kMode>(raw[u].w);
            uint32_t m = pkmax16(pkmax16(k0, k1), pkmax16(k2, k3));
            acc = pkmax16(acc, m);
            if constexpr (kMode != kKeysNan)
                umax = pkmaxu16(umax, pkmaxu16(pkmaxu16(raw[u].x, raw[u].y),
                                               pkmaxu16(raw[u].z, raw[u].w)));
        }
        const int32_t lo = (int32_t)(int16_t)(acc & 0xffffu);
        const int32_t hi = (int32_t)acc >> 16;
        return lo > hi ? lo : hi;
    } else {
        int32_t acc = KeyTraits<4>::kNone;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            int32_t m = max(max((int32_t)dword_keys<4, kMode>(raw[u].x),
                                (int32_t)dword_keys<4, kMode>(raw[u].y)),
                            max((int32_t)dword_keys<4, kMode>(raw[u].z),
                                (int32_t)dword_keys<4, kMode>(raw[u].w)));
            acc = max(acc, m);
            if constexpr (kMode != kKeysNan)
                umax = max(umax, max(max(raw[u].x, raw[u].y), max(raw[u].z, raw[u].w)));
        }
        return acc;
    }
}

// Key of a bf16 bit pattern (low 16 bits of h16) or f32 bit pattern.
template <int EB, int kMode>
__device__ __forceinline__ int32_t key_of(uint32_t pattern) {
    if constexpr (EB == 2) return (int32_t)(int16_t)(dword_keys<2, kMode>(pattern) & 0xffffu);
    else return (int32_t)dword_keys<4, kMode>(pattern);
}

// Greatest key among the elements of one dword (two bf16 or one f32).
template <int EB, int kMode>
__device__ __forceinline__ int32_t dword_max_key(uint32_t w) {
    const uint32_t k = dword_keys<EB, kMode>(w);
    if constexpr (EB == 2) {
        const int32_t lo = (int32_t)(int16_t)(k & 0xffffu), hi = (int32_t)k >> 16;
        return lo > hi ? lo : hi;
    } else {
        return (int32_t)k;
    }
}

template <int EB, int kMode>
__device__ __forceinline__ void load_scalar(const unsigned char* p, int32_t& key, uint32_t& bits) {
    if constexpr (EB == 2) {
        const uint32_t h = *(const unsigned short*)p;
        key = key_of<2, kMode>(h);
        bits = h << 16;
    } else {
        bits = *(const uint32_t*)p;
        key = key_of<4, kMode>(bits);
    }
}

// Pack (key, column) so that the unsigned maximum is the greatest key with the
// lowest column.
__device__ __forceinline__ unsigned long long pack_kc(int32_t key, int64_t col) {
    return ((unsigned long long)((uint32_t)key ^ 0x80000000u) << 32) |
           (unsigned long long)(0xffffffffu - (uint32_t)col);
}
__device__ __forceinline__ int32_t packed_col(unsigned long long p) {
    return (int32_t)(0xffffffffu - (uint32_t)(p & 0xffffffffull));
}
__device__ __forceinline__ int32_t packed_key(unsigned long long p) {
    return (int32_t)((uint32_t)(p >> 32) ^ 0x80000000u);
}

__device__ __forceinline__ void take_better(unsigned long long& p, uint32_t& bits,
                                            unsigned long long q, uint32_t qbits) {
    if (q > p) {
        p = q;
        bits = qbits;
    }
}

// One step of a wavefront maximum of (packed, bits) by DPP: each lane takes
// the pair of the lane that `kCtrl` names when it is greater.  A lane with no
// source lane in the step (or in a row that kRowMask leaves out) reads 0,
// which ranks below every packed pair.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ void dpp_max_step(unsigned long long& p, uint32_t& bits) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)p, kCtrl, kRowMask,
                                                              0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(p >> 32), kCtrl,
                                                              kRowMask, 0xf, false);
    const uint32_t qb = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)bits, kCtrl, kRowMask, 0xf,
                                                              false);
    const unsigned long long q = ((unsigned long long)hi << 32) | lo;
    const bool take = q > p;
    p = take ? q : p;
    bits = take ? qb : bits;
}

// Unsigned 64-bit maximum of a lane's value and that of the lane `kCtrl`
// names (a DPP pattern in which every lane has a source).
template <int kCtrl>
__device__ __forceinline__ unsigned long long dpp_umax64(unsigned long long p) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)p, kCtrl, 0xf, 0xf,
                                                              false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(p >> 32), kCtrl,
                                                              0xf, 0xf, false);
    const unsigned long long q = ((unsigned long long)hi << 32) | lo;
    return q > p ? q : p;
}

// Workgroup-wide maximum of (packed, bits), and the OR of one flag per
// wavefront; every thread returns with both.  Within a wavefront, shifts of 1,
// 2, 4 and 8 lanes make lane 15 of each 16-lane row hold the row's maximum,
// and the broadcasts of lanes 15 and 31 carry it on, so that lane 63 holds the
// wavefront's.  No cross-lane step waits on LDS.  The wavefronts' results meet
// in LDS behind one barrier.
__device__ __forceinline__ bool block_reduce(unsigned long long& p, uint32_t& bits, bool flag) {
    __shared__ unsigned long long s_p[kWaves];
    __shared__ uint32_t s_b[kWaves];
    __shared__ int s_f[kWaves];
    dpp_max_step<0x111, 0xf>(p, bits);   // row_shr:1
    dpp_max_step<0x112, 0xf>(p, bits);   // row_shr:2
    dpp_max_step<0x114, 0xf>(p, bits);   // row_shr:4
    dpp_max_step<0x118, 0xf>(p, bits);   // row_shr:8
    dpp_max_step<0x142, 0xa>(p, bits);   // row_bcast:15 into rows 1 and 3
    dpp_max_step<0x143, 0xc>(p, bits);   // row_bcast:31 into rows 2 and 3
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 63) {
        s_p[wave] = p;
        s_b[wave] = bits;
        s_f[wave] = flag;
    }
    __syncthreads();
    p = s_p[0];
    bits = s_b[0];
    int any = s_f[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
        take_better(p, bits, s_p[w], s_b[w]);
        any |= s_f[w];
    }
    return any != 0;
}

__device__ __forceinline__ float bits_to_float(uint32_t b) { return __builtin_bit_cast(float, b); }

// Row geometry: elements [0, head) and [tail, V) are read one by one; the
// 16-byte aligned middle as nvec vectors.
struct RowGeom {
    int64_t head, nvec, tail;
};

__device__ __forceinline__ RowGeom row_geom(const unsigned char* row_ptr, int64_t vocab, int eb) {
    RowGeom g;
    const int64_t mis = (int64_t)((16 - ((uintptr_t)row_ptr & 15)) & 15) / eb;
    g.head = mis < vocab ? mis : vocab;
    g.nvec = (vocab - g.head) * eb / 16;
    g.tail = g.head + g.nvec * (16 / eb);
    return g;
}

// Split that owns column c.
__device__ __forceinline__ int owner_split(int64_t c, const RowGeom& g, int64_t chunk_cols,
                                           int splits) {
    if (c < g.head) return 0;
    const int64_t s = (uint32_t)(c - g.head) / (uint32_t)chunk_cols;   // both below 2^31
    return s < splits - 1 ? (int)s : splits - 1;
}

// Packed layout o_i = sum_{j<i} (max(K_j, 0) + 1), written by one workgroup:
// an exclusive scan of the row counts in chunks of kRowThreads requests.
__device__ void write_packed_offsets(int32_t num_requests, const int32_t* __restrict__ block_lens,
                                     int64_t* __restrict__ offsets) {
    __shared__ long long s_wave[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long carry = 0;
    for (int64_t c0 = 0; c0 < num_requests; c0 += kRowThreads) {
        const int64_t i = c0 + tid;
        const int32_t K = i < num_requests ? block_lens[i] : 0;
        const long long n = i < num_requests ? (long long)(K > 0 ? K : 0) + 1 : 0;
        long long incl = n;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        long long before = 0, chunk_total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const long long t = s_wave[w];
            before += (w < wave) ? t : 0;
            chunk_total += t;
        }
        __syncthreads();
        if (i < num_requests) offsets[i] = carry + before + incl - n;
        carry += chunk_total;
    }
}

// Row offsets of one workgroup's requests [first, first + count), count <= its
// 64 kBlockWaves threads, into s_off: row_offsets[i] when given, else the packed layout
// o_i = sum_{j<i} (max(K_j, 0) + 1).  For the packed layout the whole workgroup
// sums the row counts of the requests before `first`, then scans its own, so
// no request count is too large and nothing is written to global memory.
// Ends with a barrier.
template <int kBlockWaves>
__device__ __forceinline__ void block_offsets(int32_t num_requests,
                                              const int32_t* __restrict__ block_lens,
                                              const int64_t* __restrict__ row_offsets,
                                              int64_t first, int count, int64_t* s_off) {
    __shared__ long long s_before[kBlockWaves];
    __shared__ long long s_mine[kBlockWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (row_offsets) {
        if (tid < count) s_off[tid] = row_offsets[first + tid];
        __syncthreads();
        return;
    }
    long long before = 0;
    for (int64_t j = tid; j < first; j += 64 * kBlockWaves) {
        const int32_t K = block_lens[j];
        before += (long long)(K > 0 ? K : 0) + 1;
    }
    const int32_t Km = tid < count ? block_lens[first + tid] : 0;
    const long long mine = tid < count ? (long long)(Km > 0 ? Km : 0) + 1 : 0;
    long long incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const long long t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
        before += __shfl_xor(before, off, 64);
    }
    if (lane == 63) s_mine[wave] = incl;
    if (lane == 0) s_before[wave] = before;
    __syncthreads();
    long long base = 0, earlier = 0;
#pragma unroll
    for (int w = 0; w < kBlockWaves; ++w) {
        base += s_before[w];
        earlier += (w < wave) ? s_mine[w] : 0;
    }
    if (tid < count) s_off[tid] = base + earlier + incl - mine;
    __syncthreads();
}

// Where one lane's share of a tile lies: 16-byte vectors [v0, v1) of the row's
// aligned middle, in ngroups groups of kGroupVecs vectors (the last one padded
// with copies, see load_group).
struct TileSpan {
    const u32x4* vec;
    int32_t v0, v1, nv, ngroups;  // vector counts: a row has fewer than 2^28 vectors
    int tid;
};

// Group g of the lane's share.  In the tile's last group a vector past the
// tile's end is read as a copy of the tile's last vector: a copy adds no new
// value, and its column (past the end) is greater than the original's, so the
// tile's first greatest element is unchanged.  Every group is then whole, and
// the last one is loaded in the pipeline like the others.
__device__ __forceinline__ void load_group(const TileSpan& t, u32x4 (&r)[kUnroll], int32_t g) {
    const int32_t i0 = t.v0 + g * kGroupVecs + t.tid;
    const unsigned char* base = (const unsigned char*)t.vec;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        // a 32-bit byte offset from the row (a row is under 2^32 bytes)
        const uint32_t off = (uint32_t)min(i0 + u * kRowThreads, t.v1 - 1) << 4;
        r[u] = __builtin_nontemporal_load((const u32x4*)(base + off));
    }
}

// The lane's first element holding `key` in a saved group, narrowed level by
// level in column order: the first vector whose greatest key is `key`, then
// that vector's first such dword, then (bf16) the half.  Returns the element's
// index within the group's vectors' elements and its binary32 bits.
template <int EB, int kMode>
__device__ __forceinline__ void find_first(const u32x4 (&saved)[kUnroll], int32_t key, int& su,
                                           int& e, uint32_t& bits) {
    su = 0;
    u32x4 sv = saved[0];
    bool hit = false;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int32_t mk = max(max(dword_max_key<EB, kMode>(saved[u].x),
                                   dword_max_key<EB, kMode>(saved[u].y)),
                               max(dword_max_key<EB, kMode>(saved[u].z),
                                   dword_max_key<EB, kMode>(saved[u].w)));
        const bool take = !hit && mk == key;
        su = take ? u : su;
        sv = take ? saved[u] : sv;
        hit = hit || take;
    }
    int d = 3;
    uint32_t w = sv.w;
#pragma unroll
    for (int j = 2; j >= 0; --j) {                 // the first dword holding key wins
        const bool take = dword_max_key<EB, kMode>(sv[j]) == key;
        d = take ? j : d;
        w = take ? sv[j] : w;
    }
    if constexpr (EB == 2) {
        const bool low = key_of<2, kMode>(w & 0xffffu) == key;
        e = 2 * d + (low ? 0 : 1);
        bits = (low ? (w & 0xffffu) : (w >> 16)) << 16;
    } else {
        e = d;
        bits = w;
    }
}

// Key modes of rank_share beyond the three key kinds: choose raw or
// sign-magnitude keys from the first whole group (see tile_best).
constexpr int kKeysChoose = 3;

// One lane's ranking of its share of a tile: the greatest key, the first
// element holding it (as a packed (key, column)) and that element's binary32
// bits.  `mode` is uniform across the wavefront; the loop is shared and each
// group's ranking branches on it.  With kKeysChoose the wavefront ranks its
// first whole group with raw keys and keeps them if that group holds a number
// in [1, +inf] in any lane, else switches to sign-magnitude keys (ranking the
// group again from its registers).  Except with NaN keys, `umax` takes the
// greatest pattern read as unsigned (per 16-bit half for bf16).
template <int EB, typename Hook>
__device__ __forceinline__ void rank_share(const TileSpan& t, int mode, int64_t col_base,
                                           unsigned long long& packed, uint32_t& bits,
                                           uint32_t& umax, Hook&& after_first_loads) {
    constexpr int kEpv = 16 / EB;
    int32_t best_key = KeyTraits<4>::kNone;
    int32_t best_group = -1;
    u32x4 saved[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) saved[u] = (u32x4)(0u);

    auto rank_group = [&](const u32x4 (&r)[kUnroll], int32_t g) {
        int32_t gk;
        if (mode == kKeysNan) {
            gk = group_max_key<EB, kKeysNan>(r, umax);
        } else if (mode == kKeysExact) {
            gk = group_max_key<EB, kKeysExact>(r, umax);
        } else {
            gk = group_max_key<EB, kKeysRaw>(r, umax);
            if (mode == kKeysChoose) {
                const int raw_ok =
                    __ballot(gk >= kRawExactFrom && gk <= KeyTraits<EB>::kInf) != 0ull;
                mode = __builtin_amdgcn_readfirstlane(raw_ok) ? kKeysRaw : kKeysExact;
                if (mode == kKeysExact) gk = group_max_key<EB, kKeysExact>(r, umax);
            }
        }
        const bool better = gk > best_key;
        best_key = better ? gk : best_key;
        best_group = better ? g : best_group;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) saved[u] = better ? r[u] : saved[u];
    };
    // Whole groups through two register buffers in ping-pong: a group's four
    // loads are issued before the previous group is ranked, so each wavefront
    // keeps eight 16-byte loads per lane in flight while it computes.  The
    // first two groups are issued before anything else that reads memory (the
    // hook), so a tile's first data is requested as soon as it starts.  The
    // scheduling barriers keep the compiler from moving ranking work (and its
    // waits) ahead of the loads.
    if (t.ngroups > 0) {
        u32x4 ra[kUnroll], rb[kUnroll];
        load_group(t, ra, 0);
        __builtin_amdgcn_sched_barrier(0);
        after_first_loads();
        __builtin_amdgcn_sched_barrier(0);
        int32_t g = 0;
        for (; g + 2 < t.ngroups; g += 2) {
            load_group(t, rb, g + 1);
            __builtin_amdgcn_sched_barrier(0);
            rank_group(ra, g);
            load_group(t, ra, g + 2);
            __builtin_amdgcn_sched_barrier(0);
            rank_group(rb, g + 1);
        }
        if (g + 1 < t.ngroups) {
            load_group(t, rb, g + 1);
            __builtin_amdgcn_sched_barrier(0);
            rank_group(ra, g);
            rank_group(rb, g + 1);
        } else {
            rank_group(ra, g);
        }
    } else {
        after_first_loads();
    }
    if (mode == kKeysChoose) mode = kKeysExact;      // no group: sign-magnitude keys

    packed = pack_kc(KeyTraits<4>::kNone, 0x7fffffff);
    bits = 0;
    if (best_group >= 0) {
        int su, e;
        if (mode == kKeysRaw) find_first<EB, kKeysRaw>(saved, best_key, su, e, bits);
        else if (mode == kKeysExact)
            find_first<EB, kKeysExact>(saved, best_key, su, e, bits);
        else find_first<EB, kKeysNan>(saved, best_key, su, e, bits);
        const int64_t vi = (int64_t)t.v0 + best_group * kGroupVecs + su * kRowThreads + t.tid;
        packed = pack_kc(best_key, col_base + vi * kEpv + e);
    }
}

// One lane's best (key, column) and bits over its share of a tile: the
// tile's 16-byte vectors [split * chunk_vecs, ...) of the row's aligned middle,
// plus the row's unaligned head (split 0) and tail (last split) elements.
//
// kNanPass = false, the first pass.  Each wavefront ranks its first group with
// raw keys; if that group holds a number in [1, +inf] in any lane, raw keys
// rank the wavefront's whole share (every key that can win is then exact),
// else sign-magnitude keys do.  So the tile's greatest key is exact unless the
// tile holds a NaN, and `nan_seen` tells whether the lane's share holds one
// that the greatest key does not show (one with the sign bit set, or any NaN
// among the head and tail elements).
// kNanPass = true: NaN keys, for a tile known to hold a NaN.
template <int EB, bool kNanPass, typename Hook>
__device__ __forceinline__ void tile_best(const unsigned char* row_ptr, const RowGeom& geom,
                                          int64_t vocab, int64_t col_offset, int split,
                                          int splits, int64_t chunk_vecs, int tid,
                                          unsigned long long& packed, uint32_t& bits,
                                          bool& nan_seen, Hook&& after_first_loads) {
    constexpr int kScalarMode = kNanPass ? kKeysNan : kKeysExact;
    TileSpan t;
    t.vec = (const u32x4*)(row_ptr + geom.head * EB);
    t.v0 = (int32_t)(split * chunk_vecs);
    t.v1 = (int32_t)min(split * chunk_vecs + chunk_vecs, geom.nvec);
    t.nv = t.v1 > t.v0 ? t.v1 - t.v0 : 0;
    t.ngroups = (t.nv + kGroupVecs - 1) / kGroupVecs;
    t.tid = tid;
    const int64_t col_base = col_offset + geom.head;

    uint32_t umax = 0;
    if constexpr (kNanPass) {
        rank_share<EB>(t, kKeysNan, col_base, packed, bits, umax, after_first_loads);
    } else {
        rank_share<EB>(t, kKeysChoose, col_base, packed, bits, umax, after_first_loads);
        if constexpr (EB == 2)
            nan_seen = max(umax & 0xffffu, umax >> 16) > KeyTraits<2>::kNegInfPattern;
        else
            nan_seen = umax > KeyTraits<4>::kNegInfPattern;
    }

    // unaligned head and tail elements (at most 16 / EB - 1 of each)
    if (split == 0 && tid < geom.head) {
        int32_t k;
        uint32_t b;
        load_scalar<EB, kScalarMode>(row_ptr + (int64_t)tid * EB, k, b);
        take_better(packed, bits, pack_kc(k, col_offset + tid), b);
        if constexpr (!kNanPass) nan_seen = nan_seen || (b & 0x7fffffffu) > 0x7f800000u;
    }
    if (split == splits - 1 && tid < vocab - geom.tail) {
        const int64_t c = geom.tail + tid;
        int32_t k;
        uint32_t b;
        load_scalar<EB, kScalarMode>(row_ptr + c * EB, k, b);
        take_better(packed, bits, pack_kc(k, col_offset + c), b);
        if constexpr (!kNanPass) nan_seen = nan_seen || (b & 0x7fffffffu) > 0x7f800000u;
    }
}

// ------------------------------------- outputs read within the same launch
//
// In the single-launch form the last tile reads what the others wrote, from
// other XCDs.  These write and read past the XCD's own caches (agent-scope
// relaxed atomics: sc1), 64 bits at a time, so that neither side writes back or
// invalidates an L2; with kShared unset they are plain accesses.
template <bool kShared>
__device__ __forceinline__ void put(TilePartial* to, const TilePartial& t) {
    if constexpr (kShared) {
        unsigned long long* const w = (unsigned long long*)to;
        __hip_atomic_store(w, t.packed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(w + 1, ((unsigned long long)t.draft_bits << 32) | t.bits,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        *to = t;
    }
}
template <bool kShared>
__device__ __forceinline__ void put(RowRecord* to, const RowRecord& r) {
    if constexpr (kShared)
        __hip_atomic_store((unsigned long long*)to, __builtin_bit_cast(unsigned long long, r),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *to = r;
}
template <bool kShared>
__device__ __forceinline__ TilePartial get(const TilePartial* from) {
    if constexpr (kShared) {
        unsigned long long* const w = (unsigned long long*)from;
        TilePartial t;
        t.packed = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long v =
            __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        t.bits = (uint32_t)v;
        t.draft_bits = (uint32_t)(v >> 32);
        return t;
    } else {
        return *from;
    }
}
template <bool kShared>
__device__ __forceinline__ RowRecord get(const RowRecord* from) {
    if constexpr (kShared)
        return __builtin_bit_cast(
            RowRecord, __hip_atomic_load((unsigned long long*)from, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT));
    else
        return *from;
}

// ----------------------------------------------------------- stage 1 kernel

// One tile of the row pass, the body of the row kernels.  `logits` rows hold
// columns [col_offset, col_offset + vocab) of the full vocabulary (col_offset
// = 0 and vocab = V unless the rows are one tensor-parallel shard); columns are
// reported globally.  With `partials` set the tile writes a partial (split
// rows, or one shard of each row); otherwise the row is one tile and writes its
// record.  `pre` runs once, right after the tile's first loads are issued (for
// the caller's own loads).  Thread 0 writes; every thread returns.
template <int EB, bool kShared, typename Pre>
__device__ __forceinline__ void row_tile(
    const unsigned char* __restrict__ logits, int64_t vocab, int64_t col_offset, int splits,
    int64_t chunk_vecs, const int32_t* __restrict__ draft_tokens,
    TilePartial* __restrict__ partials, RowRecord* __restrict__ records,
    int32_t* __restrict__ out_argmax, Pre&& pre) {
    constexpr int kEpv = 16 / EB;
    const int tid = threadIdx.x;
    const int64_t row = blockIdx.x / splits;
    const int split = (int)(blockIdx.x - row * splits);
    const unsigned char* row_ptr = logits + row * vocab * EB;
    const RowGeom geom = row_geom(row_ptr, vocab, EB);
    const int64_t chunk_cols = chunk_vecs * kEpv;

    // The row's draft token x (uniform) and, in the tile that owns its column,
    // the pattern of z(x).  Both are read after the tile's first loads are
    // issued.  Every lane reads the pattern from one uniform address (the row's
    // first element when the tile does not own x): with no branch around the
    // load nothing waits for it before the ranking, so it overlaps the stream.
    int32_t x = 0;
    bool x_here = false, owns_x = false;
    uint32_t draft_raw = 0;
    auto after_first_loads = [&]() {
        x = draft_tokens[row];
        const int64_t x_local = (int64_t)x - col_offset;
        x_here = x_local >= 0 && x_local < vocab;
        owns_x = x_here && owner_split(x_local, geom, chunk_cols, splits) == split;
        const unsigned char* p = row_ptr + (owns_x ? x_local * EB : 0);
        if constexpr (EB == 2) draft_raw = *(const unsigned short*)p;
        else draft_raw = *(const uint32_t*)p;
        pre();
    };

    // ---- rank the tile (first pass); if it holds a NaN, rank it again to find
    // its first NaN.
    unsigned long long packed;
    uint32_t bits;
    bool nan_seen = false;
    tile_best<EB, false>(row_ptr, geom, vocab, col_offset, split, splits, chunk_vecs, tid, packed,
                         bits, nan_seen, after_first_loads);
    // Every thread learns the tile's best pair and whether any wavefront saw a
    // NaN, so every thread takes the same decision without a second barrier.
    const bool wave_nan = __ballot(nan_seen) != 0ull;
    const bool any_nan = block_reduce(packed, bits, wave_nan);
    if (any_nan || packed_key(packed) > KeyTraits<EB>::kInf) {
        __syncthreads();                 // every thread has read the first reduction
        tile_best<EB, true>(row_ptr, geom, vocab, col_offset, split, splits, chunk_vecs, tid,
                            packed, bits, nan_seen, [] {});
        block_reduce(packed, bits, false);
    }
    if (tid != 0) return;
    const uint32_t draft_bits = owns_x ? (EB == 2 ? draft_raw << 16 : draft_raw) : 0u;

    if (partials != nullptr) {           // combined by the scan
        TilePartial tp;
        tp.packed = packed;
        tp.bits = bits;
        tp.draft_bits = draft_bits;      // meaningful in the owning tile only
        put<kShared>(partials + blockIdx.x, tp);
        return;
    }

    // ---- one tile per row: the row record (one binary32 subtraction)
    const int32_t y = packed_col(packed);
    RowRecord rec;
    if (x_here) {                        // the whole vocabulary: x_here = x in [0, V)
        rec.regret = bits_to_float(bits) - bits_to_float(draft_bits);
        rec.y_flags = (uint32_t)y | ((x != y) ? kMismatchBit : 0u);
    } else {
        rec.regret = __builtin_huge_valf();
        rec.y_flags = (uint32_t)y | kMismatchBit | kBadDraftBit;
    }
    put<kShared>(records + row, rec);
    if (out_argmax) out_argmax[row] = y;
}

// The row pass as its own kernel, followed by the scan kernel.  Block 0 also
// writes the packed row offsets of the requests when `packed_offsets` is set,
// after its first loads are issued: a test of that argument ahead of the row
// pass would make every tile wait for its arguments twice before its first
// load.  Five wavefronts per SIMD: the two load buffers and the clamped offsets
// of the last group fit in 96 VGPRs with no spill (at six, 80 VGPRs, an
// earlier form spilled to scratch and ran 25% slower).
template <int EB>
__global__ __launch_bounds__(kRowThreads) __attribute__((amdgpu_waves_per_eu(5))) void asd_row_kernel(
    const unsigned char* __restrict__ logits, int64_t vocab, int64_t col_offset, int splits,
    int64_t chunk_vecs, const int32_t* __restrict__ draft_tokens,
    TilePartial* __restrict__ partials, RowRecord* __restrict__ records,
    int32_t* __restrict__ out_argmax, int32_t num_requests,
    const int32_t* __restrict__ block_lens, int64_t* __restrict__ packed_offsets) {
    row_tile<EB, false>(logits, vocab, col_offset, splits, chunk_vecs, draft_tokens, partials,
                        records, out_argmax, [&] {
                            if (blockIdx.x == 0 && packed_offsets != nullptr)
                                write_packed_offsets(num_requests, block_lens, packed_offsets);
                        });
}

// ----------------------------------------------------------- stage 2 kernel

struct ScanArgs {
    int32_t num_requests;
    int32_t request_blocks;      // workgroups that scan requests; the rest write argmax rows
    int64_t total_rows;
    int64_t vocab;
    int elem_bytes;
    int splits;
    int64_t chunk_vecs;
    const unsigned char* logits; // row addresses only (alignment -> split ownership)
    const int32_t* draft_tokens;
    const int32_t* block_lens;
    const int64_t* offsets;
    const float* tau;
    const int32_t* exc_cap;
    float2* budget;
    const RowRecord* records;    // splits == 1 and no shards
    const TilePartial* partials; // split rows: [row][split]; shards: [shard][row]
    int64_t shard_vocab;         // > 0: partials come from vocabulary shards of this width
    const unsigned long long* row_best;   // LM-head pass: each row's greatest (key, column)
    const uint32_t* row_draft_bits;       // LM-head pass: each row's draft logit
    int32_t* commit_tokens;               // commit in the same pass, or nullptr
    int64_t commit_capacity;
    int64_t* commit_seq_len;
    int32_t* commit_done;
    int raw_gate;                         // gate on r <= g (q read as 1)
    int32_t* out_accept_len;
    int32_t* out_next_token;
    float* out_regret;
    int32_t* out_argmax;
};

// Greatest (key, column) of a row's split partials and the gathered draft logit.
template <bool kShared>
__device__ __forceinline__ void combine_row(const ScanArgs& A, int64_t row, int32_t x,
                                            unsigned long long& packed, uint32_t& bits,
                                            uint32_t& draft_bits) {
    const bool x_valid = x >= 0 && (int64_t)x < A.vocab;
    if (A.row_best) {                    // LM-head pass: value bits from the exact key
        packed = A.row_best[row];
        const int32_t key = packed_key(packed);
        bits = key >= 0 ? (uint32_t)key : (0x80000000u | (uint32_t)(-(int64_t)key));
        draft_bits = x_valid ? A.row_draft_bits[row] : 0u;
        return;
    }
    const TilePartial* parts;
    int64_t stride;
    int owner = -1;
    if (A.shard_vocab > 0) {             // shard k holds columns [k W, (k + 1) W)
        parts = A.partials + row;
        stride = A.total_rows;
        if (x_valid) owner = (int)min((int64_t)x / A.shard_vocab, (int64_t)A.splits - 1);
    } else {                             // tiles of one row
        parts = A.partials + row * A.splits;
        stride = 1;
        const unsigned char* row_ptr = A.logits + row * A.vocab * A.elem_bytes;
        const RowGeom geom = row_geom(row_ptr, A.vocab, A.elem_bytes);
        if (x_valid) owner = owner_split(x, geom, A.chunk_vecs * (16 / A.elem_bytes), A.splits);
    }
    packed = 0;
    bits = 0;
    draft_bits = 0;
    // Partials are read eight at a time so that their loads are in flight together.
    for (int s0 = 0; s0 < A.splits; s0 += 8) {
        TilePartial tp[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (s0 + j < A.splits) tp[j] = get<kShared>(parts + (s0 + j) * stride);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (s0 + j < A.splits) {
                take_better(packed, bits, tp[j].packed, tp[j].bits);
                if (s0 + j == owner) draft_bits = tp[j].draft_bits;
            }
        }
    }
}

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// Algorithm 1 for request i, whose rows start at o, by one wavefront: lanes
// are block positions.  Each lane forms its row's record (or combines the
// row's partials); the wavefront walks the mismatches in position order.
// Wave-uniform: every lane of the wavefront calls it with the same i and o.
// The per-request inputs of Algorithm 1 (block length, ledger, gate, cap and
// committed length), loaded together so that their loads are in flight at
// once, ahead of the rows.
struct RequestIn {
    int32_t K_given;
    int32_t M;
    float2 ledger;
    float g;
    int64_t L;
};

__device__ __forceinline__ RequestIn load_request(const ScanArgs& A, int64_t i) {
    RequestIn q;
    q.K_given = A.block_lens[i];
    q.ledger = A.budget[i];
    q.g = A.tau[i];
    q.M = A.exc_cap[i];
    q.L = A.commit_tokens ? A.commit_seq_len[i] : 0;
    return q;
}

template <bool kShared>
__device__ __forceinline__ void scan_request(const ScanArgs& A, int64_t i, int64_t o,
                                             const RequestIn& q) {
    const int lane = threadIdx.x & 63;
    const int32_t K_given = q.K_given;
    const int32_t K = K_given > 0 ? K_given : 0;      // a negative K is read as 0
    const int64_t L = q.L;
    if (K_given < 0 && lane == 0) atomicOr(&asd_error_word, kErrNegativeK);
    if (!(o >= 0 && o + (int64_t)K < A.total_rows)) {
        if (lane == 0) {
            A.out_accept_len[i] = 0;
            A.out_next_token[i] = -1;
            if (A.commit_tokens && A.commit_done) A.commit_done[i] = 0;
            atomicOr(&asd_error_word, kErrRows);
        }
        return;
    }
    const float B = q.ledger.x;
    const float s = q.ledger.y;
    const float g = q.g;
    const int32_t M = q.M;
    const bool strict = (B == 0.0f);   // Algorithm 1: B = 0 -> exact greedy verification

    int32_t a = 0, N = 0, next = -1;
    float C = 0.0f;
    bool done = false;
    for (int64_t c0 = 0; c0 <= K; c0 += 64) {
        const int64_t p = c0 + lane;                  // 0-based position; p == K: bonus row
        const bool have = p <= K;
        const bool is_draft = p < K;
        uint32_t y = 0;
        bool mism = false, bad = false;
        float r = 0.0f;
        if (have) {
            const int64_t row = o + p;
            if (A.records != nullptr) {
                const RowRecord rec = get<kShared>(A.records + row);
                y = rec.y_flags & kArgmaxMask;
                mism = (rec.y_flags & kMismatchBit) != 0u;
                bad = (rec.y_flags & kBadDraftBit) != 0u;
                r = rec.regret;
            } else {
                const int32_t x = A.draft_tokens[row];
                unsigned long long packed;
                uint32_t bits, draft_bits;
                combine_row<kShared>(A, row, x, packed, bits, draft_bits);
                y = (uint32_t)packed_col(packed);
                bad = !(x >= 0 && (int64_t)x < A.vocab);
                mism = bad || (uint32_t)x != y;
                r = bad ? __builtin_huge_valf() : bits_to_float(bits) - bits_to_float(draft_bits);
            }
            if (A.out_regret) A.out_regret[row] = is_draft ? r : 0.0f;
        }
        if (done) continue;

        // Mismatches among this chunk's draft positions, and those that pass
        // the local gate r <= g q (q = K - p, i.e. K - i + 1 for i = p + 1;
        // q = 1 for the raw-gate variant).
        const int32_t q = A.raw_gate ? 1 : K - (int32_t)p;
        const bool gate = (double)r <= (double)g * (double)q;
        const unsigned long long mism_mask = __ballot(is_draft && mism);
        const unsigned long long ok_mask = __ballot(is_draft && mism && !bad && gate);
        int stop = -1;
        if (strict) {
            if (mism_mask) stop = __builtin_ctzll(mism_mask);
        } else {
            for (unsigned long long m = mism_mask; m != 0ull; m &= m - 1ull) {
                const int j = __builtin_ctzll(m);
                const float rj = __builtin_bit_cast(float, lane_u32(__builtin_bit_cast(uint32_t, r), j));
                const float C_new = C + rj;
                const int32_t N_new = N + 1;
                const float s_new = s + C_new;
                if (!(((ok_mask >> j) & 1ull) && s_new <= B && N_new <= M)) {
                    stop = j;
                    break;
                }
                C = C_new;
                N = N_new;
            }
        }
        if (stop >= 0) {                              // first infeasible position
            a = (int32_t)(c0 + stop);
            next = (int32_t)lane_u32(y, stop);         // recovery token y*_{a+1}
            done = true;
        } else if (K - c0 < 64) {                     // the bonus row is in this chunk
            a = K;
            next = (int32_t)lane_u32(y, (int)(K - c0));
            done = true;
        }
    }
    if (lane == 0) {
        if (N > 0) A.budget[i].y = s + C;             // s' = s + C_a
        A.out_accept_len[i] = a;
        A.out_next_token[i] = next;
    }
    if (A.commit_tokens) {
        // The commit (Sec. 3.3): x_1..x_a then y*_{a+1} at the request's
        // committed length, when they fit below capacity.
        const bool ok = next >= 0 && L >= 0 && L + (int64_t)a + 1 <= A.commit_capacity;
        if (ok) {
            int32_t* dst = A.commit_tokens + i * A.commit_capacity + L;
            for (int64_t j = lane; j <= a; j += 64) dst[j] = j < a ? A.draft_tokens[o + j] : next;
        }
        if (lane == 0) {
            if (ok) A.commit_seq_len[i] = L + (int64_t)a + 1;
            if (A.commit_done) A.commit_done[i] = ok ? a + 1 : 0;
            if (!ok) atomicOr(&asd_error_word, kErrCommit);
        }
    }
}

__global__ __launch_bounds__(kScanThreads) void asd_scan_kernel(const ScanArgs A) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    if ((int32_t)blockIdx.x >= A.request_blocks) {
        // Argmax of every row when rows were split (one lane per row).
        const int64_t row = (int64_t)(blockIdx.x - A.request_blocks) * kScanThreads + tid;
        if (row < A.total_rows) {
            unsigned long long packed;
            uint32_t bits, draft_bits;
            combine_row<false>(A, row, -1, packed, bits, draft_bits);
            A.out_argmax[row] = packed_col(packed);
        }
        return;
    }

    const int64_t i = (int64_t)blockIdx.x * (kScanThreads / 64) + wave;   // wave-uniform
    if (i >= A.num_requests) return;
    const RequestIn q = load_request(A, i);
    int64_t o;
    if (A.offsets) {
        o = A.offsets[i];
    } else {
        // Packed layout, few requests: this wavefront sums the row counts of
        // the requests before it.
        long long part = 0;
#pragma unroll 4
        for (int64_t j = lane; j < i; j += 64) {
            const int32_t Kj = A.block_lens[j];
            part += (long long)(Kj > 0 ? Kj : 0) + 1;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) part += __shfl_xor(part, off, 64);
        o = part;
    }
    scan_request<false>(A, i, o, q);
}

// ---------------------------------------------- single-launch verification
//
// For plans with few tiles and few requests the call is bound by latency, and
// the second launch of the scan is a large share of it.  Here the row pass and
// the scan run in one launch: every tile counts itself done on a counter once
// its record or partial is written, and the one tile that finds itself last
// runs Algorithm 1 for every request, one wavefront per request, writes the
// argmax of split rows and resets the counter to zero for the next call.  No
// tile waits for another.  The records and partials pass by the L2s (put and
// get above), so the counter takes no release and no acquire, each of which
// costs a pass over an L2: 9 rows of 32,000 f32 7.7 us on the GPU, 8.2 with them,
// and 270 tiles 11.3 for 14.3.  The counter must be zero when the call starts: it
// lives in a header of the library's workspaces that is zeroed when they are
// allocated, and every call leaves it at zero.
//
// In the language's terms the relaxed counter orders nothing.  The hand-over
// relies on gfx950: an agent-scope store (sc1) is written through to the memory
// that all XCDs share and leaves vmcnt when it has arrived there, so a writer
// that waits for vmcnt(0) before it counts has published its output; an
// agent-scope load (sc1) is not served from an L2's older copy; and the reader
// issues its loads after the barrier that follows the counter's return.  These are
// the steps by which the compiler itself makes an agent-scope release and acquire,
// without the write-back and the invalidation, which only plain accesses need;
// nothing but put's outputs passes between workgroups here.
// Small plans have less than a tile per CU, so the kernel takes the registers
// it needs (no occupancy bound).
static_assert(kSingleLaunchMaxRequests <= 2 * kWaves, "two requests per wavefront at most");

template <int EB>
__global__ __launch_bounds__(kRowThreads) void asd_row_scan_kernel(const unsigned char* __restrict__ logits, int64_t vocab, int splits,
                    int64_t chunk_vecs, TilePartial* __restrict__ partials,
                    RowRecord* __restrict__ records, unsigned* __restrict__ counter,
                    const ScanArgs A) {
    // Every tile loads the requests' inputs and row offsets during its row pass,
    // right after its first loads are issued (the few requests of a
    // single-launch plan: wavefront w takes requests w and w + 4), so that the
    // last tile's scan waits only for the rows.
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    RequestIn q[2];
    int64_t o[2];
    auto preload = [&]() {
        const int n = A.num_requests;            // <= kSingleLaunchMaxRequests <= 64
        const int32_t Kl = lane < n ? A.block_lens[lane] : 0;
        long long incl = lane < n ? (long long)(Kl > 0 ? Kl : 0) + 1 : 0;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        const long long excl = incl - (lane < n ? (long long)(Kl > 0 ? Kl : 0) + 1 : 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = wave + 4 * j;
            if (k < n) {
                q[j] = load_request(A, k);
                o[j] = A.offsets ? A.offsets[k] : (int64_t)__shfl(excl, k, 64);
            }
        }
    };
    row_tile<EB, true>(logits, vocab, 0, splits, chunk_vecs, A.draft_tokens, partials, records,
                       splits == 1 ? A.out_argmax : nullptr, preload);
    __shared__ int s_last;
    if (threadIdx.x == 0) {
        // This thread's output has reached the memory that every XCD reads.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const unsigned prev =
            __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = prev == gridDim.x - 1;
        asm volatile("" ::: "memory");    // no tile's output is read ahead of this
    }
    __syncthreads();
    if (!s_last) return;

#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (wave + 4 * j < A.num_requests) scan_request<true>(A, wave + 4 * j, o[j], q[j]);
    if (splits > 1 && A.out_argmax) {
        for (int64_t row = threadIdx.x; row < A.total_rows; row += kRowThreads) {
            unsigned long long packed;
            uint32_t bits, draft_bits;
            combine_row<true>(A, row, -1, packed, bits, draft_bits);
            A.out_argmax[row] = packed_col(packed);
        }
    }
    if (threadIdx.x == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Packed row offsets for the calls that have no row kernel before the scan.
__global__ __launch_bounds__(kRowThreads) void asd_offsets_kernel(
    int32_t num_requests, const int32_t* __restrict__ block_lens, int64_t* __restrict__ offsets) {
    write_packed_offsets(num_requests, block_lens, offsets);
}

ScanArgs scan_args(const CallArgs& a, int64_t rows, int64_t vocab, int elem_bytes) {
    ScanArgs A{};
    A.num_requests = a.num_requests;
    A.request_blocks = (int32_t)((a.num_requests + kScanThreads / 64 - 1) / (kScanThreads / 64));
    A.total_rows = rows;
    A.vocab = vocab;
    A.elem_bytes = elem_bytes;
    A.logits = (const unsigned char*)a.logits;
    A.draft_tokens = a.draft_tokens;
    A.block_lens = a.block_lens;
    A.offsets = a.row_offsets;
    A.tau = a.tau;
    A.exc_cap = a.exc_cap;
    A.budget = a.budget;
    A.out_accept_len = a.out_accept_len;
    A.out_next_token = a.out_next_token;
    A.out_regret = a.out_regret;
    A.out_argmax = a.out_argmax;
    A.commit_tokens = a.commit_tokens;
    A.commit_capacity = a.commit_capacity;
    A.commit_seq_len = a.commit_seq_len;
    A.commit_done = a.commit_done;
    A.raw_gate = a.raw_gate ? 1 : 0;
    return A;
}

hipError_t launch_scan(const ScanArgs& A, bool argmax_rows, hipStream_t stream) {
    const int64_t row_blocks =
        (argmax_rows && A.out_argmax) ? (A.total_rows + kScanThreads - 1) / kScanThreads : 0;
    asd_scan_kernel<<<(unsigned)(A.request_blocks + row_blocks), kScanThreads, 0, stream>>>(A);
    return hipGetLastError();
}

template <typename... Args>
hipError_t launch_row(int elem_bytes, dim3 grid, hipStream_t stream, Args... args) {
    if (elem_bytes == 2)
        asd_row_kernel<2><<<grid, kRowThreads, 0, stream>>>(args...);
    else
        asd_row_kernel<4><<<grid, kRowThreads, 0, stream>>>(args...);
    return hipGetLastError();
}

// --------------------------------------------- opportunity statistic (Eq. 4)

// Counts of Eq. 4 over one batch, one wavefront per request with lanes =
// draft positions.  The ballot of target-greedy drafts gives, for every
// position, the length of the run of greedy drafts that follows it (trailing
// ones of the mask above the position, carried across 64-position chunks from
// the block's end).  A mismatch at position i with r_i <= tau and a following
// run of at least p greedy drafts (which also gives i + p <= K) counts for
// (tau, p): with lanes = pairs, the wavefront walks the chunk's mismatches and
// every lane tests its pair against each, or, where there are fewer pairs than
// mismatches, it walks the pairs and every position is tested against each.
// Counts gather in registers (the first 64 pairs) and LDS, then in the caller's
// uint64 accumulators.
//
// A chain of memory round trips bounds it, so the pairs' thresholds are read
// with the block lengths.  Workgroups have 16 wavefronts because all of them add
// to the same few accumulators, one after another.  256 requests of 16 drafts,
// 35 pairs: 4.4 us a call; with four wavefronts, one ballot per pair and the
// thresholds read in the loop 7.8 us.  The shorter walk is for calls of few pairs
// and many mismatches: 256 requests of 64 drafts that all mismatch, one pair 4.4
// us, over the mismatches 8.3; of 256 drafts 5.9 and 22.8.
constexpr int kOppWaves = 16;
constexpr int kOppMostRequests = 64;     // of one workgroup

__global__ __launch_bounds__(64 * kOppWaves) void asd_opportunity_kernel(
    const int32_t* __restrict__ draft_tokens, const int32_t* __restrict__ row_argmax,
    const float* __restrict__ row_regret, int64_t vocab, int32_t num_requests,
    int64_t total_rows, const int32_t* __restrict__ block_lens,
    const int64_t* __restrict__ row_offsets, const float* __restrict__ taus, int32_t num_taus,
    const int32_t* __restrict__ ps, int32_t num_ps, unsigned long long* __restrict__ counts,
    unsigned long long* __restrict__ mismatches, int per_block) {
    __shared__ uint32_t s_counts[kMaxOpportunityPairs];
    __shared__ float s_tau[kMaxOpportunityPairs];      // of pair k
    __shared__ int32_t s_p[kMaxOpportunityPairs];
    __shared__ uint32_t s_mism;
    __shared__ int64_t s_off[kOppMostRequests];
    __shared__ int32_t s_len[kOppMostRequests];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int pairs = num_taus * num_ps;
    const int64_t first = (int64_t)blockIdx.x * per_block;
    const int count = (int)min((int64_t)per_block, (int64_t)num_requests - first);
    if (tid < count) s_len[tid] = block_lens[first + tid];
    for (int k = tid; k < pairs; k += 64 * kOppWaves) {
        s_tau[k] = taus[k / num_ps];
        s_p[k] = ps[k % num_ps];
        s_counts[k] = 0u;
    }
    if (tid == 0) s_mism = 0u;
    block_offsets<kOppWaves>(num_requests, block_lens, row_offsets, first, count, s_off);   // + barrier

    // The first 64 pairs, one per lane, and their counts stay in registers.
    const float t0 = lane < pairs ? s_tau[lane] : 0.0f;
    const int32_t need0 = lane < pairs ? s_p[lane] : 0;
    uint32_t n0 = 0;
    // How many of the mismatches w count for this lane's (t, need): over the
    // mismatches, or over the pairs of the first `here` lanes.
    auto walk = [](unsigned long long w, float r, int32_t run, float t, int32_t need) {
        uint32_t n = 0;
        for (; w != 0ull; w &= w - 1ull) {
            const int j = __builtin_ctzll(w);
            const float rj = __builtin_bit_cast(float, lane_u32(__builtin_bit_cast(uint32_t, r), j));
            const int32_t run_j = (int32_t)lane_u32((uint32_t)run, j);
            n += rj <= t && run_j >= need;
        }
        return n;
    };
    auto walk_shorter = [&](unsigned long long w, float r, int32_t run, float t, int32_t need,
                            int here) {
        if (here >= (int)__builtin_popcountll(w)) return walk(w, r, run, t, need);
        uint32_t n = 0;
        for (int j = 0; j < here; ++j) {
            const float tj = __builtin_bit_cast(float, lane_u32(__builtin_bit_cast(uint32_t, t), j));
            const int32_t need_j = (int32_t)lane_u32((uint32_t)need, j);
            const unsigned long long q = __ballot(r <= tj && run >= need_j) & w;
            n = lane == j ? (uint32_t)__builtin_popcountll(q) : n;
        }
        return n;
    };

    for (int kq = wave; kq < count; kq += kOppWaves) {            // wave-uniform
        const int32_t K = __builtin_amdgcn_readfirstlane(s_len[kq]);
        const int64_t o = s_off[kq];
        if (K >= 0 && o >= 0 && o + (int64_t)K < total_rows) {
            // Chunks from the block's end: `carry` = greedy run starting at the
            // first position after the chunk.
            int32_t carry = 0;
            uint32_t mism_total = 0;
            const int64_t nchunks = ((int64_t)K + 63) / 64;
            for (int64_t c = nchunks - 1; c >= 0; --c) {
                const int64_t p = c * 64 + lane;      // 0-based draft position
                const bool have = p < K;
                bool match = false;
                float r = 0.0f;
                if (have) {
                    const int32_t x = draft_tokens[o + p];
                    const int32_t y = row_argmax[o + p];
                    r = row_regret[o + p];
                    match = x >= 0 && (int64_t)x < vocab && x == y;
                }
                const unsigned long long m = __ballot(have && match);
                const int n_here = (int)min((int64_t)64, (int64_t)K - c * 64);
                // trailing ones of the mask above this lane, within the chunk
                const unsigned long long above = lane < 63 ? (m >> (lane + 1)) : 0ull;
                const int ones = (int)__builtin_ctzll(~above);   // < 64 - lane
                const int32_t run = lane + 1 + ones >= n_here ? n_here - 1 - lane + carry : ones;
                const unsigned long long mm = __ballot(have && !match);
                mism_total += (uint32_t)__builtin_popcountll(mm);
                if (mm) {
                    n0 += walk_shorter(mm, r, run, t0, need0, min(pairs, 64));
                    int k = 64 + lane;                // the other pairs: whole groups, the rest
                    for (; k - lane + 64 <= pairs; k += 64) {
                        const uint32_t n = walk(mm, r, run, s_tau[k], s_p[k]);
                        if (n != 0) atomicAdd(&s_counts[k], n);
                    }
                    if (k - lane < pairs) {
                        const bool pair = k < pairs;
                        const uint32_t n = walk_shorter(mm, r, run, pair ? s_tau[k] : 0.0f,
                                                        pair ? s_p[k] : 0, pairs - (k - lane));
                        if (pair && n != 0) atomicAdd(&s_counts[k], n);
                    }
                }
                // greedy run starting at this chunk's first position
                const int lead = m == ~0ull ? 64 : (int)__builtin_ctzll(~m);
                carry = lead >= n_here ? n_here + carry : lead;
            }
            if (lane == 0 && mism_total) atomicAdd(&s_mism, mism_total);
        }
    }
    if (lane < pairs && n0 != 0) atomicAdd(&s_counts[lane], n0);
    __syncthreads();
    for (int k = tid; k < pairs; k += 64 * kOppWaves)
        if (s_counts[k]) atomicAdd(counts + k, (unsigned long long)s_counts[k]);
    if (tid == 0 && s_mism) atomicAdd(mismatches, (unsigned long long)s_mism);
}

// --------------------------------------------------------- commit (Sec. 3.3)

// The commit after verification: request i appends its emitted tokens x_1..x_a
// and y*_{a+1} to its token buffer at its committed length and advances that
// length (the extent the target and draft caches keep) by a + 1.  Each
// workgroup takes `per_block` consecutive requests, one wavefront per request
// at a time, lanes writing consecutive tokens.
__global__ __launch_bounds__(kScanThreads) void asd_commit_kernel(
    const int32_t* __restrict__ draft_tokens, const int32_t* __restrict__ block_lens,
    const int64_t* __restrict__ row_offsets, int32_t num_requests, int64_t total_rows,
    const int32_t* __restrict__ accept_len, const int32_t* __restrict__ next_token,
    int32_t* __restrict__ tokens, int64_t capacity, int64_t* __restrict__ seq_len,
    int32_t* __restrict__ committed, int per_block) {
    __shared__ int64_t s_off[kScanThreads];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t first = (int64_t)blockIdx.x * per_block;
    const int count = (int)min((int64_t)per_block, (int64_t)num_requests - first);
    block_offsets<kScanThreads / 64>(num_requests, block_lens, row_offsets, first, count, s_off);
    for (int k = wave; k < count; k += kScanThreads / 64) {       // wave-uniform
        const int64_t i = first + k;
        const int32_t K_given = block_lens[i];
        const int32_t K = K_given > 0 ? K_given : 0;  // a negative K is read as 0
        const int64_t o = s_off[k];
        const int32_t a = accept_len[i];
        const int32_t next = next_token[i];
        const int64_t L = seq_len[i];
        const bool rows_ok = o >= 0 && o + (int64_t)K < total_rows;
        const bool ok = rows_ok && next >= 0 && L >= 0 && a >= 0 && a <= K &&
                        L + (int64_t)a + 1 <= capacity;
        if (ok) {
            int32_t* dst = tokens + i * capacity + L;
            for (int64_t j = lane; j <= a; j += 64) dst[j] = j < a ? draft_tokens[o + j] : next;
        }
        if (lane == 0) {
            if (ok) seq_len[i] = L + (int64_t)a + 1;
            if (committed) committed[i] = ok ? a + 1 : 0;
            const uint32_t err = (K_given < 0 ? kErrNegativeK : 0u) | (rows_ok ? 0u : kErrRows) |
                                 (rows_ok && next >= 0 && !ok ? kErrCommit : 0u);
            if (err) atomicOr(&asd_error_word, err);
        }
    }
}

// ------------------------------------------- LM-head-fused row pass (MFMA)
//
// z = H W^T for hidden states H [M, K] and output weights W [N, K] (both bf16,
// K-contiguous), in binary32 on v_mfma_f32_16x16x32_bf16, reduced at once to
// each row's greatest (key, column) and the draft token's logit: the M x N
// logits never reach memory.
//
// One workgroup of eight wavefronts, two per SIMD, per tile of 256 weight rows
// (vocabulary columns) x 32 kNr hidden-state rows.  The weights are the A
// operand and the hidden states the B operand, so that a lane's accumulators
// hold vocabulary columns of one hidden-state row and the ranking runs within
// lanes.  Wavefront w covers columns 64 (w % 4) .. + 64 and rows
// 16 kNr (w / 4) .. + 16 kNr as 4 x kNr MFMA tiles.  Operand layout (lane l,
// element e): row l % 16 of the operand's 16, k = 8 (l / 16) + e; accumulator v
// of lane l is column 4 (l / 16) + v, hidden-state row l % 16.
//
// K steps of 64 go through LDS stages of 128-B rows, three for the weights and
// two for the hidden states.  Global -> LDS copies are buffer loads that write
// LDS directly (no VGPR staging); rows past M or N read as zero from the buffer
// resource.  The 16-B chunk c of row r is stored at chunk c ^ lm_swz(r), which
// keeps both the copies and the fragment reads free of bank conflicts.  The
// weights miss L2 far more often than the hidden states, which every workgroup
// reads, so their copies get two K steps to land: with two stages each, making
// every weight copy an L2 hit took 544 rows (d = 5,120) from 781 to 575 us, every
// hidden-state copy to 783.  Three stages, same box: 544 rows 802 -> 690 us; 4,352
// rows 4,753 -> 4,530; 2,816 rows of 129,280 columns, d = 7,168, 3,659 -> 3,472.
// (Touching the weights ahead, one load per line, was slower: 904 us and up.)
//
// Software pipeline of one wavefront: the fragments of the next k-slice of 32
// are read while the current slice's MFMAs issue.  The barrier that publishes
// the next stage sits kJ0 row groups into the second slice's MFMAs, which cover
// the last reads of the current stage; the next stage's first reads and the
// copies into the freed stage overlap the rest.
//
// What bounds large calls is the chip's power.  4,352 rows, 151,936 columns, d =
// 5,120, Gaussian data: 4.46-4.73 ms (1,430-1,520 TFLOP/s, by box) at 1.4-1.8 GHz
// with the matrix cores 81-84% busy; on data of ones the kernel clocks 2.4 GHz.  So it is
// built to spend little energy per flop: 16x16x32 MFMAs, which move half the
// accumulator bytes of 32x32x16 (registers-only probe 1,955 against 1,725
// TFLOP/s; this kernel's 32x32x16 predecessor took 5.08 ms on the same box),
// operands repeated from one MFMA to the next, and an epilogue within lanes
// (0.085 ms of the call; the predecessor's went through LDS, 0.15-0.2 ms).
// With every copy an L2 hit it would take 4.2 ms, with no copies 3.7 ms.
constexpr int kLmCols = 256;             // weight rows of a tile
constexpr int kLmK = 64;
constexpr int kLmThreads = 512;
// Up to this many row tiles read a weight tile, at about the same time: its
// copies are non-temporal, as in the stream kernel below.  255 rows, d = 5,120:
// 444 us cached, 386 us so; 144 rows of 128,256 columns, d = 7,168: 346 and 319;
// two row tiles, 408 rows of 129,280 columns, d = 7,168: 676 and 630; 272 rows,
// d = 5,120: 470 and 457.  With three, which miss each other's copies more often,
// it loses: 544 rows 692 and 716.
constexpr int kLmOnceMaxRowTiles = 2;
static_assert(kLmOnceMaxRowTiles <= kLmheadFewRowTiles, "these take the smaller groups");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
#define ASD_LDS __attribute__((address_space(3)))

constexpr int kLmStreamMaxRows = 128;    // fewer rows stream the weights
// Whole tiles against even shares, over 1 to 128 rows and 1,000 to 151,936
// columns: 5-7% faster at d = 128 to 1,024 (64 rows of 16,384 columns, d = 256,
// 11.7 us for 15.5; 33 rows of 40,000, d = 512, 19.9 for 22.8), level from 1,536
// on, where single calls of a part-full round lose up to 16% (d = 3,072).
constexpr int kLmStreamShortK = 1024;
constexpr int kWaitLds = 0xc07f;         // s_waitcnt lgkmcnt(0)
constexpr int kRsrcWord3 = 0x00020000;   // raw buffer, 32-bit data format

// A 16-byte LDS read serves 16 lanes at a time: lanes 0-3, 12-15 and 20-27 of
// each half wavefront, then the others.  Fragment reads put row l % 16 and
// chunk l / 16 on lane l, two rows to the 256 B of all banks, so the rows of
// one parity in such a group need distinct chunks: this gives them.
__device__ __forceinline__ int lm_swz(int r) { return (r >> 1) & 7; }

// Global -> LDS copies are written in asm: they fill LDS and no registers, and
// the compiler, which cannot tell a ring's stages apart, would wait for all of
// them before any fragment read.  The wait states before a copy cover a resource
// or LDS address that has just been written.  m0 is reserved: the compiler keeps
// nothing in it and sets it before each use of its own (there is none here), so
// it is not among the clobbers, where it would only draw a warning.
template <bool kNonTemporal>
__device__ __forceinline__ void lm_lds_copy(u32x4 rsrc, int voff, int k0b, uint32_t lds) {
    if constexpr (kNonTemporal)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                     :
                     : "s"(lds), "v"(voff), "s"(rsrc), "s"(k0b)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :
                     : "s"(lds), "v"(voff), "s"(rsrc), "s"(k0b)
                     : "memory");
}

__device__ __forceinline__ void lm_lds_copy_dword(u32x4 rsrc, int voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rsrc)
                 : "memory");
}

template <int kOutstanding>
__device__ __forceinline__ void lm_stage_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kOutstanding) : "memory");
}

// Waits for the oldest stage with `later` whole stages (at most kMost) of kPer
// copies per wavefront behind it.
template <int kMost, int kPer>
__device__ __forceinline__ void lm_stage_wait(int later) {
    if constexpr (kMost == 0) {
        lm_stage_barrier<0>();
    } else {
        if (later >= kMost) lm_stage_barrier<kMost * kPer>();
        else lm_stage_wait<kMost - 1, kPer>(later);
    }
}

__device__ __forceinline__ u32x4 lm_rsrc(const unsigned char* base, int bytes) {
    const uint64_t p = (uint64_t)base;
    u32x4 r;
    r.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    r.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu));
    r.z = (uint32_t)__builtin_amdgcn_readfirstlane(bytes);
    r.w = (uint32_t)kRsrcWord3;
    return r;
}

// One stage of one operand: tile rows 0 .. 32 kBlocks - 1, bytes [k0b, k0b +
// 128) of each.  Row r of the tile starts at byte r * K2 of the buffer.
// Wavefronts 0..3, one per SIMD, copy; wavefront w copies the 1-KB blocks w,
// w + 4, ..., each 8 rows, and lane l fills 16-B position l % 8 of row l / 8
// with k-chunk (l % 8) ^ lm_swz(row).  The other wavefront of each SIMD issues
// none, so it keeps the matrix core busy while its partner's copies are issued
// (measured faster than all eight wavefronts copying).
template <int kBlocks, bool kOnce>
__device__ __forceinline__ void lm_copy_stage(u32x4 rs, int K2, int k0b, int wave, int lane,
                                              uint32_t lds) {
    if (wave >= 4) return;
    const int c = (lane & 7) ^ lm_swz((wave & 1) * 8 + (lane >> 3));
    int voff = (wave * 8 + (lane >> 3)) * K2 + c * 16;
#pragma unroll
    for (int u = 0; u < kBlocks; ++u) {
        // The empty asm keeps the offsets in one register: hoisted out of the K
        // loop they would take one register per block, and spill.
        asm volatile("" : "+v"(voff));
        lm_lds_copy<kOnce>(rs, voff, k0b, lds + (u * 4 + wave) * 1024);
        voff += 32 * K2;
    }
}

struct LmCtx {
    u32x4 rh, rw;
    const unsigned char* ring;
    uint32_t lds;        // LDS address of the ring
    int K2, wave, lane;
    int offA, offB;      // bytes from a stage to this lane's first fragment of slice 0
};

__device__ __forceinline__ bf16x8 lm_frag(const LmCtx& x, int off, int tile) {
    return *(const bf16x8*)(x.ring + off + tile * 16 * 2 * kLmK);
}

// c += a b.  Written in asm so that an accumulator keeps its registers: the
// compiler gives the builtin's result registers of its own, which the 256 of
// two wavefronts per SIMD do not hold at 256-row tiles (it spilled in the K
// loop).  The operands come from LDS reads, which the compiler waits for, and
// an accumulator is next used at least three MFMAs later; who reads it
// otherwise waits with lm_mfma_drain first.
__device__ __forceinline__ void lm_mfma(const bf16x8& a, const bf16x8& b, f32x4& c) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// Waits out the matrix core's write of the last results; the compiler reads
// none of them before.
template <int kNr>
__device__ __forceinline__ void lm_mfma_drain(f32x4 (&acc)[4][kNr]) {
    asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < kNr; ++j) asm volatile("" : "+v"(acc[i][j]));
}

// MFMAs of row groups [kFrom, kTo) of one slice.  With `kRead`, the fragments
// at bytes `fa` and `fb` of the ring replace the consumed ones: the weight
// fragments go to `an`, and each row group's hidden-state fragment into the
// register it was consumed from, right after its MFMAs.  The reads whose
// registers are free from the start (the weights' and those of the row groups
// before kFrom) are spread over the first row groups.  Odd row groups take the
// weight fragments in reverse, so that consecutive MFMAs always share an operand
// (registers-only probe, Gaussian operands: 2,050 against 2,020 TFLOP/s; the chip
// is power limited and a repeated operand costs less).  The scheduling barriers
// hold the compiler to this order: an earlier read of a fragment would need a
// second register for it, and registers are what this kernel is short of; a
// later one would be waited for.
template <int kNr, int kFrom, int kTo, bool kRead>
__device__ __forceinline__ void lm_slice(const LmCtx& x, int fa, int fb, const bf16x8 (&a)[4],
                                         bf16x8 (&an)[4], bf16x8 (&b)[kNr],
                                         f32x4 (&acc)[4][kNr]) {
    constexpr int kFree = 4 + kFrom, kGroups = kTo - kFrom;
    constexpr int kEven = kGroups > 0 ? (kFree + kGroups - 1) / kGroups : 0;
    constexpr int kEach = kFrom > 0 && kEven < 2 ? 2 : kEven;   // the next slice's first operands early
#pragma unroll
    for (int j = kFrom; j < kTo; ++j) {
        const int first = (j - kFrom) * kEach;
        const int n = kFree - first < 0 ? 0 : kFree - first < kEach ? kFree - first : kEach;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = j & 1 ? 3 - i : i;
            lm_mfma(a[t], b[j], acc[t][j]);
            if constexpr (kRead) {
#pragma unroll
                for (int e = (i * n + 2) / 4; e < ((i + 1) * n + 2) / 4; ++e) {
                    const int f = first + e;
                    __builtin_amdgcn_sched_barrier(0);
                    if (f < 4) an[f < 4 ? f : 0] = lm_frag(x, fa, f);
                    else b[f < 4 ? 0 : f - 4] = lm_frag(x, fb, f - 4);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if constexpr (kRead) {
            __builtin_amdgcn_sched_barrier(0);
            b[j] = lm_frag(x, fb, j);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// One K step on the weight stage at ring byte wc and the hidden-state stage at
// hc, whose slice 0 fragments are in (a0, b); (wn, hn) are the next step's.  Once
// they are no longer read, hc takes the copies of the stage after next (byte kh
// of each row) and wc those of the one after that (kw).
template <int kNr, int kJ0, bool kOnce>
__device__ __forceinline__ void lm_step(const LmCtx& x, int wc, int wn, int hc, int hn, int kh,
                                        int kw, bf16x8 (&a0)[4], bf16x8 (&a1)[4],
                                        bf16x8 (&b)[kNr], f32x4 (&acc)[4][kNr]) {
    lm_slice<kNr, 0, kNr, true>(x, (x.offA ^ 64) + wc, (x.offB ^ 64) + hc, a0, a1, b, acc);
    __builtin_amdgcn_sched_barrier(0);
    lm_slice<kNr, 0, kJ0, false>(x, 0, 0, a1, a0, b, acc);
    lm_stage_barrier<8>();        // all but this wavefront's copies of the weights after next
    lm_copy_stage<kNr, false>(x.rh, x.K2, kh, x.wave, x.lane, x.lds + hc);
    lm_copy_stage<8, kOnce>(x.rw, x.K2, kw, x.wave, x.lane, x.lds + wc);
    lm_slice<kNr, kJ0, kNr, true>(x, x.offA + wn, x.offB + hn, a1, a0, b, acc);
    __builtin_amdgcn_sched_barrier(0);
}

// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (one hidden-state row).
__device__ __forceinline__ int32_t lm_row_max(int32_t v) {
    v = max(v, __shfl_xor(v, 16, 64));
    return max(v, __shfl_xor(v, 32, 64));
}

// Ranks 16 hidden-state rows (one per lane l % 16, rows past M have `have`
// unset) over 4 kElems columns: the four lanes of a row, lq = l / 16, hold
// kElems logits each, element e at column wcol0 + 16 (e / 4) + 4 lq + e % 4.
// The greatest raw pattern read as a signed integer is the exact maximum when
// it is a number in [1, +inf] and the row holds no NaN (columns past N are +0
// then, and cannot win).  Most rows end there: only a row whose maximum reaches
// `best`, its greatest key when this tile started, looks for the column (a stale
// `best` is lower, and costs an update that changes nothing).  Rows with a NaN or no positive number rank with exact keys.  The
// lane that holds the column of the row's draft token x writes its logit.
template <int kElems>
__device__ __forceinline__ unsigned long long lm_rank_rows(const uint32_t (&u)[kElems], int lq,
                                                           int64_t wcol0, int64_t N, bool have,
                                                           int32_t best) {
    int32_t sm = (int32_t)u[0];
    uint32_t um = u[0];
#pragma unroll
    for (int e = 1; e < kElems; ++e) {
        sm = max(sm, (int32_t)u[e]);
        um = max(um, u[e]);
    }
    const bool nan = um > KeyTraits<4>::kNegInfPattern || sm > KeyTraits<4>::kInf;
    sm = lm_row_max(sm);
    unsigned long long packed = 0;                    // ranks below every key
    if (__ballot(have && (nan || sm < 1)) != 0ull) {
        int32_t bk = (int32_t)0x80000000;
        int64_t bc = wcol0;
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
            const int64_t c = wcol0 + 16 * (e >> 2) + 4 * lq + (e & 3);
            const int32_t k = c < N ? f32_key(u[e]) : (int32_t)0x80000000;
            if (k > bk) {                             // strict: lowest column on ties
                bk = k;
                bc = c;
            }
        }
        packed = pack_kc(bk, bc);
        unsigned long long o = __shfl_xor(packed, 16, 64);
        packed = o > packed ? o : packed;
        o = __shfl_xor(packed, 32, 64);
        packed = o > packed ? o : packed;
        if (packed_key(packed) < best) packed = 0;
    } else if (__ballot(have && sm >= best) != 0ull) {
        int32_t c = 4 * kElems;
#pragma unroll
        for (int e = kElems - 1; e >= 0; --e)         // the lane's first equal column
            c = (int32_t)u[e] == sm ? 16 * (e >> 2) + 4 * lq + (e & 3) : c;
        c = min(c, __shfl_xor(c, 16, 64));
        c = min(c, __shfl_xor(c, 32, 64));
        if (sm >= best) packed = pack_kc(sm, wcol0 + c);
    }
    return have ? packed : 0;
}

// The lane that holds the column of its row's draft token x (of the columns of
// lm_rank_rows) writes its logit.
template <int kElems>
__device__ __forceinline__ void lm_draft_logit(const uint32_t (&u)[kElems], int lq, int64_t wcol0,
                                               int64_t N, int64_t row, bool have, int32_t x,
                                               uint32_t* row_draft_bits) {
    const int64_t xo = (int64_t)x - wcol0;
    const bool mine =
        have && xo >= 0 && xo < 4 * kElems && (int64_t)x < N && (((int)xo >> 2) & 3) == lq;
    if (__ballot(mine) != 0ull) {
        const int e0 = ((int)xo >> 4) * 4 + ((int)xo & 3);
        uint32_t z = 0;
#pragma unroll
        for (int e = 0; e < kElems; ++e) z |= e == e0 ? u[e] : 0u;   // no indexing: registers
        if (mine) row_draft_bits[row] = z;
    }
}

// A row's greatest key so far over all tiles, read past the caches that other
// tiles' atomics do not pass.
__device__ __forceinline__ int32_t lm_best_key(const unsigned long long* row_best, int64_t row) {
    return packed_key(
        __hip_atomic_load(row_best + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

template <int kNr, int kGroup, bool kOnce>
__global__ __launch_bounds__(kLmThreads) void asd_lmhead_kernel(
    const unsigned char* __restrict__ hidden, const unsigned char* __restrict__ weight,
    int64_t M, int64_t N, int64_t K, uint32_t tiles_m, uint32_t tiles,
    const int32_t* __restrict__ draft_tokens, unsigned long long* __restrict__ row_best,
    uint32_t* __restrict__ row_draft_bits) {
    constexpr int kRows = 32 * kNr;
    constexpr int kJ0 = kNr >= 6 ? 2 : 1;
    constexpr int kW = kLmCols * 2 * kLmK, kH = kRows * 2 * kLmK;     // bytes of a stage
    constexpr int kH0 = 3 * kW, kH1 = kH0 + kH;
    __shared__ __attribute__((aligned(1024))) unsigned char ring[3 * kW + 2 * kH];
    int32_t* const s_draft = (int32_t*)ring;             // once the K loop is over
    int32_t* const s_best = s_draft + kRows;
    unsigned long long* const s_top = (unsigned long long*)(s_best + kRows);   // [4][kRows]

    // XCD-aware order: workgroup i runs on XCD i % 8, and each XCD takes a run
    // of consecutive positions.  Positions run over groups of kGroup weight
    // tiles (slowest), row tiles, then the weight tiles of the group (fastest):
    // the tiles of a group start together and read each hidden-state slice
    // once between them from L2, and a group of weight tiles serves the row
    // tiles that the XCD runs alongside it.
    const uint32_t linear = blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8;
    const uint32_t group = linear / (kGroup * tiles_m), within = linear % (kGroup * tiles_m);
    // Divisions run on the vector unit: back to scalars, or each copy loops
    // over the values its resource could have.
    const int rt = __builtin_amdgcn_readfirstlane((int)(within / kGroup));
    const int ct = __builtin_amdgcn_readfirstlane((int)(group * kGroup + within % kGroup));
    if (linear >= tiles || (int64_t)ct * kLmCols >= N) return;
    const int64_t row0 = (int64_t)rt * kRows, col0 = (int64_t)ct * kLmCols;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar LDS targets
    const int wv = wave & 3, wr = wave >> 2;

    LmCtx x;
    x.K2 = (int)(K * 2);
    x.rh = lm_rsrc(hidden + row0 * x.K2, (int)(min((int64_t)kRows, M - row0) * x.K2));
    x.rw = lm_rsrc(weight + col0 * x.K2, (int)(min((int64_t)kLmCols, N - col0) * x.K2));
    x.ring = ring;
    x.lds = (uint32_t)(uintptr_t)(unsigned char ASD_LDS*)ring;
    x.wave = wave;
    x.lane = lane;
    const int chunk = (lane >> 4) ^ lm_swz(lane & 15);
    x.offA = (wv * 64 + (lane & 15)) * 2 * kLmK + chunk * 16;
    x.offB = (wr * 16 * kNr + (lane & 15)) * 2 * kLmK + chunk * 16;

    // K / 64 is even.  Copies past the last stage are clamped to it: they
    // refill a stage that is no longer read, and the fragments read after the
    // last stage are never used.
    const int KT = (int)(K / kLmK);
    int32_t my_draft = -1, my_best = 0x7fffffff;   // of row tid, for the epilogue
    if (tid < kRows && row0 + tid < M) {
        my_draft = draft_tokens[row0 + tid];
        my_best = lm_best_key(row_best, row0 + tid);
    }
    asm volatile("" : "+v"(my_draft), "+v"(my_best));   // here, not after the copies
    lm_copy_stage<kNr, false>(x.rh, x.K2, 0, wave, lane, x.lds + kH0);
    lm_copy_stage<8, kOnce>(x.rw, x.K2, 0, wave, lane, x.lds);
    lm_copy_stage<8, kOnce>(x.rw, x.K2, 2 * kLmK, wave, lane, x.lds + kW);
    f32x4 acc[4][kNr];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < kNr; ++j) acc[i][j] = (f32x4)(0.0f);
    lm_stage_barrier<8>();
    lm_copy_stage<kNr, false>(x.rh, x.K2, 2 * kLmK, wave, lane, x.lds + kH1);
    lm_copy_stage<8, kOnce>(x.rw, x.K2, min(2, KT - 1) * 2 * kLmK, wave, lane, x.lds + 2 * kW);
    bf16x8 a0[4], a1[4], b[kNr];
#pragma unroll
    for (int i = 0; i < 4; ++i) a0[i] = lm_frag(x, x.offA, i);
#pragma unroll
    for (int j = 0; j < kNr; ++j) b[j] = lm_frag(x, x.offB + kH0, j);
    lm_mfma_drain<kNr>(acc);                  // the zeros are written before an MFMA reads them
    __builtin_amdgcn_s_waitcnt(kWaitLds);     // else the loop's first wait counts scalar loads too
    int w0 = 0, w1 = kW, w2 = 2 * kW;         // weight stages of steps s, s + 1 and s + 2
    for (int s = 0; s < KT; s += 2) {
        auto at = [&](int step) { return min(step, KT - 1) * 2 * kLmK; };
        lm_step<kNr, kJ0, kOnce>(x, w0, w1, kH0, kH1, at(s + 2), at(s + 3), a0, a1, b, acc);
        lm_step<kNr, kJ0, kOnce>(x, w1, w2, kH1, kH0, at(s + 3), at(s + 4), a0, a1, b, acc);
        const int t = w0;
        w0 = w2;
        w2 = w1;
        w1 = t;
    }
    lm_mfma_drain<kNr>(acc);
    lm_stage_barrier<0>();                    // no copy and no fragment read outlives the K loop
    if (tid < kRows) {
        s_draft[tid] = my_draft;
        s_best[tid] = my_best;
    }
    __syncthreads();

    // ---- epilogue.  The four wavefronts of a row meet in LDS and the workgroup
    // updates the row once: the updates of the tiles that run side by side meet
    // on the same few rows, and with one of each wavefront they were what bound
    // calls of few K steps (129 rows, d = 128: 32,000 columns 21.4 us, 15.5 so;
    // 128,256 columns 38.7, 25.4; at 256 rows 44.9, 31.1; d = 1,024, 87.1, 74.8).
    const int64_t wcol0 = col0 + wv * 64;
    int le = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(le));              // recomputed, not kept through the K loop
#pragma unroll
    for (int j = 0; j < kNr; ++j) {
        const int r = wr * 16 * kNr + j * 16 + (le & 15);        // tile row
        __builtin_amdgcn_sched_barrier(0);
        uint32_t u[16];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                // The element is copied out before its bits are taken: a bit
                // cast of the vector element itself read element 0 for every v.
                const float val = acc[i][j][v];
                u[4 * i + v] = __float_as_uint(val);
            }
        const bool have = row0 + r < M;
        const unsigned long long p = lm_rank_rows<16>(u, le >> 4, wcol0, N, have, s_best[r]);
        if (le < 16) s_top[wv * kRows + r] = p;
        lm_draft_logit<16>(u, le >> 4, wcol0, N, row0 + r, have, s_draft[r], row_draft_bits);
    }
    __syncthreads();
    if (tid < kRows) {
        unsigned long long p = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) p = max(p, s_top[w * kRows + tid]);
        if (p != 0) atomicMax(row_best + row0 + tid, p);
    }
}

// ---- few rows: the weights' stream
//
// Up to 128 hidden-state rows.  The call is then bound by reading the weights
// once, and the tile kernel above leaves most of the memory idle (one 32-KB
// stage per CU in flight, a last round of tiles that is part full).  Here the
// workgroups that the CUs hold at once take equal shares of the weight rows, in
// tiles of 16 kVt kWaves, and stream them without a break: K steps of kK run
// through a ring of kStages LDS stages, kStages - 1 of them in flight, across
// the tiles of a share.  Wavefront w copies and multiplies the tile's weight
// rows 16 kVt w .. against every hidden-state row (16 kRt at most), in the
// operand layouts of the tile kernel, and keeps each row's greatest pair in
// registers; the workgroup updates the rows once, at its end.
//
//  - The weights are read once: their copies are non-temporal (9 rows of the
//    headline vocabulary, d = 5,120: 264 us cached, 238 us so).
//  - Each copied row is at least a whole 128-B line per step.  With fragments
//    loaded straight into registers (64 B of 16 rows per load) the same call
//    took 293 us.
//  - A logit is one chain of MFMAs over the k-slices of 32 in ascending order,
//    as in the tile kernel, whatever workgroup holds its column: equal weight
//    rows tie exactly, and a row's logits do not depend on the rows beside it.
//    (K loops that start at another step in each workgroup spread weight rows a
//    multiple of 4 KB apart over more memory channels: 151,936 columns, 32 rows,
//    d = 2,048, 106.6 us for 124.5; d = 4,096, 197.9 for 202.6.  They sum equal
//    rows in different orders, so the greater of two duplicates was a matter of
//    rounding.)
//
// 151,936 columns, d = 5,120, call times on one box against the tile kernel above
// on the same rows: 9 rows 234 us (6.7 TB/s) against 302; 32 rows 232 / 303; 64
// rows 252 / 309; 128 rows 313 / 326.
//
// Each K step waits until at most the copies of the later stages are outstanding
// (they complete in order), then meets the other wavefronts: the step's stage is
// whole, and the stage before it is read out and takes the next copies.
template <int kWaves, int kVt, int kRt, int kK, int kStages>
__global__ __launch_bounds__(64 * kWaves) void asd_lmhead_stream_kernel(
    const unsigned char* __restrict__ hidden, const unsigned char* __restrict__ weight,
    int32_t M, int64_t K, uint32_t share, uint32_t extra, const int32_t* __restrict__ draft_tokens,
    unsigned long long* __restrict__ row_best, uint32_t* __restrict__ row_draft_bits) {
    static_assert(kK == 64 || kK == 128, "rows of one or two cache lines");
    constexpr int kCols = 16 * kVt * kWaves, kPitch = 2 * kK;
    constexpr int kStageBytes = (kCols + 16 * kRt) * kPitch;
    constexpr int kDraftBytes = (16 * kRt + 63) / 64 * 256;
    constexpr int kW = kVt * kK / 32, kH = kRt * kK / 32 / kWaves;   // blocks a wavefront copies
    static_assert(kH * kWaves * 32 == kRt * kK && kStages >= 2, "every wavefront copies alike");
    __shared__ __attribute__((aligned(1024))) unsigned char ring[kStages * kStageBytes + kDraftBytes];
    const int32_t* const s_draft = (const int32_t*)(ring + kStages * kStageBytes);
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K2 = (int)(K * 2), KT = (int)(K / kK);
    // This workgroup's weight rows, an equal share, in tiles of kCols.
    const uint32_t bid = blockIdx.x;
    const int64_t first = (int64_t)bid * share + min(bid, extra);
    const int64_t end = first + share + (bid < extra);
    const int steps = (int)((end - first + kCols - 1) / kCols) * KT;
    const u32x4 rh = lm_rsrc(hidden, M * K2);
    auto tile_rsrc = [&](int64_t col) {
        return lm_rsrc(weight + col * K2, (int)(min((int64_t)kCols, end - col) * K2));
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(unsigned char ASD_LDS*)ring;

    // 1-KB blocks of 512 / kK rows; the 16-B position p of row r holds k-chunk
    // p ^ swz(r) (no bank conflicts in copies and fragment reads).
    auto swz = [](int r) { return kK == 64 ? lm_swz(r & 15) : r & 15; };
    constexpr int kLanes = kK / 8;                       // lanes, and 16-B chunks, of a row
    auto lane_offset = [&](int block) {
        const int row = block * (64 / kLanes) + lane / kLanes;
        return row * K2 + ((lane % kLanes) ^ swz(row)) * 16;
    };
    int vw[kW], vh[kH];
#pragma unroll
    for (int u = 0; u < kW; ++u) vw[u] = lane_offset(wave * kW + u);
#pragma unroll
    for (int u = 0; u < kH; ++u) vh[u] = lane_offset(wave * kH + u);
    // The next step to copy: of tile `ccol`, byte `ck` of each row.
    int64_t ccol = first;
    u32x4 rw = tile_rsrc(ccol);
    int ck = 0;
    auto copy_next = [&](int slot) {
        const uint32_t base = lds0 + slot * kStageBytes;
#pragma unroll
        for (int u = 0; u < kW; ++u) lm_lds_copy<true>(rw, vw[u], ck, base + (wave * kW + u) * 1024);
#pragma unroll
        for (int u = 0; u < kH; ++u)
            lm_lds_copy<false>(rh, vh[u], ck, base + kCols * kPitch + (wave * kH + u) * 1024);
        ck += kPitch;
        if (ck == K2) {
            ck = 0;
            ccol += kCols;
            if (ccol < end) rw = tile_rsrc(ccol);
        }
    };
    // The draft tokens, by the oldest copies of all.
    const u32x4 rd = lm_rsrc((const unsigned char*)draft_tokens, M * 4);
#pragma unroll
    for (int u = 0; u < (16 * kRt + 63) / 64; ++u)
        lm_lds_copy_dword(rd, (u * 64 + lane) * 4, lds0 + kStages * kStageBytes + u * 256);
    unsigned long long top[kRt];              // greatest (key, column) of this wavefront's columns
#pragma unroll
    for (int j = 0; j < kRt; ++j) top[j] = 0; // ranks below every key
    for (int t = 0; t < kStages - 1 && t < steps; ++t) copy_next(t);
    f32x4 acc[kVt][kRt];
#pragma unroll
    for (int i = 0; i < kVt; ++i)
#pragma unroll
        for (int j = 0; j < kRt; ++j) acc[i][j] = (f32x4)(0.0f);
    const int offA = (wave * 16 * kVt + lr) * kPitch + ((lq ^ swz(lr)) << 4);
    const int offB = (kCols + lr) * kPitch + ((lq ^ swz(lr)) << 4);
    int slot = 0, k_left = KT;
    int64_t wcol0 = first + wave * 16 * kVt;
    for (int t = 0; t < steps; ++t) {
        lm_stage_wait<kStages - 2, kW + kH>(steps - 1 - t);
        if (t + kStages - 1 < steps) copy_next(slot == 0 ? kStages - 1 : slot - 1);
        const unsigned char* const st = ring + slot * kStageBytes;
#pragma unroll
        for (int k = 0; k < kK / 32; ++k) {
            bf16x8 a[kVt];
#pragma unroll
            for (int i = 0; i < kVt; ++i)
                a[i] = *(const bf16x8*)(st + (offA ^ (k * 64)) + i * 16 * kPitch);
#pragma unroll
            for (int j = 0; j < kRt; ++j) {
                const bf16x8 b = *(const bf16x8*)(st + (offB ^ (k * 64)) + j * 16 * kPitch);
#pragma unroll
                for (int i = 0; i < kVt; ++i)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i][j], 0, 0, 0);
            }
        }
        slot = slot == kStages - 1 ? 0 : slot + 1;
        if (--k_left == 0) {                  // the tile is whole: rank it
#pragma unroll
            for (int j = 0; j < kRt; ++j) {
                uint32_t u[4 * kVt];
#pragma unroll
                for (int i = 0; i < kVt; ++i) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float val = acc[i][j][v];
                        u[4 * i + v] = __float_as_uint(val);
                    }
                    acc[i][j] = (f32x4)(0.0f);
                }
                const bool have = j * 16 + lr < M;
                const unsigned long long p =
                    lm_rank_rows<4 * kVt>(u, lq, wcol0, end, have, packed_key(top[j]));
                top[j] = max(top[j], p);
                lm_draft_logit<4 * kVt>(u, lq, wcol0, end, j * 16 + lr, have, s_draft[j * 16 + lr],
                                        row_draft_bits);
            }
            k_left = KT;
            wcol0 += kCols;
        }
    }

    // The workgroup's greatest pair of each row updates the row's if it reaches
    // it (read first: one atomic per row and workgroup at most).
    __syncthreads();                          // the ring is read out
    unsigned long long* const s_top = (unsigned long long*)ring;     // [kWaves][16 kRt]
#pragma unroll
    for (int j = 0; j < kRt; ++j)
        if (lq == 0) s_top[wave * 16 * kRt + j * 16 + lr] = top[j];
    __syncthreads();
    if (tid < 16 * kRt && tid < M) {
        unsigned long long p = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) p = max(p, s_top[w * 16 * kRt + tid]);
        if (packed_key(p) >= lm_best_key(row_best, tid)) atomicMax(row_best + tid, p);
    }
}

// As many workgroups as the CUs hold at once (160 KB of LDS each), none with
// fewer than 64 columns where that can be helped.  Up to kLmStreamShortK hidden
// values only as many as whole tiles need: a tile that is part full saves reads,
// which short K loops do not wait for, and costs its fragments, its ranking and
// another workgroup's updates of the same rows.
template <int kWaves, int kVt, int kRt, int kK, int kStages>
void launch_lmhead_stream(hipStream_t stream, const void* hidden, const void* weight, int64_t rows,
                          int64_t vocab, int64_t d, int num_cus, const int32_t* draft_tokens,
                          unsigned long long* best, uint32_t* draft_bits) {
    constexpr int kStageBytes = (16 * kVt * kWaves + 16 * kRt) * 2 * kK;
    constexpr int kPerCu = 160 * 1024 / (kStageBytes * kStages + (16 * kRt + 63) / 64 * 256);
    static_assert(kPerCu >= 1, "the ring fits the LDS of a CU");
    constexpr int kCols = 16 * kVt * kWaves;
    const int64_t slots = (int64_t)num_cus * kPerCu;
    const int64_t tiles = (vocab + slots * kCols - 1) / (slots * kCols);     // of a workgroup
    const int64_t grid = d <= kLmStreamShortK ? (vocab + tiles * kCols - 1) / (tiles * kCols)
                                              : min((vocab + 63) / 64, slots);
    asd_lmhead_stream_kernel<kWaves, kVt, kRt, kK, kStages><<<(unsigned)grid, 64 * kWaves, 0, stream>>>(
        (const unsigned char*)hidden, (const unsigned char*)weight, (int32_t)rows, d,
        (uint32_t)(vocab / grid), (uint32_t)(vocab % grid), draft_tokens, best, draft_bits);
}

template <int kNr>
void launch_lmhead_tiles(int64_t grid, hipStream_t stream, const void* hidden, const void* weight,
                         int64_t rows, int64_t vocab, int64_t d, int64_t tiles_m, int64_t tiles,
                         int64_t group, const int32_t* draft_tokens, unsigned long long* best,
                         uint32_t* draft_bits) {
    auto kernel = asd_lmhead_kernel<kNr, kLmheadGroupFew, true>;
    if constexpr (kNr >= lmhead_least_height(kLmOnceMaxRowTiles + 1))
        if (tiles_m > kLmOnceMaxRowTiles) kernel = asd_lmhead_kernel<kNr, kLmheadGroupFew, false>;
    if constexpr (kNr >= lmhead_least_height(kLmheadFewRowTiles + 1))
        if (group == kLmheadGroup) kernel = asd_lmhead_kernel<kNr, kLmheadGroup, false>;
    kernel<<<(unsigned)grid, kLmThreads, 0, stream>>>(
        (const unsigned char*)hidden, (const unsigned char*)weight, rows, vocab, d, (uint32_t)tiles_m,
        (uint32_t)tiles, draft_tokens, best, draft_bits);
}

__global__ void asd_fill_u64_kernel(unsigned long long* p, int64_t n, unsigned long long v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------- matrix-core probe
//
// The matrix-core work of asd_lmhead_kernel's 256-row tiles with no memory
// traffic: a workgroup of eight wavefronts, each wavefront issuing 64
// v_mfma_f32_16x16x32_bf16 per K step of 64 into its 4 x 8 accumulator tiles,
// with operand fragments held in registers.  Each thread reads six fragments
// once from the caller's buffer and forms four sets from them (the elements
// rotated within each fragment), two sets to a k-slice of 32, so that the
// matrix cores see data of the caller's distribution (the power a matrix core
// draws depends on its operands' bits).  Workgroup w reads the data of
// workgroup w % 64, which then stays in the cache.  Run over as many workgroups
// and steps as an LM-head launch, its duration is the practical matrix-core
// ceiling of that launch under the chip's power limit.  Thread 0 of each
// workgroup writes the binary32 bits of the sum of its accumulators.
constexpr int kProbeVecs = 6;                  // 16-byte fragments read per thread

template <int R>
__device__ __forceinline__ bf16x8 rotate_elements(bf16x8 v) {
    return __builtin_shufflevector(v, v, R % 8, (R + 1) % 8, (R + 2) % 8, (R + 3) % 8,
                                   (R + 4) % 8, (R + 5) % 8, (R + 6) % 8, (R + 7) % 8);
}

__global__ __launch_bounds__(kLmThreads) void asd_mfma_probe_kernel(
    const bf16x8* __restrict__ operands, int64_t vectors, int64_t steps,
    uint32_t* __restrict__ out) {
    bf16x8 a[2][4], b[2][8];
    const int64_t first = ((int64_t)(blockIdx.x % 64) * kLmThreads + threadIdx.x) * kProbeVecs;
#pragma unroll
    for (int k = 0; k < kProbeVecs; ++k) {
        const bf16x8 f = operands[(first + k) % vectors];
        if (k < 4) {
            a[0][k] = f;
            a[1][k] = rotate_elements<2>(f);
        } else {
            b[0][k - 4] = f;
            b[1][k - 4] = rotate_elements<2>(f);
        }
        b[0][2 + k] = rotate_elements<1>(f);
        b[1][2 + k] = rotate_elements<3>(f);
    }
    f32x4 acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = (f32x4)(0.0f);
    for (int64_t s = 0; s < steps; ++s) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][i], b[t][j], acc[i][j], 0, 0, 0);
    }
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x = acc[i][j][v];
                sum += x;
            }
    if (threadIdx.x == 0) out[blockIdx.x] = __float_as_uint(sum);
}

// ------------------------------------------------------- read probe
//
// The row kernel's access pattern with no ranking: one workgroup per row,
// groups of four 16-byte non-temporal loads per lane issued before any wait,
// each vector folded into a per-lane XOR.  Its duration is the practical read
// ceiling of that pattern.  A lane whose fold equals kProbeMark stores it to
// *out (keeps the loads live; callers can plant the mark to check the read).
constexpr uint32_t kProbeMark = 0x9e3779b9u;

__global__ __launch_bounds__(kRowThreads) __attribute__((amdgpu_waves_per_eu(8))) void
asd_read_probe_kernel(const unsigned char* __restrict__ buf, int64_t row_bytes,
                      uint32_t* __restrict__ out) {
    const u32x4* vec = (const u32x4*)(buf + (int64_t)blockIdx.x * row_bytes);
    const int64_t nvec = row_bytes / 16;
    uint32_t acc = 0;
    int64_t i = threadIdx.x;
    for (; i + (kUnroll - 1) * kRowThreads < nvec; i += kGroupVecs) {
        u32x4 r[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) r[u] = __builtin_nontemporal_load(vec + i + u * kRowThreads);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) acc ^= r[u].x ^ r[u].y ^ r[u].z ^ r[u].w;
    }
    for (; i < nvec; i += kRowThreads) {
        const u32x4 v = __builtin_nontemporal_load(vec + i);
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == kProbeMark) *out = acc;
}

}  // namespace

// ------------------------------------------------------------------ launch

hipError_t launch_verify(const Plan& plan, const CallArgs& a, void* workspace,
                         unsigned* counter, hipStream_t stream) {
    unsigned char* ws = (unsigned char*)workspace;
    RowRecord* records = (RowRecord*)(ws + plan.off_records);
    TilePartial* partials = plan.splits > 1 ? (TilePartial*)(ws + plan.off_partials) : nullptr;

    if (counter != nullptr && single_launch(plan)) {
        ScanArgs A = scan_args(a, plan.rows, plan.vocab, plan.elem_bytes);
        A.splits = plan.splits;
        A.chunk_vecs = plan.chunk_vecs;
        A.offsets = a.row_offsets;                      // NULL: packed, formed in LDS
        A.records = plan.splits == 1 ? records : nullptr;
        A.partials = partials;
        A.shard_vocab = 0;
        const dim3 grid((unsigned)(plan.rows * plan.splits));
        if (plan.elem_bytes == 2)
            asd_row_scan_kernel<2><<<grid, kRowThreads, 0, stream>>>(
                (const unsigned char*)a.logits, plan.vocab, plan.splits, plan.chunk_vecs, partials,
                records, counter, A);
        else
            asd_row_scan_kernel<4><<<grid, kRowThreads, 0, stream>>>(
                (const unsigned char*)a.logits, plan.vocab, plan.splits, plan.chunk_vecs, partials,
                records, counter, A);
        return hipGetLastError();
    }

    int64_t* packed = a.row_offsets ? nullptr : (int64_t*)(ws + plan.off_offsets);

    const dim3 grid((unsigned)(plan.rows * plan.splits));
    int32_t* row_argmax = plan.splits == 1 ? a.out_argmax : nullptr;
    hipError_t err = launch_row(plan.elem_bytes, grid, stream, (const unsigned char*)a.logits,
                                plan.vocab, (int64_t)0, plan.splits, plan.chunk_vecs,
                                a.draft_tokens, partials, records, row_argmax, a.num_requests,
                                a.block_lens, packed);
    if (err != hipSuccess) return err;

    ScanArgs A = scan_args(a, plan.rows, plan.vocab, plan.elem_bytes);
    A.splits = plan.splits;
    A.chunk_vecs = plan.chunk_vecs;
    A.offsets = a.row_offsets ? a.row_offsets : packed;
    A.records = plan.splits == 1 ? records : nullptr;   // record mode only when rows are whole
    A.partials = partials;
    A.shard_vocab = 0;
    return launch_scan(A, plan.splits > 1, stream);
}

hipError_t launch_row_pass(const Plan& plan, const void* logits, const int32_t* draft_tokens,
                          void* out_partials, hipStream_t stream) {
    return launch_row(plan.elem_bytes, dim3((unsigned)(plan.rows * plan.splits)), stream,
                      (const unsigned char*)logits, plan.vocab, (int64_t)0, plan.splits,
                      plan.chunk_vecs, draft_tokens, (TilePartial*)out_partials,
                      (RowRecord*)nullptr, (int32_t*)nullptr, (int32_t)0,
                      (const int32_t*)nullptr, (int64_t*)nullptr);
}

hipError_t launch_shard_argmax(int elem_bytes, const void* shard_logits, int64_t shard_vocab,
                               int64_t vocab_offset, int64_t rows, const int32_t* draft_tokens,
                               void* out_partials, hipStream_t stream) {
    const int64_t nvec = shard_vocab * elem_bytes / 16;
    int64_t chunk = (nvec + kRowThreads - 1) / kRowThreads * kRowThreads;
    if (chunk < kRowThreads) chunk = kRowThreads;
    return launch_row(elem_bytes, dim3((unsigned)rows), stream,
                      (const unsigned char*)shard_logits, shard_vocab, vocab_offset, 1, chunk,
                      draft_tokens, (TilePartial*)out_partials, (RowRecord*)nullptr,
                      (int32_t*)nullptr, (int32_t)0, (const int32_t*)nullptr,
                      (int64_t*)nullptr);
}

hipError_t launch_verify_partials(const void* partials, int num_shards, int64_t shard_vocab,
                                  int64_t vocab, int64_t rows, const CallArgs& a,
                                  int64_t* packed_offsets, hipStream_t stream) {
    if (!a.row_offsets && packed_offsets) {
        asd_offsets_kernel<<<1, kRowThreads, 0, stream>>>(a.num_requests, a.block_lens,
                                                          packed_offsets);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    ScanArgs A = scan_args(a, rows, vocab, 2);
    A.splits = num_shards;
    A.chunk_vecs = 0;
    A.offsets = a.row_offsets ? a.row_offsets : packed_offsets;   // NULL: summed per wavefront
    A.records = nullptr;
    A.partials = (const TilePartial*)partials;
    A.shard_vocab = shard_vocab;
    return launch_scan(A, true, stream);
}

// Requests per workgroup of the commit and opportunity kernels: one per
// wavefront while the packed layout's per-workgroup prefix sums stay short
// (at most 8,192 requests before a workgroup), else 64, so that those sums
// total about n^2 / 128 loads.
static int requests_per_block(int32_t num_requests, const int64_t* row_offsets, int waves) {
    return (row_offsets || num_requests <= 8192) ? waves : kOppMostRequests;
}

hipError_t launch_opportunity(const int32_t* draft_tokens, const int32_t* row_argmax,
                              const float* row_regret, int64_t vocab, int32_t num_requests,
                              int64_t total_rows, const int32_t* block_lens,
                              const int64_t* row_offsets, const float* taus, int32_t num_taus,
                              const int32_t* ps, int32_t num_ps, unsigned long long* counts,
                              unsigned long long* mismatches, hipStream_t stream) {
    const int per_block = requests_per_block(num_requests, row_offsets, kOppWaves);
    const unsigned blocks = (unsigned)((num_requests + per_block - 1) / per_block);
    asd_opportunity_kernel<<<blocks, 64 * kOppWaves, 0, stream>>>(
        draft_tokens, row_argmax, row_regret, vocab, num_requests, total_rows, block_lens,
        row_offsets, taus, num_taus, ps, num_ps, counts, mismatches, per_block);
    return hipGetLastError();
}

hipError_t launch_commit(const int32_t* draft_tokens, const int32_t* block_lens,
                         const int64_t* row_offsets, int32_t num_requests, int64_t total_rows,
                         const int32_t* accept_len, const int32_t* next_token, int32_t* tokens,
                         int64_t capacity, int64_t* seq_len, int32_t* committed,
                         hipStream_t stream) {
    const int per_block = requests_per_block(num_requests, row_offsets, kScanThreads / 64);
    const unsigned blocks = (unsigned)((num_requests + per_block - 1) / per_block);
    asd_commit_kernel<<<blocks, kScanThreads, 0, stream>>>(
        draft_tokens, block_lens, row_offsets, num_requests, total_rows, accept_len, next_token,
        tokens, capacity, seq_len, committed, per_block);
    return hipGetLastError();
}

hipError_t launch_lmhead_verify(const void* hidden, const void* weight, int64_t d,
                                int64_t vocab, int64_t rows, const CallArgs& a, void* workspace,
                                int num_cus, hipStream_t stream) {
    unsigned char* ws = (unsigned char*)workspace;
    unsigned long long* best = (unsigned long long*)ws;
    uint32_t* draft_bits = (uint32_t*)(ws + lmhead_draft_offset(rows));
    asd_fill_u64_kernel<<<(unsigned)((rows + 255) / 256), 256, 0, stream>>>(best, rows, 0ull);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    if (rows <= kLmStreamMaxRows) {
        // The rows rounded up to a power of two of 16-row groups.  One group
        // leaves LDS for two workgroups per CU (with four waves); for eight
        // groups wide tiles read the hidden states less often (128 rows, d =
        // 5,120: 316 us with 256 columns, 323-328 us with 128), but their ring
        // is one stage shorter, which costs more where a CU has one narrow tile
        // only (128 rows, vocabulary 32,000: d = 1,024, 30.1 against 27.5 us; d =
        // 4,096, 78.8 against 65.8).
        auto launch = rows <= 16   ? launch_lmhead_stream<4, 1, 1, 128, 3>
                      : rows <= 32 ? launch_lmhead_stream<8, 1, 2, 128, 3>
                      : rows <= 64 ? launch_lmhead_stream<8, 1, 4, 128, 3>
                      : vocab > (int64_t)128 * num_cus ? launch_lmhead_stream<8, 2, 8, 64, 3>
                                                       : launch_lmhead_stream<8, 1, 8, 64, 4>;
        launch(stream, hidden, weight, rows, vocab, d, num_cus, a.draft_tokens, best, draft_bits);
    } else {
        const int64_t tiles_m = lmhead_row_tiles(rows);
        const int64_t group = tiles_m <= kLmheadFewRowTiles ? kLmheadGroupFew : kLmheadGroup;
        // positions: row tiles x the weight tiles rounded up to whole groups
        const int64_t tiles =
            tiles_m * group * (((vocab + kLmCols - 1) / kLmCols + group - 1) / group);
        const int64_t grid = (tiles + 7) / 8 * 8;
        const int64_t nr = lmhead_tile_height(rows);
        auto launch = nr == 5   ? launch_lmhead_tiles<5>
                      : nr == 6 ? launch_lmhead_tiles<6>
                      : nr == 7 ? launch_lmhead_tiles<7>
                                : launch_lmhead_tiles<8>;
        launch(grid, stream, hidden, weight, rows, vocab, d, tiles_m, tiles, group,
               a.draft_tokens, best, draft_bits);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    ScanArgs A = scan_args(a, rows, vocab, 2);
    A.splits = 1;
    A.chunk_vecs = 0;
    A.offsets = a.row_offsets;
    if (!A.offsets && a.num_requests > kWaveOffsetsMaxRequests) {
        int64_t* packed = (int64_t*)(ws + lmhead_offsets_offset(rows));
        asd_offsets_kernel<<<1, kRowThreads, 0, stream>>>(a.num_requests, a.block_lens, packed);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        A.offsets = packed;
    }
    A.records = nullptr;
    A.partials = nullptr;
    A.shard_vocab = 0;
    A.row_best = best;
    A.row_draft_bits = draft_bits;
    return launch_scan(A, true, stream);
}

hipError_t launch_mfma_probe(const void* operands, int64_t vectors, int64_t workgroups,
                             int64_t steps, uint32_t* out, hipStream_t stream) {
    asd_mfma_probe_kernel<<<(unsigned)workgroups, kLmThreads, 0, stream>>>(
        (const bf16x8*)operands, vectors, steps, out);
    return hipGetLastError();
}

hipError_t launch_read_probe(const void* buf, int64_t rows, int64_t row_bytes, uint32_t* out,
                             hipStream_t stream) {
    asd_read_probe_kernel<<<(unsigned)rows, kRowThreads, 0, stream>>>(
        (const unsigned char*)buf, row_bytes, out);
    return hipGetLastError();
}

}  // namespace asd
