// SparseLoCo outer step for gfx950 (MI355X): kernels and C ABI.
//
// The entry points follow the update equations of section 2.1 of the paper:
// compress (pseudo-gradient, error-feedback fold, chunk Top-kappa, Q, residual;
// per replica, or for all replicas of a single-node simulation at once),
// aggregate (mean over replicas), outer_update (outer SGD), and aggregate_update
// (the last two in one pass).  Nothing here is a dense contraction, so no matrix
// cores are used: the kernels stream 16-byte-per-lane non-temporal accesses, keep
// each 4096-element chunk in registers (16 values per lane, 256 lanes) and use
// LDS only for the small hand-offs of the selection and for the dense
// accumulator of the mean.
//
// Element layout of a chunk inside a workgroup: lane `tid` holds, for slot
// s = 0..3 and j = 0..3, local index  s*1024 + tid*4 + j  (one float4 per slot).
// A chunk is addressed as 64 local rows of 64 elements: local index idx sits at
// element  offset + (idx >> 6) * stride + (idx & 63)  of its tensor.  A flat chunk
// has stride 64 (every load instruction of the workgroup then covers 4 KiB
// contiguous); a 64 x 64 tile of a matrix has stride = number of columns (256-byte
// row segments).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <new>
#include <type_traits>
#include <vector>

#include "launch_rules.h"
#include "sparseloco.h"

namespace {

constexpr int kChunk = SPLC_CHUNK;
constexpr int kThreads = 256;            // one workgroup per chunk
constexpr int kCandCap = 448;            // candidates the exact selection handles (seven per lane; two strip workgroups'
                                         // shares of the LDS end here)
constexpr int kFilterKappaMax = 256;     // the candidate filter needs kappa <= number of lanes

struct ChunkDesc {
    uint32_t tensor;                     // index into the pointer tables
    uint32_t n_c;                        // elements in this chunk (kChunk unless it is an edge chunk)
    uint64_t offset;                     // element offset of local index 0 inside its tensor
    uint32_t stride;                     // elements between local rows: 64 (flat) or the matrix's columns (tile)
    uint8_t h;                           // local rows present (1..64)
    uint8_t w;                           // width of every row but the last
    uint8_t last_w;                      // width of the last row (flat tail), = w for a tile
    uint8_t vec;                         // bit 0: complete (all 4096 elements present), every 4-element vector whole;
                                         // bit 1: and every row of a bf16 array starts at a dword
    uint32_t id;                         // chunk number (position of its message in pairs / scales / values)
    uint32_t reserved;
};
static_assert(sizeof(ChunkDesc) == 32, "chunk table entries are 32 bytes");

// Address of lane tid's 4-element vector in slot s (local rows 16 s + tid / 16, columns 4 (tid % 16)...).
// The slot part is uniform and stays in scalar registers; the per-lane part is one 32-bit byte
// offset shared by all slots and arrays (a chunk spans less than 4 GiB: stride < 2^24).
template <class T>
__device__ __forceinline__ T* vec_at(T* origin, const ChunkDesc& d, int tid, int s) {
    const uint32_t lane_bytes = ((uint32_t)(tid >> 4) * d.stride + (uint32_t)(tid & 15) * 4u) * (uint32_t)sizeof(T);
    const uint64_t slot_bytes = (uint64_t)((uint32_t)s * 16u * d.stride) * sizeof(T);
    using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return reinterpret_cast<T*>(reinterpret_cast<Byte*>(origin) + slot_bytes + lane_bytes);
}
// Edge chunks, four elements at a time.  Of the four elements of lane tid in slot s the first n are present (absent ones
// are always the last: rows end, they do not begin, inside a vector).  A lane with n < 4 reads the vector that ENDS at its
// last element, which `pull` then brings to the front, and a lane with none reads the one that ends at the chunk's first
// (up to) four: every lane loads unconditionally, all of a lane's loads are in flight at once, and an edge chunk costs
// little more than a complete one (compress, against element by element: 23 tiles of 37- and 141-column matrices 14.0 -> 9.0 us, 1075
// tiles of 42 columns 23.1 -> 14.6; three tensors of which two end in a tail 7.6 -> 6.0).  What a vector holds before its row belongs
// to the same tensor and is thrown away; where nothing need lie there (`narrow`: the first rows of a matrix of fewer than four
// columns, a tensor of fewer than four elements) the four are read one by one, the tensor's first in place of those before it.
struct EdgeVec {
    uint32_t n;                          // elements present
    uint32_t from4;                      // first element read, relative to the chunk's origin, plus 4
};
__device__ __forceinline__ EdgeVec edge_vec(const ChunkDesc& d, int tid, int s) {
    const uint32_t lr = (uint32_t)s * 16u + ((uint32_t)tid >> 4), lc = ((uint32_t)tid & 15u) * 4u;
    const uint32_t width = lr + 1 < d.h ? d.w : (lr + 1 == d.h ? d.last_w : 0u);
    const uint32_t n = width > lc ? (width - lc < 4u ? width - lc : 4u) : 0u;
    const uint32_t w0 = d.h > 1 ? d.w : d.last_w;
    return {n, n ? lr * d.stride + lc + n : (w0 < 4u ? w0 : 4u)};
}
__device__ __forceinline__ bool narrow(const ChunkDesc& d) {
    return d.offset == 0 && (d.h > 1 ? d.w : d.last_w) < 4;       // (any other chunk has four elements before its origin)
}
// Whether slot s (16 rows) of a chunk holds anything.  The tail of a tensor, mostly, is a few rows: the aggregation and the
// outer update leave its other slots out (4000 chunks of 40 elements: outer update 8.7 -> 5.3 us, mean over 17 replicas, kappa
// 300, 13.6 -> 10.7; edge chunks that use all four take up to 0.2 us longer a launch).
template <bool VEC>
__device__ __forceinline__ bool slot_used(const ChunkDesc& d, int s) { return VEC || splc::slot_used(d.h, s); }
// Where the vector of `v` starts in an array whose element at the chunk's origin is *origin.
template <class T>
__device__ __forceinline__ T* edge_at(T* origin, EdgeVec v) {
    using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return reinterpret_cast<T*>(reinterpret_cast<Byte*>(origin) - 4 * sizeof(T) + (uint64_t)(v.from4 * (uint32_t)sizeof(T)));
}
// The n elements at the end of four to the front, +0 behind them.
__device__ __forceinline__ void pull(uint32_t n, float& a, float& b, float& c, float& d) {
    const bool one = (n & 1u) != 0, two = n == 1u || n == 2u;     // by 4 - n: 3 = 1 + 2, 2, 1
    a = one ? b : a; b = one ? c : b; c = one ? d : c;
    a = two ? c : a; b = two ? d : b;
    a = n > 0 ? a : 0.f; b = n > 1 ? b : 0.f; c = n > 2 ? c : 0.f; d = n > 3 ? d : 0.f;
}
enum { MODE_PARAMS_F32 = 0, MODE_DIRECT_F32 = 1, MODE_DIRECT_BF16 = 2 };

// Streaming accesses: every dense array is touched exactly once per launch, so loads and stores
// carry the non-temporal hint (measured on MI355X: 3 reads + 1 write streams at ~6.0 TB/s with
// the hint against ~5.6 TB/s without).
// The vector types promise only 4-byte alignment: rows of a tile start at any multiple of 4 bytes,
// and global memory accepts dword-aligned multi-dword accesses.
typedef float vfloat4 __attribute__((ext_vector_type(4), aligned(4)));

// Every tensor lives in global memory; saying so lets the compiler emit global_ instead of flat_
// instructions.
#define SPLC_GLOBAL __attribute__((address_space(1)))
typedef uint32_t vuint2 __attribute__((ext_vector_type(2), aligned(2)));        // rows of bf16 may start at any element
__device__ __forceinline__ float4 stream_load4(const float* p) {
    vfloat4 v = __builtin_nontemporal_load((const SPLC_GLOBAL vfloat4*)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 stream_load4(const uint16_t* p) {       // four bf16
    vuint2 v = __builtin_nontemporal_load((const SPLC_GLOBAL vuint2*)p);
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ float4 cached_load4(const float* p) {
    vfloat4 v = *(const SPLC_GLOBAL vfloat4*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 cached_load4(const uint16_t* p) {
    vuint2 v = *(const SPLC_GLOBAL vuint2*)p;
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ float4 edge_load4_narrow(const float* origin, EdgeVec v) {
    auto at = [&](uint32_t j) { return origin[v.from4 + j < 4 ? 0u : v.from4 + j - 4]; };
    return make_float4(at(0), at(1), at(2), at(3));
}
__device__ __forceinline__ uint2 edge_load4_narrow(const uint16_t* origin, EdgeVec v) {
    auto at = [&](uint32_t j) { return (uint32_t)origin[v.from4 + j < 4 ? 0u : v.from4 + j - 4]; };
    return make_uint2(at(0) | at(1) << 16, at(2) | at(3) << 16);
}
template <bool STREAM, class T>
__device__ __forceinline__ auto load4(const T* p) {
    if constexpr (STREAM) return stream_load4(p);
    else return cached_load4(p);
}
__device__ __forceinline__ void stream_store4(float* p, float4 v) {
    vfloat4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, (SPLC_GLOBAL vfloat4*)p);
}
template <bool STREAM>
__device__ __forceinline__ void store4(float* p, float4 v) {
    vfloat4 t = {v.x, v.y, v.z, v.w};
    if constexpr (STREAM) stream_store4(p, v);
    else *(SPLC_GLOBAL vfloat4*)p = t;
}
// Whether the rows of a complete chunk are whole cache lines.  Those of a tile in a matrix whose row length is no
// multiple of 32 floats share their first and last line with the neighbouring tiles, and are accessed without the hint: with it
// the lines are gone from the L2 when the neighbour asks for them (20M parameters in rows of 3687, mean 30 -> 17 us; the
// one-launch step of two replicas 201 -> 128; compress of 6000 tiles of 1219 columns, loads and store with it / neither: from
// parameters 97 / 66 us, in no cache 100 / 82, from fp32 76 / 49, 78 / 63, from bf16 67 / 43, 87 / 56).
__device__ __forceinline__ bool whole_lines(const ChunkDesc& d) { return d.stride % 32u == 0; }

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// e' = fl(fl(beta * e) + delta), delta = fl(theta_outer - theta_local) or given (section 2.1, lines 1-2).
__device__ __forceinline__ float fold(float beta, float e, float delta) {
    return __fadd_rn(__fmul_rn(beta, e), delta);
}

// One slot folded: from parameters, from an fp32 or from a bf16 pseudo-gradient (bf16 -> fp32 is the exact widening: the
// 16 bits become the upper half of the word).
__device__ __forceinline__ void fold4(float beta, float4 e, float4 o, float4 l, float* x) {
    x[0] = fold(beta, e.x, __fsub_rn(o.x, l.x));
    x[1] = fold(beta, e.y, __fsub_rn(o.y, l.y));
    x[2] = fold(beta, e.z, __fsub_rn(o.z, l.z));
    x[3] = fold(beta, e.w, __fsub_rn(o.w, l.w));
}
__device__ __forceinline__ void fold4(float beta, float4 e, float4 delta, float* x) {
    x[0] = fold(beta, e.x, delta.x);
    x[1] = fold(beta, e.y, delta.y);
    x[2] = fold(beta, e.z, delta.z);
    x[3] = fold(beta, e.w, delta.w);
}
__device__ __forceinline__ void fold4(float beta, float4 e, uint2 delta, float* x) {
    x[0] = fold(beta, e.x, __uint_as_float(delta.x << 16));
    x[1] = fold(beta, e.y, __uint_as_float(delta.x & 0xFFFF0000u));
    x[2] = fold(beta, e.z, __uint_as_float(delta.y << 16));
    x[3] = fold(beta, e.w, __uint_as_float(delta.y & 0xFFFF0000u));
}

// All loads of a lane are in flight before the first is waited for.
template <int MODE, class Chunk>
__device__ __forceinline__ void load_fold(const void* __restrict__ a, const void* __restrict__ b, const float* __restrict__ e,
                                          float beta, float (&x)[16], const Chunk& chunk) {
    using Source = typename std::conditional<MODE == MODE_DIRECT_BF16, uint16_t, float>::type;
    const float* pe = e + chunk.d.offset;
    const Source* pa = static_cast<const Source*>(a) + chunk.d.offset;
    float4 ev[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) ev[s] = chunk.load(pe, s);
    decltype(chunk.load(pa, 0)) av[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) av[s] = chunk.load(pa, s);
    if constexpr (MODE == MODE_PARAMS_F32) {
        const float* pb = static_cast<const float*>(b) + chunk.d.offset;
        float4 bv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) bv[s] = chunk.load(pb, s);
#pragma unroll
        for (int s = 0; s < 4; ++s) fold4(beta, ev[s], av[s], bv[s], x + 4 * s);
    } else {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) fold4(beta, ev[s], av[s], x + 4 * s);
    }
}
// The present ones (bits of `there`, the lowest first) of four elements of an edge chunk.
__device__ __forceinline__ void store_edge(float* p, uint32_t there, float4 v) {
    if (there == 0xFu) {
        store4<false>(p, v);
    } else {
        if (there & 1u) p[0] = v.x;
        if (there & 2u) p[1] = v.y;
        if (there & 4u) p[2] = v.z;
    }
}

// What lane tid reads and writes of slot s of the array whose element at the chunk's origin is *p.  What is read of an
// edge chunk is still to be pulled.
template <bool STREAM>
struct CompleteChunk {
    const ChunkDesc& d;
    int tid;
    template <class T> __device__ __forceinline__ auto load(const T* p, int s) const { return load4<STREAM>(vec_at(p, d, tid, s)); }
    __device__ __forceinline__ void store(float* p, int s, float4 v) const { store4<STREAM>(vec_at(p, d, tid, s), v); }
};
template <bool NARROW>
struct EdgeChunk {
    const ChunkDesc& d;
    int tid;
    template <class T> __device__ __forceinline__ auto load(const T* p, int s) const {
        const EdgeVec v = edge_vec(d, tid, s);
        if constexpr (NARROW) return edge_load4_narrow(p, v);
        else return load4<false>(edge_at(p, v));
    }
    __device__ __forceinline__ void store(float* p, int s, float4 v) const {
        store_edge(vec_at(p, d, tid, s), (1u << edge_vec(d, tid, s).n) - 1u, v);
    }
};
// use(chunk) with the way this chunk is accessed.  hint: a complete one in any case with the streaming hint.
template <bool VEC, class Use>
__device__ __forceinline__ void with_chunk(const ChunkDesc& d, int tid, Use use, bool hint = false) {
    if constexpr (VEC) {
        // (the statements that say which side this is keep the compiler from merging the two, which drops the hint)
        if (whole_lines(d) || hint) {
            asm volatile("; whole lines from here");
            use(CompleteChunk<true>{d, tid});
            asm volatile("; whole lines to here");
        } else {
            asm volatile("; shared lines from here");
            use(CompleteChunk<false>{d, tid});
            asm volatile("; shared lines to here");
        }
    } else {
        if (narrow(d)) use(EdgeChunk<true>{d, tid});
        else use(EdgeChunk<false>{d, tid});
    }
}
// The present elements of an edge chunk to the front of their vectors, +0 for absent ones; returns the mask of the
// present ones (bit el: element el of lane tid).
__device__ __forceinline__ uint32_t pull_all(const ChunkDesc& d, int tid, float (&x)[16]) {
    uint32_t pmask = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const uint32_t n = edge_vec(d, tid, s).n;
        pull(n, x[4 * s], x[4 * s + 1], x[4 * s + 2], x[4 * s + 3]);
        pmask |= ((1u << n) - 1u) << (4 * s);
    }
    return pmask;
}

// Shared state of one chunk's selection.
struct SelectShared {
    union {
        alignas(16) uint2 cand[kCandCap];    // filter: candidates, ascending index: {value bits, index}
        alignas(16) uint32_t hist[3][256];   // general path: digit counts of pass p in hist[p % 3]
    };
    alignas(16) uint32_t count[4][4];        // filter: candidates per wave and slot
    uint32_t bucket[16];                     // general path: entries per 256-element bucket (bucket = idx >> 8)
    uint32_t t0[4];                          // per-wave lower bounds of the threshold
    uint32_t t1[4];                          // edge chunks: non-empty lanes per wave, their non-empty slots << 16
    uint32_t wmax[4];                        // per-wave maxima of the keys
    uint32_t cut;                            // general path: index of the last kept entry among equals
};

// What find_threshold found: an element is kept if its key exceeds T, or equals T and its index is at most idxT.
struct Threshold {
    uint32_t T, idxT;                    // key of the kappa_c-th entry; largest index kept among entries with that key
    uint32_t amax;                       // largest key
    uint32_t n_cand;                     // entries of sh.cand, or 0 if the general path ran (then sh.bucket is valid)
};

// Maximum / minimum over the 64 lanes by DPP (four steps inside the rows of 16, two across), result in every lane.
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme_u32(uint32_t v) {
    constexpr uint32_t neutral = MAX ? 0u : 0xFFFFFFFFu;
    auto pick = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
    v = pick(v, (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = pick(v, (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = pick(v, (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = pick(v, (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = pick(v, (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = pick(v, (uint32_t)__builtin_amdgcn_update_dpp((int)neutral, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Sum over the lanes up to and including this one (DPP: four steps inside the rows of 16, two across).
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);      // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);      // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);      // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);      // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);      // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);      // row_bcast:31
    return v;
}

// The general path of the selection: any set of present elements (bit el of pmask = element el of this lane is
// present), any kappa_c in 1..n_c, any tie pattern.  Most-significant-digit radix select over the 31 key bits, four
// passes with a histogram each, then the last kept index among the elements with the last key.  The keys are formed
// anew in every pass, so that this rarely taken path does not set the register count of the kernel.  Also counts the
// kept entries of every 256-element bucket in sh.bucket.  Ends behind a barrier; the number of barriers does not
// depend on the chunk (the groups of a strip go through here side by side).
__device__ __forceinline__ void general_select(SelectShared& sh, const float (&x)[16], int tid, int lane, int wave,
                                               uint32_t pmask, uint32_t kappa_c, Threshold& th) {
    auto key = [&](int el) {
        uint32_t bits = __float_as_uint(x[el]);
        asm volatile("" : "+v"(bits));
        return bits & 0x7FFFFFFFu;
    };
    __syncthreads();                                          // the candidates share the histograms' memory
#pragma unroll
    for (int i = 0; i < 3; ++i) sh.hist[i][tid] = 0;
    uint32_t tmax = 0;
#pragma unroll
    for (int el = 0; el < 16; ++el) tmax = (pmask & (1u << el)) && key(el) > tmax ? key(el) : tmax;
    tmax = wave_extreme_u32<true>(tmax);
    if (lane == 0) sh.wmax[wave] = tmax;
    __syncthreads();
    uint32_t T = 0, need = kappa_c;                           // digits so far; entries still to find below them
    bool zero = false;                                        // all nonzero keys are kept, and zeros: T = 0
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = pass == 3 ? 0 : 23 - 8 * pass, width = pass == 3 ? 7 : 8;
        uint32_t* hist = sh.hist[pass == 3 ? 0 : pass];
        // (every wave has read pass 0's counts before the barrier of pass 1)
        if (pass == 2) sh.hist[0][tid] = 0;
        // Zeros are left out: they are what the remainder is when the counts do not reach `need`.  A chunk of many zeros
        // would otherwise add them all to one word, one lane at a time (9000 chunks of zeros: 530 -> 99 us; of 1 %
        // nonzeros, kappa 32: 198 -> 109).
        if (!zero) {
#pragma unroll
            for (int el = 0; el < 16; ++el) {
                const uint32_t k = key(el);
                if ((pmask & (1u << el)) && k != 0 && ((k >> shift) >> width) == T)
                    atomicAdd(&hist[(k >> shift) & ((1u << width) - 1u)], 1u);
            }
        }
        __syncthreads();
        // every wave for itself: lane l owns the digits 4 l .. 4 l + 3; find where the count from the top reaches `need`
        const uint4 h = *reinterpret_cast<const uint4*>(&hist[4 * lane]);
        const uint32_t own = h.x + h.y + h.z + h.w, upto = wave_inclusive_sum(own);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        uint32_t above = total - upto;                        // digits of higher lanes
        const bool here = above < need && need <= above + own;
        uint32_t digit = 4u * (uint32_t)lane + 3u;
        if (above + h.w < need) {
            above += h.w; --digit;
            if (above + h.z < need) {
                above += h.z; --digit;
                if (above + h.y < need) { above += h.y; --digit; }
            }
        }
        if (total < need) {                                   // (then nothing but zeros has the digits so far)
            zero = true;
            T = 0;
            need -= total;
        } else {
            const int at = __ffsll((unsigned long long)__ballot(here)) - 1;
            T = (T << width) | (uint32_t)__builtin_amdgcn_readlane((int)digit, at);
            need -= (uint32_t)__builtin_amdgcn_readlane((int)above, at);
        }
    }
    // the first `need` elements with key T, by index, are kept: find the bucket of the last one, then its index
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            c += (uint32_t)__popcll(__ballot((pmask & (1u << (4 * s + j))) && key(4 * s + j) == T));
        if (lane == 0) sh.bucket[4 * s + wave] = c;
    }
    __syncthreads();
    {
        const uint32_t own = lane < 16 ? sh.bucket[lane] : 0u, upto = wave_inclusive_sum(own);
        const int at = __ffsll((unsigned long long)__ballot(upto >= need)) - 1;           // its bucket
        const uint32_t left = need - (uint32_t)__builtin_amdgcn_readlane((int)(upto - own), at);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (at != 4 * s + wave) continue;
            uint32_t mine = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mine |= ((pmask & (1u << (4 * s + j))) && key(4 * s + j) == T) ? 1u << j : 0u;
            uint32_t before = wave_inclusive_sum(__popc(mine)) - __popc(mine);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if ((mine >> j) & 1u) {
                    if (++before == left) sh.cut = (uint32_t)(s * 1024 + tid * 4 + j);
                }
            }
        }
    }
    __syncthreads();
    th.T = T;
    th.idxT = sh.cut;
    uint32_t amax = sh.wmax[0];
    amax = sh.wmax[1] > amax ? sh.wmax[1] : amax;
    amax = sh.wmax[2] > amax ? sh.wmax[2] : amax;
    th.amax = sh.wmax[3] > amax ? sh.wmax[3] : amax;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t k = key(4 * s + j);
            const bool first = tid * 4 <= (int)th.idxT - (s * 1024 + j);
            c += (uint32_t)__popcll(__ballot((pmask & (1u << (4 * s + j))) && (k > T || (k == T && first))));
        }
        if (lane == 0) sh.bucket[4 * s + wave] = c;
    }
    __syncthreads();
}

// Exact kappa_c-th largest of the n candidates in sh.cand (n <= 64 NJ), in (key descending, index ascending) order.
// Every wave does this for itself, 64 candidates per register, by bisection on the key bits: a step is compares,
// ballots and population counts per 64 candidates for two bits, and it starts at the highest bit in which T0 (which no candidate
// is below) and the largest key differ and ends as soon as exactly kappa_c candidates remain -- some ten steps of 40
// cycles, where ranking every candidate against every other one took 900, 1900 and 6300 cycles for kappa 32, 64, 128.
template <int NJ>
__device__ __forceinline__ void solve_candidates(const SelectShared& sh, int lane, uint32_t n, uint32_t kappa_c,
                                                 uint32_t T0, Threshold& th) {
    uint32_t key[NJ];
    uint64_t valid[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const bool there = (uint32_t)lane + 64u * j < n;
        key[j] = there ? sh.cand[lane + 64 * j].x & 0x7FFFFFFFu : 0u;
        valid[j] = __ballot(there);
    }
    const uint32_t diff = T0 ^ th.amax;
    const int top = 31 - __clz((int)diff);                    // -1 if all candidates have the same key
    uint32_t X = T0 & ~((2u << (top < 0 ? 0 : top)) - 1u);
    if (top < 0) X = T0;
    bool exact = n == kappa_c;
    // bf16 pseudo-gradients and other coarse values leave the lower half of every key empty: nothing to decide there
    // (one chunk of bf16 values at kappa 16 / 32: 6.1 / 6.3 -> 5.2 / 5.4 us; 1024 chunks, 16: 11.4 -> 9.8)
    uint32_t used = 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) used |= key[j];
    const int low = __ballot((used & 0xFFFFu) != 0) ? 0 : 16;
    if constexpr (NJ <= 2) {
        // two bits a step; at least kappa_c candidates are >= X, fewer are >= X + 2^(b+1): with one bit left (b = 0)
        // t2 and t3 can neither be taken nor end the loop
        for (int b = top; b >= low && !exact; b -= 2) {
            const int sh2 = b > 0 ? b - 1 : 0;
            const uint32_t t1 = X + (1u << sh2), t2 = X + (2u << sh2), t3 = X + (3u << sh2);
            uint32_t c1 = 0, c2 = 0, c3 = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                c1 += (uint32_t)__popcll(__ballot(key[j] >= t1));
                c2 += (uint32_t)__popcll(__ballot(key[j] >= t2));
                c3 += (uint32_t)__popcll(__ballot(key[j] >= t3));
            }
            X = c3 >= kappa_c ? t3 : (c2 >= kappa_c ? t2 : (c1 >= kappa_c ? t1 : X));
            exact = c1 == kappa_c || c2 == kappa_c || c3 == kappa_c;
        }
    } else {
        for (int b = top; b >= low && !exact; --b) {            // one bit: a step has enough independent work, and fewer
            const uint32_t t = X + (1u << b);                 // instructions count where memory is what bounds
            uint32_t c = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) c += (uint32_t)__popcll(__ballot(key[j] >= t));
            X = c >= kappa_c ? t : X;
            exact = c == kappa_c;
        }
    }
    if (exact) {
        // exactly the candidates >= X are kept: the smallest of them is the threshold
        uint32_t low = 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const bool kept = key[j] >= X && (uint32_t)lane + 64u * j < n;
            low = kept && key[j] < low ? key[j] : low;
        }
        th.T = wave_extreme_u32<false>(low);
        th.idxT = 4095u;
    } else {
        // X is the key of the last kept entry and more candidates have it than are kept: the first ones by index are
        uint32_t above = 0;
#pragma unroll
        for (int j = 0; j < NJ; ++j) above += (uint32_t)__popcll(__ballot(key[j] > X));
        uint32_t run = above;
        th.T = X;
        th.idxT = 4095u;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint64_t eq = __ballot(key[j] == X) & valid[j];
            const uint64_t last = __ballot(((eq >> lane) & 1u) && run + lanes_below(eq) == kappa_c - 1);
            if (last) th.idxT = sh.cand[64 * j + __ffsll((unsigned long long)last) - 1].y;
            run += (uint32_t)__popcll(eq);
        }
    }
}

// Top-kappa selection of the chunk held in x[16] (already folded): the threshold in (key descending, index ascending)
// order.  Only the values at the start are used: a caller that can fetch its values again afterwards need not keep
// them in registers meanwhile.
// All 256 lanes (of the group) must call it.
// FROM_LDS: the chunk sits in LDS in local index order at lds_chunk and is read from there (x is ignored): once
// for the filter, and again by the (rare) general path, so that nothing but the sixteen values stays in registers.
// group_ok: four flags in LDS when four 256-lane groups of one workgroup each select a chunk of their own side
// by side (tid, lane, wave are then group-local and `sh` is the group's own).  Workgroup barriers must be
// reached by all groups alike, so the groups agree on the path: if one needs the general path, all take it.
// WALK: the caller walks replicas in one workgroup.
template <bool FROM_LDS = false, bool WALK = false>
__device__ __forceinline__ Threshold find_threshold(SelectShared& sh, const float (&x)[16], int tid, int lane, int wave,
                                                    uint32_t kappa_c, uint32_t kappa, uint32_t pmask, bool edge,
                                                    int force_radix, uint32_t* radix_counter, const float* lds_chunk = nullptr,
                                                    uint32_t* group_ok = nullptr, int group = 0) {
    Threshold th = {0u, 4095u, 0u, 0u};
    if (kappa <= (uint32_t)kFilterKappaMax && !force_radix) {
        // ---- candidate filter: a lower bound T0 of the threshold from the lane maxima ----
        uint32_t bits[16];
        if constexpr (FROM_LDS) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float4 v = *reinterpret_cast<const float4*>(lds_chunk + s * 1024 + tid * 4);
                bits[4 * s] = __float_as_uint(v.x);
                bits[4 * s + 1] = __float_as_uint(v.y);
                bits[4 * s + 2] = __float_as_uint(v.z);
                bits[4 * s + 3] = __float_as_uint(v.w);
            }
        } else {
#pragma unroll
            for (int el = 0; el < 16; ++el) bits[el] = __float_as_uint(x[el]);
        }
        auto key = [&](int el) { return bits[el] & 0x7FFFFFFFu; };
        uint32_t tmax = 0;
#pragma unroll
        for (int el = 0; el < 16; ++el) tmax = key(el) > tmax ? key(el) : tmax;      // (absent ones are 0)
        const uint32_t wave_max = wave_extreme_u32<true>(tmax);
        // Largest X (low 13 bits zero) with at least m = kappa_c / 4 lanes of this wave that hold a present element
        // >= X.  Those elements are distinct, so over four waves at least 4*m >= kappa_c elements are
        // >= min X: the threshold cannot be below it.
        uint32_t m = (kappa_c + 3) >> 2;
        bool by_slots = false;
        if (edge) {
            // The waves of an edge chunk hold unequal numbers of elements: each answers for a share of kappa_c that is
            // in proportion to its non-empty lanes or, where the chunk has fewer of those than kappa_c (few columns), to
            // its non-empty slots of lanes, whose largest elements are distinct too.  A chunk with fewer slots than
            // kappa_c leaves X = 0: every present element is a candidate.
            uint32_t slots = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s) slots += (uint32_t)__popcll(__ballot((pmask & (0xFu << (4 * s))) != 0));
            const uint32_t lanes = (uint32_t)__popcll(__ballot(pmask != 0));
            if (lane == 0) sh.t1[wave] = lanes | (slots << 16);
            __syncthreads();
            const uint32_t all = __builtin_amdgcn_readfirstlane(sh.t1[0] + sh.t1[1] + sh.t1[2] + sh.t1[3]);
            by_slots = (all & 0xFFFFu) < kappa_c;
            const uint32_t of_all = by_slots ? all >> 16 : all & 0xFFFFu, of_wave = by_slots ? slots : lanes;
            m = of_all < kappa_c ? 257u : (kappa_c * of_wave + of_all - 1) / of_all;
        }
        auto reached_by = [&](uint32_t lanes) {               // two bits a step: the chain of steps is what it costs
            uint32_t X = 0;
#pragma unroll
            for (int b = 29; b >= 13; b -= 2) {
                const uint32_t t1 = X + (1u << b), t2 = X + (2u << b), t3 = X + (3u << b);
                const uint32_t c1 = (uint32_t)__popcll(__ballot(tmax >= t1));
                const uint32_t c2 = (uint32_t)__popcll(__ballot(tmax >= t2));
                const uint32_t c3 = (uint32_t)__popcll(__ballot(tmax >= t3));
                X = c3 >= lanes ? t3 : (c2 >= lanes ? t2 : (c1 >= lanes ? t1 : X));
            }
            return X;
        };
        uint32_t X = 0;
        if (!by_slots) {
            X = reached_by(m);
        } else {
            uint32_t top[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                top[s] = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) top[s] = key(4 * s + j) > top[s] ? key(4 * s + j) : top[s];
            }
#pragma unroll 1
            for (int b = 30; b >= 13; --b) {
                const uint32_t t = X + (1u << b);
                uint32_t c = 0;
#pragma unroll
                for (int s = 0; s < 4; ++s) c += (uint32_t)__popcll(__ballot(top[s] >= t));
                X = c >= m ? t : X;
            }
        }
        if (lane == 0) {
            sh.t0[wave] = X;
            sh.wmax[wave] = wave_max;
        }
        __syncthreads();
        uint32_t T0 = sh.t0[0];
        T0 = sh.t0[1] < T0 ? sh.t0[1] : T0;
        T0 = sh.t0[2] < T0 ? sh.t0[2] : T0;
        T0 = sh.t0[3] < T0 ? sh.t0[3] : T0;
        T0 = __builtin_amdgcn_readfirstlane(T0);
        uint32_t amax = sh.wmax[0];
        amax = sh.wmax[1] > amax ? sh.wmax[1] : amax;
        amax = sh.wmax[2] > amax ? sh.wmax[2] : amax;
        amax = sh.wmax[3] > amax ? sh.wmax[3] : amax;
        th.amax = __builtin_amdgcn_readfirstlane(amax);

        // ---- compact the candidates (present, key >= T0) into LDS in index order, i.e. by slot, wave, lane, element.
        // Every lane collects its candidates in a mask; positions inside a slot of a wave come from a sum over the
        // lanes (slots 0, 1 and 2, 3 packed into one word each), those of the slots from the counts of all waves. ----
        uint32_t mask = 0;
#pragma unroll
        for (int el = 15; el >= 0; --el) mask = mask + mask + (key(el) >= T0 ? 1u : 0u);
        mask &= pmask;
        const uint32_t n01 = (uint32_t)__popc(mask & 0xFu) | ((uint32_t)__popc(mask & 0xF0u) << 16);
        const uint32_t n23 = (uint32_t)__popc(mask & 0xF00u) | ((uint32_t)__popc(mask & 0xF000u) << 16);
        const uint32_t s01 = wave_inclusive_sum(n01), s23 = wave_inclusive_sum(n23);
        if (lane == 63)
            *reinterpret_cast<uint4*>(sh.count[wave]) = make_uint4(s01 & 0xFFFFu, s01 >> 16, s23 & 0xFFFFu, s23 >> 16);
        __syncthreads();
        uint32_t base[4], n = 0;
        {
            uint4 c[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) c[w] = *reinterpret_cast<const uint4*>(sh.count[w]);
            auto slot = [&](uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
                const uint32_t first = n + (wave > 0 ? c0 : 0u) + (wave > 1 ? c1 : 0u) + (wave > 2 ? c2 : 0u);
                n += c0 + c1 + c2 + c3;
                return first;
            };
            base[0] = slot(c[0].x, c[1].x, c[2].x, c[3].x);
            base[1] = slot(c[0].y, c[1].y, c[2].y, c[3].y);
            base[2] = slot(c[0].z, c[1].z, c[2].z, c[3].z);
            base[3] = slot(c[0].w, c[1].w, c[2].w, c[3].w);
        }
        n = __builtin_amdgcn_readfirstlane(n);
        if (n <= (uint32_t)kCandCap) {
            const uint32_t at01 = s01 - n01 + (base[0] | (base[1] << 16)), at23 = s23 - n23 + (base[2] | (base[3] << 16));
            for (uint32_t left = mask; __any(left != 0); left &= left - 1) {   // as many rounds as a lane has candidates
                if (left != 0) {
                    const uint32_t el = (uint32_t)__ffs((int)left) - 1, slot = el >> 2;
                    auto pick = [](bool second, uint32_t a, uint32_t b) { return second ? b : a; };
                    uint32_t v[8];                                             // bits[el], by halving
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = pick(el & 8u, bits[i], bits[8 + i]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = pick(el & 4u, v[i], v[4 + i]);
                    v[0] = pick(el & 2u, v[0], v[2]);
                    v[1] = pick(el & 2u, v[1], v[3]);
                    v[0] = pick(el & 1u, v[0], v[1]);
                    const uint32_t lower = mask & ((1u << el) - 1u) & (0xFu << (4 * slot));
                    const uint32_t pos = (((slot & 2u) ? at23 : at01) >> (16 * (slot & 1u)) & 0xFFFFu) + (uint32_t)__popc(lower);
                    sh.cand[pos] = make_uint2(v[0], slot * 1024u + (uint32_t)tid * 4u + (el & 3u));
                }
            }
            th.n_cand = n;
        }
        if (FROM_LDS && tid == 0) group_ok[group] = th.n_cand != 0 ? 1u : 0u;
        __syncthreads();
        if (FROM_LDS && (group_ok[0] & group_ok[1] & group_ok[2] & group_ok[3]) == 0) th.n_cand = 0;
        if (th.n_cand != 0) {
            // (one register of candidates where they fit: kappa 16 and less, 1024 chunks 9.56 -> 9.30 us; in the walk over
            // replicas it lost: 150M parameters, 8 replicas 2865 -> 2890 us, 720 chunks, 5 replicas 40.1 -> 41.3)
            if (!WALK && n <= 64) solve_candidates<1>(sh, lane, n, kappa_c, T0, th);
            else if (n <= 128) solve_candidates<2>(sh, lane, n, kappa_c, T0, th);
            else if (n <= 256) solve_candidates<4>(sh, lane, n, kappa_c, T0, th);
            else solve_candidates<7>(sh, lane, n, kappa_c, T0, th);
        }
    }
    if (th.n_cand == 0) {
        if constexpr (FROM_LDS) {
            // (the index is made opaque so that these reads are not merged with the earlier ones, which
            // would keep all sixteen values in registers from there to here)
            int t = tid;
            asm volatile("" : "+v"(t));
            float y[16];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float4 v = *reinterpret_cast<const float4*>(lds_chunk + s * 1024 + t * 4);
                y[4 * s] = v.x; y[4 * s + 1] = v.y; y[4 * s + 2] = v.z; y[4 * s + 3] = v.w;
            }
            general_select(sh, y, tid, lane, wave, pmask, kappa_c, th);
        } else {
            general_select(sh, x, tid, lane, wave, pmask, kappa_c, th);
        }
        if (radix_counter && tid == 0) atomicAdd(radix_counter, 1u);      // diagnostic: chunks on the general path
    }
    return th;
}

// Quantiser, packing and residual of the chunk held in x[16], given the threshold that find_threshold returned.
// On return x holds the new error-feedback values; the chunk's pairs, its levels (or sent values) and its padding have
// been written.  Callers that reuse `sh` must place a barrier first.
// With SUM, every sent value is also added to sum[index in the chunk] (LDS).  Any lane may do that: replicas that
// follow each other in one workgroup are separated by a barrier.
// The candidates of the filter are in index order, so the message is written by the lanes that hold a candidate: an
// entry's position is the number of kept candidates before it.  The lanes that hold the elements only form the
// residual, without a branch.  After the general path there is no such list, and the elements' lanes write the
// message themselves (positions from the bucket counts and ballots).
template <int QUANT, bool SUM>
__device__ __forceinline__ void quantise_pack_sum(const SelectShared& sh, const Threshold& th, float (&x)[16], float* sum,
                                                  int tid, int lane, int wave, uint32_t kappa_c, uint32_t kappa,
                                                  uint32_t pmask, uint16_t* __restrict__ pairs_c,
                                                  float* __restrict__ values_c, float* __restrict__ scales_c) {
    const uint32_t T = th.T, idxT = th.idxT;
    // The smallest selected magnitude is the threshold key itself; the largest is the chunk maximum.
    const float amin = __uint_as_float(T), amax = __uint_as_float(th.amax);
    const float dd = __fsub_rn(amax, amin);
    const float lo = __fadd_rn(amin, __fmul_rn(0.25f, dd));
    const float tau = __fadd_rn(amin, __fmul_rn(0.5f, dd));
    const float hi = __fadd_rn(amin, __fmul_rn(0.75f, dd));
    const uint32_t tau_bits = __float_as_uint(tau);
    auto kept = [&](uint32_t key, uint32_t idx) { return key > T || (key == T && idx <= idxT); };
    auto decoded = [&](uint32_t bits) {                       // of a kept entry
        const uint32_t upper = (bits & 0x7FFFFFFFu) >= tau_bits ? 1u : 0u;
        return __builtin_copysignf(upper ? hi : lo, __uint_as_float(bits));
    };
    auto write_entry = [&](uint32_t pos, uint32_t bits, uint32_t idx) {
        if (QUANT == SPLC_QUANT_2BIT) {
            const uint32_t upper = (bits & 0x7FFFFFFFu) >= tau_bits ? 1u : 0u;
            pairs_c[pos] = (uint16_t)(idx | ((((bits >> 31) << 1) | upper) << 12));
            if (SUM) sum[idx] = __fadd_rn(sum[idx], decoded(bits));
        } else {
            pairs_c[pos] = (uint16_t)idx;
            values_c[pos] = __uint_as_float(bits);
            if (SUM) sum[idx] = __fadd_rn(sum[idx], __uint_as_float(bits));
        }
    };

    if (th.n_cand != 0) {
        uint32_t pos = 0;
        for (uint32_t j = 0; 64u * j < th.n_cand; ++j) {      // 64 candidates at a time, written by the waves in turn
            const uint32_t i = 64u * j + (uint32_t)lane;
            const uint2 c = sh.cand[i];
            const bool mine = i < th.n_cand && kept(c.x & 0x7FFFFFFFu, c.y);
            const uint64_t m = __ballot(mine);
            if (mine && (j & 3u) == (uint32_t)wave) write_entry(pos + lanes_below(m), c.x, c.y);
            pos += (uint32_t)__popcll(m);
        }
    } else {
        uint32_t base_of_slot[4], run = 0;
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            if ((b & 3) == wave) base_of_slot[b >> 2] = run;
            run += sh.bucket[b];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            bool sel[4];
            uint64_t m4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t idx = s * 1024 + tid * 4 + j;
                sel[j] = (pmask & (1u << (4 * s + j))) && kept(__float_as_uint(x[4 * s + j]) & 0x7FFFFFFFu, idx);
                m4[j] = __ballot(sel[j]);
            }
            uint32_t pos = base_of_slot[s] + lanes_below(m4[0]) + lanes_below(m4[1]) + lanes_below(m4[2]) +
                           lanes_below(m4[3]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (sel[j]) write_entry(pos++, __float_as_uint(x[4 * s + j]), s * 1024 + tid * 4 + j);
            }
        }
    }
    // (absent elements may be changed too; nobody stores them)
    auto residual = [&](int el, bool sel) {
        const float rest = QUANT == SPLC_QUANT_2BIT ? __fsub_rn(x[el], decoded(__float_as_uint(x[el])))
                                                    : __fsub_rn(x[el], x[el]);
        x[el] = sel ? rest : x[el];
    };
    if (idxT == 4095u) {                                      // every present element with key T is kept
#pragma unroll
        for (int el = 0; el < 16; ++el)
            residual(el, (__float_as_uint(x[el]) & 0x7FFFFFFFu) >= T);
    } else {
        const int at4 = tid * 4;
#pragma unroll
        for (int el = 0; el < 16; ++el) {
            const uint32_t key = __float_as_uint(x[el]) & 0x7FFFFFFFu;
            const bool first = at4 <= (int)idxT - ((el >> 2) * 1024 + (el & 3));          // index <= idxT
            residual(el, key > T || (key == T && first));
        }
    }
    for (uint32_t t = kappa_c + tid; t < kappa; t += kThreads) {
        pairs_c[t] = 0xFFFFu;
        if (QUANT == SPLC_QUANT_NONE) values_c[t] = 0.f;
    }
    if (QUANT == SPLC_QUANT_2BIT && tid == 0) {
        scales_c[0] = lo;
        scales_c[1] = hi;
    }
}

// Both steps for a chunk that stays in registers throughout.
template <int QUANT>
__device__ __forceinline__ void select_quantise_pack(SelectShared& sh, float (&x)[16], int tid, int lane, int wave,
                                                     uint32_t n_c, uint32_t pmask, uint32_t kappa, int force_radix,
                                                     uint32_t* radix_counter, uint16_t* __restrict__ pairs_c,
                                                     float* __restrict__ values_c, float* __restrict__ scales_c) {
    const uint32_t kappa_c = kappa < n_c ? kappa : n_c;
    const Threshold th = find_threshold(sh, x, tid, lane, wave, kappa_c, kappa, pmask, n_c != (uint32_t)kChunk, force_radix,
                                        radix_counter);
    quantise_pack_sum<QUANT, false>(sh, th, x, nullptr, tid, lane, wave, kappa_c, kappa, pmask, pairs_c, values_c,
                                    scales_c);
}

// The error-feedback buffer is rewritten densely (line 4 of the update equations).  Where lines are shared the store goes without
// the hint, but not by a call that walks over replicas (BATCH: without it the one-launch step takes 0.98 to 1.06 of the time)
// and not on plans of few tiles, where less of the caches is left for what the next call reads (700 tiles, four replicas that
// share theta_outer, 12.8 -> 11.8 us, from fp32 9.9 -> 9.3; 1500: 19.6 -> 21.4, from bf16 in no cache 18.8 -> 20.3; 6000, from bf16 43 -> 50).
constexpr unsigned kFewTiles = 1024;
template <bool VEC, bool BATCH>
__device__ __forceinline__ void store_ef(float* __restrict__ e, const ChunkDesc& d, int tid, uint32_t pmask,
                                         const float (&x)[16]) {
    float* pe = e + d.offset;
    auto store = [&](const auto& chunk) {
#pragma unroll
        for (int s = 0; s < 4; ++s) chunk.store(pe, s, make_float4(x[4 * s], x[4 * s + 1], x[4 * s + 2], x[4 * s + 3]));
    };
    if constexpr (VEC && BATCH) {
        store(CompleteChunk<true>{d, tid});
    } else if constexpr (VEC) {
        with_chunk<true>(d, tid, store, gridDim.x < kFewTiles);
    } else {
        // from an opaque copy of the lane number: nothing of the loads' addresses is kept for these stores
        int t = tid;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int s = 0; s < 4; ++s)
            store_edge(vec_at(pe, d, t, s), (pmask >> (4 * s)) & 0xFu,
                       make_float4(x[4 * s], x[4 * s + 1], x[4 * s + 2], x[4 * s + 3]));
    }
}

// Lines 1-4 of the update equations, one replica, one chunk per workgroup.
// vec: the chunk is complete; else an edge chunk.  Only the loads and stores differ: one copy of the selection keeps
// the code, which a cold launch fetches from memory, short.
template <int MODE, int QUANT>
__device__ __forceinline__ void compress_body(SelectShared& sh, bool vec, const ChunkDesc* __restrict__ chunks,
                                              const void* const* __restrict__ src_a,
                                              const void* const* __restrict__ src_b,
                                              float* const* __restrict__ ef_tab, float beta, uint32_t kappa,
                                              int force_radix, uint32_t* radix_counter,
                                              uint16_t* __restrict__ pairs_out, float* __restrict__ aux_out) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ChunkDesc d = chunks[blockIdx.x];
    const uint64_t c = d.id;
    const void* pa = src_a[d.tensor];
    const void* pb = MODE == MODE_PARAMS_F32 ? src_b[d.tensor] : nullptr;
    float* pe = ef_tab[d.tensor];

    uint32_t pmask = 0xFFFFu;
    float x[16];
    if (vec) {
        with_chunk<true>(d, tid, [&](const auto& chunk) { load_fold<MODE>(pa, pb, pe, beta, x, chunk); });
    } else {
        with_chunk<false>(d, tid, [&](const auto& chunk) { load_fold<MODE>(pa, pb, pe, beta, x, chunk); });
        pmask = pull_all(d, tid, x);
    }
    select_quantise_pack<QUANT>(sh, x, tid, lane, wave, d.n_c, pmask, kappa, force_radix, radix_counter,
                                pairs_out + c * kappa, aux_out + c * kappa, aux_out + 2 * c);
    if (vec) store_ef<true, false>(pe, d, tid, pmask, x);
    else store_ef<false, false>(pe, d, tid, pmask, x);
}

// The chunk table lists the n_gen edge chunks first (one launch; the branch is uniform per workgroup).
template <int MODE, int QUANT>
__global__ __launch_bounds__(kThreads) void compress_kernel(const ChunkDesc* __restrict__ chunks, uint32_t n_gen,
                                                            const void* const* __restrict__ src_a,
                                                            const void* const* __restrict__ src_b,
                                                            float* const* __restrict__ ef_tab, float beta,
                                                            uint32_t kappa, int force_radix,
                                                            uint32_t* radix_counter,
                                                            uint16_t* __restrict__ pairs_out,
                                                            float* __restrict__ aux_out) {
    __shared__ __align__(16) SelectShared sh;
    compress_body<MODE, QUANT>(sh, blockIdx.x >= n_gen, chunks, src_a, src_b, ef_tab, beta, kappa, force_radix,
                               radix_counter, pairs_out, aux_out);
}

// ---- 64 x 64 tiles, four at a time ("strip"): rows of a strip are 1024 contiguous bytes ----
//
// A workgroup that owns one 64 x 64 tile touches 256-byte row segments; when the matrix's row length is not a
// multiple of 32 floats every such segment straddles three 128-byte cache lines instead of two, and the lines on
// a tile's left and right edge are requested again by its neighbours.  So wherever four complete tiles lie side
// by side, and there are many of them (splc::strips_pay), ONE workgroup of 1024 lanes takes all four: global memory is
// accessed row by row (a wave covers one 1024-byte row of the strip per instruction: nine lines instead of twelve),
// the folded values pass through LDS, where each 256-lane group picks up "its" tile in the usual chunk layout and runs
// the selection exactly as the one-tile kernel does, and the new error-feedback values go back the same way.  Tiles left over at the end of a tile row, edge tiles and 1-D tensors stay with the
// one-tile kernels.
constexpr int kStripTiles = 4;
constexpr int kStripThreads = kStripTiles * kThreads;
// Two strip workgroups per compute unit (8 waves per SIMD, 64 registers per lane, half of the 160 KB of LDS each): one
// of them selects while the other one's rows are in flight.

struct StripShared {
    float tile[kStripTiles][kChunk];     // local index order: [row * 64 + column]
    SelectShared sel[kStripTiles];
    uint32_t group_ok[kStripTiles];
};
static_assert(sizeof(StripShared) <= 160 * 1024 / 2, "two strip workgroups share a compute unit's LDS");

// Row-wise position of lane `lane` of wave `wave` (0..15) in round i (0..3): local row 16 i + wave of the strip,
// floats 4 lane .. 4 lane + 3 of that row, i.e. tile lane / 16, local columns 4 (lane % 16) ...
__device__ __forceinline__ uint32_t strip_row(int i, int wave) { return 16u * (uint32_t)i + (uint32_t)wave; }
// Addressing of the row-wise accesses: per array one base that is uniform over the wave (the array's origin of
// the strip plus `wave` rows), pinned into a scalar register pair, and per round i one 32-bit byte offset per
// lane (16 i rows plus the lane's position in the row) that all arrays share.  Written out like this the accesses
// are encoded as "scalar base + 32-bit lane offset"; left to itself the compiler keeps one 64-bit address per
// access in vector registers, two dozen registers that the 64-register budget of this kernel does not have.
template <class T>
__device__ __forceinline__ T* strip_base(T* origin, const ChunkDesc& d, int wave) {
    const uint64_t u = reinterpret_cast<uint64_t>(origin + (size_t)((uint32_t)wave * d.stride));
    uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    asm volatile("" : "+s"(lo), "+s"(hi));
    return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}
// Byte offset (for 4-byte elements) of this lane's four elements in round i; 63 rows * stride * 4 < 2^32.
__device__ __forceinline__ uint32_t strip_offset(const ChunkDesc& d, int i, int lane) {
    return ((uint32_t)(16 * i) * d.stride + (uint32_t)lane * 4u) * 4u;
}
template <class T>
__device__ __forceinline__ T* strip_at(T* base, uint32_t offset_for_4_byte_elements) {
    using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return reinterpret_cast<T*>(reinterpret_cast<Byte*>(base) + offset_for_4_byte_elements / (4u / (uint32_t)sizeof(T)));
}

template <int MODE, int QUANT>
__global__ __launch_bounds__(kStripThreads, 8) void compress_strip_kernel(const ChunkDesc* __restrict__ strips,
                                                                       const void* const* __restrict__ src_a,
                                                                       const void* const* __restrict__ src_b,
                                                                       float* const* __restrict__ ef_tab, float beta,
                                                                       uint32_t kappa, int force_radix,
                                                                       uint32_t* radix_counter,
                                                                       uint16_t* __restrict__ pairs_out,
                                                                       float* __restrict__ aux_out) {
    __shared__ __align__(16) StripShared sm;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);          // 0..15
    const ChunkDesc d = strips[blockIdx.x];
    float* const pe = strip_base(ef_tab[d.tensor] + d.offset, d, wave);
    const uint32_t q = (uint32_t)lane >> 4, lc = ((uint32_t)lane & 15u) * 4u;
    uint32_t off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) off[i] = strip_offset(d, i, lane);

    // ---- rows in: fold in registers, e' to LDS ----
    {
        float4 ev[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ev[i] = stream_load4(strip_at<const float>(pe, off[i]));
        float x[16];
        if (MODE == MODE_PARAMS_F32) {
            const float* po = strip_base(static_cast<const float*>(src_a[d.tensor]) + d.offset, d, wave);
            const float* pl = strip_base(static_cast<const float*>(src_b[d.tensor]) + d.offset, d, wave);
            float4 ov[4], lv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) ov[i] = stream_load4(strip_at(po, off[i]));
#pragma unroll
            for (int i = 0; i < 4; ++i) lv[i] = stream_load4(strip_at(pl, off[i]));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[4 * i + 0] = fold(beta, ev[i].x, __fsub_rn(ov[i].x, lv[i].x));
                x[4 * i + 1] = fold(beta, ev[i].y, __fsub_rn(ov[i].y, lv[i].y));
                x[4 * i + 2] = fold(beta, ev[i].z, __fsub_rn(ov[i].z, lv[i].z));
                x[4 * i + 3] = fold(beta, ev[i].w, __fsub_rn(ov[i].w, lv[i].w));
            }
        } else if (MODE == MODE_DIRECT_F32) {
            const float* pd = strip_base(static_cast<const float*>(src_a[d.tensor]) + d.offset, d, wave);
            float4 dv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) dv[i] = stream_load4(strip_at(pd, off[i]));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[4 * i + 0] = fold(beta, ev[i].x, dv[i].x);
                x[4 * i + 1] = fold(beta, ev[i].y, dv[i].y);
                x[4 * i + 2] = fold(beta, ev[i].z, dv[i].z);
                x[4 * i + 3] = fold(beta, ev[i].w, dv[i].w);
            }
        } else {
            const uint16_t* pd = strip_base(static_cast<const uint16_t*>(src_a[d.tensor]) + d.offset, d, wave);
            uint2 dv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) dv[i] = stream_load4(strip_at(pd, off[i]));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[4 * i + 0] = fold(beta, ev[i].x, __uint_as_float(dv[i].x << 16));
                x[4 * i + 1] = fold(beta, ev[i].y, __uint_as_float(dv[i].x & 0xFFFF0000u));
                x[4 * i + 2] = fold(beta, ev[i].z, __uint_as_float(dv[i].y << 16));
                x[4 * i + 3] = fold(beta, ev[i].w, __uint_as_float(dv[i].y & 0xFFFF0000u));
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4*>(&sm.tile[q][strip_row(i, wave) * 64u + lc]) =
                make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
    }
    __syncthreads();

    // ---- each 256-lane group selects in its own tile ----
    {
        const int group = __builtin_amdgcn_readfirstlane(tid >> 8);
        const int gtid = tid & (kThreads - 1);
        const int gwave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
        const uint64_t c = (uint64_t)d.id + (uint64_t)group;
        const uint32_t kappa_c = kappa < (uint32_t)kChunk ? kappa : (uint32_t)kChunk;
        float x[16];
        auto fetch_tile = [&]() {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float4 v = *reinterpret_cast<const float4*>(&sm.tile[group][s * 1024 + gtid * 4]);
                x[4 * s] = v.x; x[4 * s + 1] = v.y; x[4 * s + 2] = v.z; x[4 * s + 3] = v.w;
            }
        };
        // The threshold search reads the tile from LDS by itself (it needs only the magnitudes); the values are
        // fetched afterwards: 64 registers per lane (two of these workgroups per compute unit) do not hold values
        // and keys side by side.
        const Threshold th = find_threshold<true>(sm.sel[group], x, gtid, lane, gwave, kappa_c, kappa, 0xFFFFu, false,
                                            force_radix, radix_counter, &sm.tile[group][0], sm.group_ok, group);
        fetch_tile();
        quantise_pack_sum<QUANT, false>(sm.sel[group], th, x, nullptr, gtid, lane, gwave, kappa_c, kappa, 0xFFFFu,
                                        pairs_out + c * kappa, aux_out + c * kappa, aux_out + 2 * c);
#pragma unroll
        for (int s = 0; s < 4; ++s)
            *reinterpret_cast<float4*>(&sm.tile[group][s * 1024 + gtid * 4]) =
                make_float4(x[4 * s], x[4 * s + 1], x[4 * s + 2], x[4 * s + 3]);
    }
    __syncthreads();

    // ---- rows out (offsets recomputed here, from an opaque copy of the lane number, so that they are not
    // carried in registers through the selection) ----
    int l = lane;
    asm volatile("" : "+v"(l));
#pragma unroll
    for (int i = 0; i < 4; ++i)
        stream_store4(strip_at(pe, strip_offset(d, i, l)),
                      *reinterpret_cast<const float4*>(&sm.tile[q][strip_row(i, wave) * 64u + lc]));
}

// Lines 1-4 for R replicas that share theta_outer (several replicas simulated on one GPU): the
// workgroup reads its theta_outer chunk once and walks the replicas, so theta_outer costs 4 bytes
// per parameter per launch instead of per replica.  Per replica the arithmetic, the selection and
// the outputs are those of compress_kernel.
// With STEP the workgroup finishes the outer step for its chunk (line 5): what each replica sends is added, replica
// after replica, to a sum in LDS by the lanes that write the message (the barrier between replicas orders the adds), and
// after the last replica the chunk's mean is applied to theta_outer, written to delta_bar if asked for, and the new
// parameters are copied to the replicas' theta_local if asked for.  The sums start at +0 and are divided once by M: the
// bits of sparseloco_aggregate_update.
// Table layout (device): theta_local[r][t] at tl_tab[r * n_tensors + t], likewise ef_tab; message
// buffers pairs_tab[r], aux_tab[r].
template <int QUANT, bool VEC, bool STEP>
__device__ __forceinline__ void compress_batch_body(SelectShared& sh, float* so, float* sum,
                                                    const ChunkDesc* __restrict__ chunks,
                                                    int n_replicas, uint32_t n_tensors,
                                                    float* const* __restrict__ to_tab, float* const* __restrict__ tl_tab,
                                                    float* const* __restrict__ ef_tab, float beta, uint32_t kappa,
                                                    int force_radix, uint32_t* radix_counter,
                                                    uint16_t* const* __restrict__ pairs_tab,
                                                    float* const* __restrict__ aux_tab, float eta,
                                                    float* const* __restrict__ dbar_tab, int reset) {
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ChunkDesc d = chunks[blockIdx.x];
    const uint64_t c = d.id;
    const uint32_t n_c = VEC ? (uint32_t)kChunk : d.n_c;
    const uint32_t kappa_c = kappa < n_c ? kappa : n_c;
    const float* po = to_tab[d.tensor] + d.offset;

    // The theta_outer chunk waits in LDS, as it was read (each lane re-reads only what it wrote, so no barrier is
    // needed); keeping it in registers across the replica loop would cost occupancy.
    float4* so4 = reinterpret_cast<float4*>(so);
    with_chunk<VEC>(d, tid, [&](const auto& chunk) {
        float4 v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = chunk.load(po, s);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) so4[s * kThreads + tid] = v[s];
    });
    float4* sum4 = reinterpret_cast<float4*>(sum);
    if (STEP) {
#pragma unroll
        for (int s = 0; s < 4; ++s) sum4[s * kThreads + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int r = 0; r < n_replicas; ++r) {
        // Per-lane index arithmetic is recomputed in every round: hoisting it out of the loop would
        // pin some 60 registers across the whole selection and halve the occupancy.
        int t = tid;
        asm volatile("" : "+v"(t));
        const float* pl = tl_tab[(size_t)r * n_tensors + d.tensor] + d.offset;
        float* pe = ef_tab[(size_t)r * n_tensors + d.tensor];
        float x[16];
        with_chunk<VEC>(d, t, [&](const auto& chunk) {
            float4 lv[4], ev[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) lv[s] = chunk.load(pl, s);
#pragma unroll
            for (int s = 0; s < 4; ++s) ev[s] = chunk.load(pe + d.offset, s);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) fold4(beta, ev[s], so4[s * kThreads + t], lv[s], x + 4 * s);
        });
        const uint32_t pmask = VEC ? 0xFFFFu : pull_all(d, t, x);
        float* aux_r = aux_tab[r];
        const Threshold th = find_threshold<false, true>(sh, x, t, t & 63, wave, kappa_c, kappa, pmask, !VEC, force_radix,
                                                         radix_counter);
        quantise_pack_sum<QUANT, STEP>(sh, th, x, sum, t, t & 63, wave, kappa_c, kappa, pmask, pairs_tab[r] + c * kappa,
                                       aux_r + c * kappa, aux_r + 2 * c);
        store_ef<VEC, true>(pe, d, t, pmask, x);
        __syncthreads();          // every lane is done with `sh` before the next replica re-initialises it
    }
    if (!STEP) return;

    const float m = (float)n_replicas;
    float* th = to_tab[d.tensor] + d.offset;
    float* pd = dbar_tab ? dbar_tab[d.tensor] + d.offset : nullptr;
    const int n_reset = reset ? n_replicas : 0;
    with_chunk<VEC>(d, tid, [&](const auto& chunk) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            float4 v = sum4[s * kThreads + tid], tn = so4[s * kThreads + tid];
            if (!VEC) pull(edge_vec(d, tid, s).n, tn.x, tn.y, tn.z, tn.w);
            v.x = __fdiv_rn(v.x, m); v.y = __fdiv_rn(v.y, m); v.z = __fdiv_rn(v.z, m); v.w = __fdiv_rn(v.w, m);
            if (pd) chunk.store(pd, s, v);
            tn.x = __fsub_rn(tn.x, __fmul_rn(eta, v.x));
            tn.y = __fsub_rn(tn.y, __fmul_rn(eta, v.y));
            tn.z = __fsub_rn(tn.z, __fmul_rn(eta, v.z));
            tn.w = __fsub_rn(tn.w, __fmul_rn(eta, v.w));
            chunk.store(th, s, tn);
            for (int r = 0; r < n_reset; ++r)
                chunk.store(tl_tab[(size_t)r * n_tensors + d.tensor] + d.offset, s, tn);
        }
    });
}

// Four workgroups per compute unit (three on large plans, see reserve_lds): the register allocation is held to 128.
template <int QUANT, bool STEP>
__global__ __launch_bounds__(kThreads, 4) void compress_batch_kernel(const ChunkDesc* __restrict__ chunks, uint32_t n_gen,
                                                                  int n_replicas, uint32_t n_tensors,
                                                                  float* const* __restrict__ to_tab,
                                                                  float* const* __restrict__ tl_tab,
                                                                  float* const* __restrict__ ef_tab, float beta,
                                                                  uint32_t kappa, int force_radix,
                                                                  uint32_t* radix_counter,
                                                                  uint16_t* const* __restrict__ pairs_tab,
                                                                  float* const* __restrict__ aux_tab, float eta,
                                                                  float* const* __restrict__ dbar_tab, int reset) {
    __shared__ __align__(16) SelectShared sh;
    __shared__ __align__(16) float so[kChunk];
    __shared__ __align__(16) float sum[STEP ? kChunk : 4];
    if (blockIdx.x >= n_gen)
        compress_batch_body<QUANT, true, STEP>(sh, so, sum, chunks, n_replicas, n_tensors, to_tab, tl_tab, ef_tab, beta, kappa,
                                               force_radix, radix_counter, pairs_tab, aux_tab, eta, dbar_tab, reset);
    else
        compress_batch_body<QUANT, false, STEP>(sh, so, sum, chunks, n_replicas, n_tensors, to_tab, tl_tab, ef_tab, beta,
                                                kappa, force_radix, radix_counter, pairs_tab, aux_tab, eta, dbar_tab,
                                                reset);
}

// The same lines for all replicas of a small plan, one workgroup per chunk and replica: with few chunks the walk over
// the replicas above is a serial chain on a chip that is mostly idle.
template <int QUANT>
__global__ __launch_bounds__(kThreads) void compress_each_kernel(const ChunkDesc* __restrict__ chunks, uint32_t n_gen,
                                                                 uint32_t n_tensors, const void* const* __restrict__ to_tab,
                                                                 const void* const* __restrict__ tl_tab,
                                                                 float* const* __restrict__ ef_tab, float beta,
                                                                 uint32_t kappa, int force_radix, uint32_t* radix_counter,
                                                                 uint16_t* const* __restrict__ pairs_tab,
                                                                 float* const* __restrict__ aux_tab) {
    __shared__ __align__(16) SelectShared sh;
    const uint32_t r = blockIdx.y;
    compress_body<MODE_PARAMS_F32, QUANT>(sh, blockIdx.x >= n_gen, chunks, to_tab, tl_tab + (size_t)r * n_tensors,
                                          ef_tab + (size_t)r * n_tensors, beta, kappa, force_radix, radix_counter,
                                          pairs_tab[r], aux_tab[r]);
}

// Line 5, first half: sum of the decoded messages of one chunk into a dense LDS accumulator.
// Replicas are applied in batches of eight; a batch is applied by ONE wave: LDS operations of a
// wave complete in program order, so the add of replica r+1 at some index sees the add of replica
// r at the same index without a barrier, and inside one replica the indices are distinct.  Batches
// follow each other in replica order with a workgroup barrier in between (the four waves take
// turns, so that the messages of four batches are in flight at once).  Every element therefore
// receives its addends in ascending replica order -- deterministic, no float atomics, no sort.
constexpr int kAggBatch = 8;

template <int QUANT, int KP, int N>
struct MessageBatch {
    uint32_t p[N][KP];
    float val[N][KP];                    // unquantised: the values
    float level[N];                      // quantised: the two levels, in the even and the odd lanes

    // Fetch replicas r0 .. r0 + N - 1 of chunk c.  Every load is unconditional -- a replica or an entry past the last one repeats
    // that one, and is not applied -- so that the pointers of all of them are on their way together, and then all their
    // messages: under a condition each replica's pointers are waited for before the next one's are requested.  The levels
    // come by vector loads because a wait for LDS would wait for scalar ones too.
    __device__ __forceinline__ void load(uint64_t c, uint32_t kappa, uint32_t kappa_c, int r0, int n_replicas,
                                         const uint16_t* const* __restrict__ pairs_tab,
                                         const float* const* __restrict__ aux_tab, int lane) {
        const SPLC_GLOBAL uint16_t* pr[N];
        const SPLC_GLOBAL float* ar[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int r = r0 + i < n_replicas ? r0 + i : n_replicas - 1;
            pr[i] = (const SPLC_GLOBAL uint16_t*)pairs_tab[r];
            ar[i] = (const SPLC_GLOBAL float*)aux_tab[r];
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t at[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) at[k] = lane + 64 * k < kappa_c ? lane + 64 * k : kappa_c - 1;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (QUANT == SPLC_QUANT_2BIT) level[i] = (ar[i] + 2 * c)[lane & 1];
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                p[i][k] = (pr[i] + c * kappa)[at[k]];
                if (QUANT == SPLC_QUANT_NONE) val[i][k] = (ar[i] + c * kappa)[at[k]];
            }
        }
    }

    // Add them to the accumulator, replica after replica.
    __device__ __forceinline__ void apply(float* acc, uint32_t kappa_c, int r0, int n_replicas, int lane) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (r0 + i < n_replicas) {
                float lo = 0.f, hi = 0.f;
                if (QUANT == SPLC_QUANT_2BIT) {
                    lo = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(level[i]), 0));
                    hi = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(level[i]), 1));
                }
#pragma unroll
                for (int k = 0; k < KP; ++k) {
                    const uint32_t t = lane + 64 * k;
                    const uint32_t idx = p[i][k] & 0xFFFu;
                    float q;
                    if (QUANT == SPLC_QUANT_2BIT) {
                        const float l = (p[i][k] & 0x1000u) ? hi : lo;
                        q = (p[i][k] & 0x2000u) ? -l : l;
                    } else {
                        q = val[i][k];
                    }
                    if (t < kappa_c) acc[idx] = __fadd_rn(acc[idx], q);
                }
                // The adds of replica r0 + i + 1 must follow those of replica r0 + i in program order (two replicas
                // may hit the same index from different lanes): keep the compiler from moving LDS accesses across.
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
};

// All lanes of the workgroup call this after the accumulator has been cleared (no barrier needed
// before the call; one is taken inside before the first add).  Ends with a barrier.
template <int QUANT, int KP, int N>
__device__ __forceinline__ void accumulate_chunk(float* acc, uint64_t c, uint32_t kappa, uint32_t kappa_c,
                                                 int n_replicas, const uint16_t* const* __restrict__ pairs_tab,
                                                 const float* const* __restrict__ aux_tab, int lane, int wave) {
    const int n_batches = (n_replicas + N - 1) / N;
    MessageBatch<QUANT, KP, N> mb;
    if (wave < n_batches) mb.load(c, kappa, kappa_c, wave * N, n_replicas, pairs_tab, aux_tab, lane);
    __syncthreads();                                   // accumulator cleared by every lane
    for (int g = 0; g < n_batches; ++g) {
        if (wave == (g & 3)) {
            mb.apply(acc, kappa_c, g * N, n_replicas, lane);
            if (g + 4 < n_batches)
                mb.load(c, kappa, kappa_c, (g + 4) * N, n_replicas, pairs_tab, aux_tab, lane);
        }
        __syncthreads();
    }
}

// Any kappa: one replica after the other, no batching (used for kappa > 256).
template <int QUANT>
__device__ __forceinline__ void accumulate_chunk_any(float* acc, uint64_t c, uint32_t kappa,
                                                     uint32_t kappa_c, int n_replicas,
                                                     const uint16_t* const* __restrict__ pairs_tab,
                                                     const float* const* __restrict__ aux_tab, int lane) {
    for (int r = 0; r < n_replicas; ++r) {
        const uint16_t* pr = pairs_tab[r] + c * kappa;
        const float* ar = aux_tab[r];
        float lo = 0.f, hi = 0.f;
        if (QUANT == SPLC_QUANT_2BIT) { lo = ar[2 * c]; hi = ar[2 * c + 1]; }
        for (uint32_t t = lane; t < kappa_c; t += 64) {
            const uint32_t p = pr[t];
            const uint32_t idx = p & 0xFFFu;
            float q;
            if (QUANT == SPLC_QUANT_2BIT) {
                const float level = (p & 0x1000u) ? hi : lo;
                q = (p & 0x2000u) ? -level : level;
            } else {
                q = ar[c * kappa + t];
            }
            acc[idx] = __fadd_rn(acc[idx], q);
            __builtin_amdgcn_wave_barrier();         // keeps the LDS accesses of successive rounds in program order
        }
    }
}

// Line 5 of the update equations.  One workgroup per chunk; all lanes clear the 16 KB LDS
// accumulator, the waves apply the messages batch by batch, all lanes divide once by M and write.
// KP: entries of a message per lane of a complete chunk (splc::entries_per_lane; 0: any kappa).  A kernel for each takes 24 to 53 registers up to
// kappa 64 where one for all took 85, so eight workgroups share a compute unit instead of five; with that and the loads of a
// batch in flight together (MessageBatch), messages that are not in a cache cost less: mean of 225,000 chunks, kappa 64,
// 8 replicas 820 -> 723 us (floor 640), 69,000 chunks, kappa 32, 32 replicas 343 -> 306, tiles of 2050 columns 414 -> 362.
// How many of them share a unit, and when theta is read: splc::aggregate_pace.
//   UPDATE = 0: delta_bar = acc / M is written densely (sparseloco_aggregate).
//   UPDATE = 1: theta = fl(theta - fl(eta * delta_bar)) is applied in the same pass, and the new theta
//               is also copied into n_reset further parameter sets (the replicas' theta_local, which
//               restart from the synchronised parameters: section 2.1, inner step); delta_bar is
//               written only if a table for it is given (sparseloco_aggregate_update).
template <int QUANT, int UPDATE, bool VEC, int KP>
__device__ __forceinline__ void aggregate_body(float* acc, const ChunkDesc* __restrict__ chunks, int n_replicas,
                                                             uint32_t kappa,
                                                             const uint16_t* const* __restrict__ pairs_tab,
                                                             const float* const* __restrict__ aux_tab,
                                                             float* const* __restrict__ dbar_tab,
                                                             float* const* __restrict__ theta_tab, float eta, int n_reset,
                                               uint32_t n_tensors, float* const* __restrict__ reset_tab, bool theta_late,
                                               splc::MeanStores stores, uint32_t entry) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ChunkDesc d = chunks[entry];
    const uint64_t c = d.id;
    const uint32_t n_c = VEC ? (uint32_t)kChunk : d.n_c;
    const uint32_t kappa_c = kappa < n_c ? kappa : n_c;
    float4* acc4 = reinterpret_cast<float4*>(acc);
    float* th = UPDATE ? theta_tab[d.tensor] + d.offset : nullptr;
    float* po = dbar_tab ? dbar_tab[d.tensor] + d.offset : nullptr;
    float4 tv[4];
    auto load_theta = [&] {
        with_chunk<VEC>(d, tid, [&](const auto& chunk) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (slot_used<VEC>(d, s)) tv[s] = chunk.load(th, s);
        });
    };
    if (UPDATE && !theta_late) load_theta();
#pragma unroll
    for (int s = 0; s < 4; ++s) acc4[s * kThreads + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    auto accumulate = [&](auto per_lane, auto batch) {
        accumulate_chunk<QUANT, decltype(per_lane)::value, decltype(batch)::value>(acc, c, kappa, kappa_c, n_replicas, pairs_tab,
                                                                                   aux_tab, lane, wave);
    };
    using std::integral_constant;
    // An edge chunk may hold fewer elements than kappa, and its messages are shorter then.  (Four entries per lane in batches
    // of four: those of eight would take the registers that let eight workgroups share a unit.)
    if (!VEC && KP != 1 && splc::entries_per_lane(kappa_c) == 1) {
        accumulate(integral_constant<int, 1>{}, integral_constant<int, kAggBatch>{});
    } else if (!VEC && (KP == 0 || KP == 4) && splc::entries_per_lane(kappa_c) == 2) {
        accumulate(integral_constant<int, 2>{}, integral_constant<int, kAggBatch>{});
    } else if (!VEC && KP == 0 && splc::entries_per_lane(kappa_c) == 4) {
        accumulate(integral_constant<int, 4>{}, integral_constant<int, kAggBatch / 2>{});
    } else if constexpr (KP > 0) {
        accumulate(integral_constant<int, KP>{}, integral_constant<int, kAggBatch>{});
    } else {
        __syncthreads();
        if (wave == 0) accumulate_chunk_any<QUANT>(acc, c, kappa, kappa_c, n_replicas, pairs_tab, aux_tab, lane);
        __syncthreads();
    }
    if (UPDATE && theta_late) load_theta();
    const float m = (float)n_replicas;
    auto finish = [&](auto quotient) {
        with_chunk<VEC>(d, tid, [&](const auto& chunk) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (!slot_used<VEC>(d, s)) break;
                float4 v = acc4[s * kThreads + tid];
                v.x = quotient(v.x); v.y = quotient(v.y); v.z = quotient(v.z); v.w = quotient(v.w);
                if (po) chunk.store(po, s, v);
                if (UPDATE) {
                    float4 t = tv[s];
                    if (!VEC) pull(edge_vec(d, tid, s).n, t.x, t.y, t.z, t.w);
                    t.x = __fsub_rn(t.x, __fmul_rn(eta, v.x));
                    t.y = __fsub_rn(t.y, __fmul_rn(eta, v.y));
                    t.z = __fsub_rn(t.z, __fmul_rn(eta, v.z));
                    t.w = __fsub_rn(t.w, __fmul_rn(eta, v.w));
                    chunk.store(th, s, t);
                    for (int r = 0; r < n_reset; ++r)
                        chunk.store(reset_tab[(size_t)r * n_tensors + d.tensor] + d.offset, s, t);
                }
            }
        });
    };
    // A power of two divides exactly like its inverse multiplies: one rounding of the same value.  (The choice is made out here,
    // for all slots at once: in their loop it slowed the division down, mean of 1000 chunks, kappa 16, 27 replicas 7.1 -> 7.6 us.)
    if ((n_replicas & (n_replicas - 1)) == 0 && (UPDATE || stores != splc::MeanStores::divided)) {
        const float inverse = __fdiv_rn(1.f, m);
        finish([=](float x) { return __fmul_rn(x, inverse); });
    } else if (VEC && !UPDATE && stores == splc::MeanStores::together) {
        float4 v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            v[s] = acc4[s * kThreads + tid];
            v[s].x = __fdiv_rn(v[s].x, m); v[s].y = __fdiv_rn(v[s].y, m); v[s].z = __fdiv_rn(v[s].z, m); v[s].w = __fdiv_rn(v[s].w, m);
        }
        __builtin_amdgcn_sched_barrier(0);
        with_chunk<VEC>(d, tid, [&](const auto& chunk) {
#pragma unroll
            for (int s = 0; s < 4; ++s) chunk.store(po, s, v[s]);
        });
    } else {
        finish([=](float x) { return __fdiv_rn(x, m); });
    }
}

template <int QUANT, int UPDATE, int KP>
__global__ __launch_bounds__(kThreads) void aggregate_kernel(const ChunkDesc* __restrict__ chunks, uint32_t n_gen,
                                                             int n_replicas, uint32_t kappa,
                                                             const uint16_t* const* __restrict__ pairs_tab,
                                                             const float* const* __restrict__ aux_tab,
                                                             float* const* __restrict__ dbar_tab,
                                                             float* const* __restrict__ theta_tab, float eta,
                                                             int n_reset, uint32_t n_tensors, bool in_runs, bool theta_late,
                                                             splc::MeanStores stores, float* const* __restrict__ reset_tab) {
    __shared__ __align__(16) float acc[kChunk];
    const uint32_t entry = in_runs ? splc::entry_in_runs(blockIdx.x, gridDim.x) : blockIdx.x;
    if (entry >= n_gen)
        aggregate_body<QUANT, UPDATE, true, KP>(acc, chunks, n_replicas, kappa, pairs_tab, aux_tab, dbar_tab, theta_tab, eta,
                                                n_reset, n_tensors, reset_tab, theta_late, stores, entry);
    else
        aggregate_body<QUANT, UPDATE, false, KP>(acc, chunks, n_replicas, kappa, pairs_tab, aux_tab, dbar_tab, theta_tab,
                                                 eta, n_reset, n_tensors, reset_tab, theta_late, stores, entry);
}

// Line 5, second half: theta = fl(theta - fl(eta * delta_bar)).
template <bool VEC>
__device__ __forceinline__ void outer_update_body(const ChunkDesc* __restrict__ chunks,
                                                  float* const* __restrict__ theta_tab,
                                                  const float* const* __restrict__ dbar_tab, float eta) {
    const int tid = threadIdx.x;
    const ChunkDesc d = chunks[blockIdx.x];
    float* th = theta_tab[d.tensor] + d.offset;
    const float* db = dbar_tab[d.tensor] + d.offset;
    with_chunk<VEC>(d, tid, [&](const auto& chunk) {
        float4 t[4], g[4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (slot_used<VEC>(d, s)) t[s] = chunk.load(th, s);
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (slot_used<VEC>(d, s)) g[s] = chunk.load(db, s);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (!slot_used<VEC>(d, s)) break;
            if (!VEC) {
                const uint32_t n = edge_vec(d, tid, s).n;
                pull(n, t[s].x, t[s].y, t[s].z, t[s].w);
                pull(n, g[s].x, g[s].y, g[s].z, g[s].w);
            }
            t[s].x = __fsub_rn(t[s].x, __fmul_rn(eta, g[s].x));
            t[s].y = __fsub_rn(t[s].y, __fmul_rn(eta, g[s].y));
            t[s].z = __fsub_rn(t[s].z, __fmul_rn(eta, g[s].z));
            t[s].w = __fsub_rn(t[s].w, __fmul_rn(eta, g[s].w));
            chunk.store(th, s, t[s]);
        }
    });
}

__global__ __launch_bounds__(kThreads) void outer_update_kernel(const ChunkDesc* __restrict__ chunks, uint32_t n_gen,
                                                                float* const* __restrict__ theta_tab,
                                                                const float* const* __restrict__ dbar_tab,
                                                                float eta) {
    if (blockIdx.x >= n_gen) outer_update_body<true>(chunks, theta_tab, dbar_tab, eta);
    else outer_update_body<false>(chunks, theta_tab, dbar_tab, eta);
}

}  // namespace

// ------------------------------------------------------------------ host side

struct sparseloco_plan {
    int device = 0;
    int n_tensors = 0;
    int kappa = 0;
    int quant = SPLC_QUANT_2BIT;
    int select = SPLC_SELECT_AUTO;
    uint32_t* radix_counter = nullptr;   // diagnostic (sparseloco_plan_set_radix_counter), normally null
    int64_t n_chunks = 0;
    int64_t n_params = 0;
    std::vector<int64_t> numel;
    int layout = SPLC_LAYOUT_FLAT;
    // Chunk table, ordered [edge chunks | complete, odd row length | other complete ones]; every entry carries its chunk
    // number.  The edge chunks, which take a little longer, come first so that they do not form the tail of the launch.
    // The compression of a large tiled plan takes complete tiles four at a time where four lie side by side ("strips", one
    // entry each: origin, stride and chunk number of the first tile); only the other chunks are in the table above.  Its
    // outer update, which is element-wise, walks the tensors as flat chunks (a table of its own).
    // One device allocation holds [chunks | strips | flat chunks of the update | every chunk one by one].
    ChunkDesc* d_chunks = nullptr;
    ChunkDesc* h_chunks = nullptr;       // pinned source of the asynchronous upload, kept until destroy
    int64_t n_entries = 0;               // entries of the chunk table (= n_chunks unless there are strips)
    int64_t n_gen = 0;                   // edge chunks among them
    int64_t n_strips = 0;
    ChunkDesc* d_strips = nullptr;       // inside d_chunks' allocation
    ChunkDesc* d_update = nullptr;       // = d_chunks for a flat plan
    int64_t n_update = 0, n_update_gen = 0;
    ChunkDesc* d_all = nullptr;          // every chunk one by one, for all other kernels (= d_chunks without strips)
    int64_t n_all_gen = 0;
};

// n_sets lists of n_tensors device pointers, set-major, resident on the device.
struct sparseloco_tensors {
    int device = 0;
    int n_tensors = 0;
    int n_sets = 0;
    int dtype = SPLC_F32;
    bool disjoint = false;               // no tensor shares memory with another (looked at where it matters: small plans)
    void** d_table = nullptr;
    void** h_table = nullptr;            // pinned source of the upload
};

// Message buffers of n_replicas replicas: device table [pairs: n_replicas][aux: n_replicas].
struct sparseloco_messages {
    int device = 0;
    int n_replicas = 0;
    int quant = SPLC_QUANT_2BIT;
    int kappa = 0;
    int64_t n_chunks = 0;
    bool disjoint = false;               // no buffer shares memory with another (as above)
    void** d_table = nullptr;
    void** h_table = nullptr;
};

namespace {

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
bool finite(float v) { return v == v && v - v == 0.f; }

int current_device_is(int device) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return SPLC_EHIP;
    return dev == device ? SPLC_OK : SPLC_EPLAN;
}

// A binding fits the plan: same device, same tensor count, the wanted element type, enough sets.
int check_tensors(const sparseloco_plan* plan, const sparseloco_tensors* t, int dtype, int min_sets) {
    if (!t) return SPLC_EINVAL;
    if (t->device != plan->device || t->n_tensors != plan->n_tensors || t->dtype != dtype) return SPLC_EPLAN;
    return t->n_sets >= min_sets ? SPLC_OK : SPLC_EINVAL;
}
int check_messages(const sparseloco_plan* plan, const sparseloco_messages* m, int min_replicas) {
    if (!m) return SPLC_EINVAL;
    if (m->device != plan->device || m->quant != plan->quant || m->kappa != plan->kappa || m->n_chunks != plan->n_chunks)
        return SPLC_EPLAN;
    return m->n_replicas >= min_replicas ? SPLC_OK : SPLC_EINVAL;
}
// Device table of set `set` of a binding (a single-set binding serves every set index).
template <class T>
T const* set_table(const sparseloco_tensors* t, int set) {
    return reinterpret_cast<T const*>(t->d_table + (size_t)(t->n_sets == 1 ? 0 : set) * (size_t)t->n_tensors);
}

// A small table of device pointers: pinned host copy + device copy, uploaded asynchronously on `stream`.
int upload_table(size_t n_ptrs, void*** h_out, void*** d_out) {
    const size_t bytes = (n_ptrs ? n_ptrs : 1) * sizeof(void*);
    if (hipHostMalloc(reinterpret_cast<void**>(h_out), bytes, hipHostMallocDefault) != hipSuccess) return SPLC_ENOMEM;
    if (hipMalloc(reinterpret_cast<void**>(d_out), bytes) != hipSuccess) return SPLC_ENOMEM;
    return SPLC_OK;
}

std::pair<uintptr_t, uintptr_t> range_of(const void* p, uint64_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    return {a, a + (uintptr_t)bytes};
}
// Whether the ranges that `collect` lists are disjoint; false without a look where the plan is too large for the answer
// to matter (replicas_side_by_side), or where memory for the list runs out.
template <class Collect>
bool on_small_plan_disjoint(const sparseloco_plan* plan, Collect collect) {
    if (plan->n_chunks > splc::kFewChunks) return false;
    try {
        std::vector<std::pair<uintptr_t, uintptr_t>> ranges;
        collect(ranges);
        return splc::disjoint(std::move(ranges));
    } catch (const std::bad_alloc&) {
        return false;
    }
}

// LDS that a launch on a large plan reserves so that only `groups_per_unit` of its workgroups, which use `used` bytes
// each, fit on a compute unit (splc::few_streams).  LDS is handed out in 1280-byte units.
unsigned reserve_lds(int groups_per_unit, size_t used) {
    const size_t share = 160 * 1024 / (size_t)groups_per_unit / 1280 * 1280;
    return used < share ? (unsigned)(share - used) : 0u;
}
unsigned reserve_lds_compress(const sparseloco_plan* plan, int64_t entries, bool from_params, size_t used) {
    return splc::few_streams(entries, plan->kappa, from_params, plan->select == SPLC_SELECT_RADIX) ? reserve_lds(3, used) : 0u;
}

template <int MODE, int QUANT>
void launch_compress(const sparseloco_plan* plan, const void* const* a, const void* const* b, float* const* ef,
                     float beta, uint16_t* pairs_out, float* aux_out, hipStream_t stream) {
    const int force_radix = plan->select == SPLC_SELECT_RADIX ? 1 : 0;
    const bool strips = splc::strips_pay(plan->n_strips, plan->kappa, MODE == MODE_PARAMS_F32);
    const int64_t entries = strips ? plan->n_entries : plan->n_chunks;
    if (strips)
        hipLaunchKernelGGL((compress_strip_kernel<MODE, QUANT>), dim3((unsigned)plan->n_strips), dim3(kStripThreads), 0,
                           stream, plan->d_strips, a, b, ef, beta, (uint32_t)plan->kappa, force_radix,
                           plan->radix_counter, pairs_out, aux_out);
    if (entries > 0)
        hipLaunchKernelGGL((compress_kernel<MODE, QUANT>), dim3((unsigned)entries), dim3(kThreads),
                           reserve_lds_compress(plan, entries, MODE == MODE_PARAMS_F32, sizeof(SelectShared)), stream,
                           strips ? plan->d_chunks : plan->d_all, (unsigned)(strips ? plan->n_gen : plan->n_all_gen), a, b,
                           ef, beta, (uint32_t)plan->kappa, force_radix, plan->radix_counter, pairs_out, aux_out);
}

template <int QUANT, int UPDATE>
void launch_aggregate(const sparseloco_plan* plan, int n_replicas, const uint16_t* const* pairs,
                      const float* const* aux, float* const* dbar, float* const* theta, float eta, int n_reset,
                      float* const* reset, hipStream_t stream) {
    const bool flat = plan->layout == SPLC_LAYOUT_FLAT;
    const bool in_runs = flat && splc::chunks_in_runs(plan->n_chunks, n_replicas, plan->kappa, QUANT == SPLC_QUANT_2BIT, UPDATE);
    const splc::AggregatePace pace =
        splc::aggregate_pace(plan->n_chunks, n_replicas, plan->kappa, QUANT == SPLC_QUANT_2BIT, flat, UPDATE);
    const unsigned reserved = pace.groups_per_unit ? reserve_lds(pace.groups_per_unit, sizeof(float) * kChunk) : 0u;
    auto launch = [&](auto per_lane) {
        hipLaunchKernelGGL((aggregate_kernel<QUANT, UPDATE, decltype(per_lane)::value>), dim3((unsigned)plan->n_chunks),
                           dim3(kThreads), reserved, stream, plan->d_all, (unsigned)plan->n_all_gen, n_replicas,
                           (uint32_t)plan->kappa, pairs, aux, dbar, theta, eta, n_reset, (uint32_t)plan->n_tensors, in_runs,
                           pace.theta_late, splc::mean_stores(plan->n_chunks, n_replicas, plan->kappa, flat), reset);
    };
    switch (splc::entries_per_lane((uint32_t)plan->kappa)) {
        case 1: launch(std::integral_constant<int, 1>{}); break;
        case 2: launch(std::integral_constant<int, 2>{}); break;
        case 4: launch(std::integral_constant<int, 4>{}); break;
        default: launch(std::integral_constant<int, 0>{}); break;
    }
}

template <int QUANT, bool STEP>
void launch_compress_batch(const sparseloco_plan* plan, int n_replicas, bool disjoint, float* const* to,
                           float* const* tl, float* const* ef, float beta, uint16_t* const* pairs, float* const* aux,
                           float eta, float* const* dbar, int reset, hipStream_t stream) {
    if (splc::replicas_side_by_side(plan->n_chunks, n_replicas, STEP, disjoint)) {
        hipLaunchKernelGGL((compress_each_kernel<QUANT>), dim3((unsigned)plan->n_chunks, (unsigned)n_replicas),
                           dim3(kThreads), 0, stream, plan->d_all, (unsigned)plan->n_all_gen, (uint32_t)plan->n_tensors,
                           reinterpret_cast<const void* const*>(to), reinterpret_cast<const void* const*>(tl), ef, beta,
                           (uint32_t)plan->kappa, plan->select == SPLC_SELECT_RADIX ? 1 : 0, plan->radix_counter, pairs,
                           aux);
        if (STEP)
            launch_aggregate<QUANT, 1>(plan, n_replicas, const_cast<const uint16_t* const*>(pairs),
                                       const_cast<const float* const*>(aux), dbar, to, eta, reset ? n_replicas : 0, tl,
                                       stream);
        return;
    }
    // (tile by tile, also where compress takes strips)
    const size_t used = sizeof(SelectShared) + sizeof(float) * (kChunk + (STEP ? kChunk : 4));
    hipLaunchKernelGGL((compress_batch_kernel<QUANT, STEP>), dim3((unsigned)plan->n_chunks), dim3(kThreads),
                       reserve_lds_compress(plan, plan->n_chunks, true, used), stream,
                       plan->d_all, (unsigned)plan->n_all_gen, n_replicas, (uint32_t)plan->n_tensors, to, tl, ef,
                       beta, (uint32_t)plan->kappa, plan->select == SPLC_SELECT_RADIX ? 1 : 0, plan->radix_counter, pairs,
                       aux, eta, dbar, reset);
}

// Shared by sparseloco_compress_batch and sparseloco_outer_step_batch.
int compress_batch_impl(const sparseloco_plan* plan, int n_replicas, const sparseloco_tensors* theta_outer,
                        const sparseloco_tensors* theta_local, const sparseloco_tensors* ef, float beta,
                        const sparseloco_messages* messages_out, bool step, float outer_lr,
                        const sparseloco_tensors* delta_bar_out, int reset, void* stream) {
    if (!plan || n_replicas < 1 || n_replicas > SPLC_MAX_REPLICAS) return SPLC_EINVAL;
    int rc;
    if ((rc = check_tensors(plan, theta_outer, SPLC_F32, 1)) != SPLC_OK) return rc;
    if (theta_outer->n_sets != 1) return SPLC_EINVAL;
    if ((rc = check_tensors(plan, theta_local, SPLC_F32, n_replicas)) != SPLC_OK) return rc;
    if ((rc = check_tensors(plan, ef, SPLC_F32, n_replicas)) != SPLC_OK) return rc;
    if ((rc = check_messages(plan, messages_out, n_replicas)) != SPLC_OK) return rc;
    if (delta_bar_out) {
        if ((rc = check_tensors(plan, delta_bar_out, SPLC_F32, 1)) != SPLC_OK) return rc;
        if (delta_bar_out->n_sets != 1) return SPLC_EINVAL;
    }
    if (!finite(beta) || !finite(outer_lr)) return SPLC_EINVAL;
    if ((rc = current_device_is(plan->device)) != SPLC_OK) return rc;
    if (plan->n_chunks == 0) return SPLC_OK;

    hipStream_t st = static_cast<hipStream_t>(stream);
    float* const* d_to = set_table<float*>(theta_outer, 0);
    float* const* d_tl = reinterpret_cast<float* const*>(theta_local->d_table);
    float* const* d_ef = reinterpret_cast<float* const*>(ef->d_table);
    uint16_t* const* d_pairs = reinterpret_cast<uint16_t* const*>(messages_out->d_table);
    float* const* d_aux = reinterpret_cast<float* const*>(messages_out->d_table + messages_out->n_replicas);
    float* const* d_dbar = delta_bar_out ? set_table<float*>(delta_bar_out, 0) : nullptr;
    const bool q2 = plan->quant == SPLC_QUANT_2BIT, apart = ef->disjoint && messages_out->disjoint;
    if (q2 && !step)
        launch_compress_batch<SPLC_QUANT_2BIT, false>(plan, n_replicas, apart, d_to, d_tl, d_ef, beta, d_pairs, d_aux,
                                                      0.f, nullptr, 0, st);
    else if (q2)
        launch_compress_batch<SPLC_QUANT_2BIT, true>(plan, n_replicas, apart, d_to, d_tl, d_ef, beta, d_pairs, d_aux,
                                                     outer_lr, d_dbar, reset, st);
    else if (!step)
        launch_compress_batch<SPLC_QUANT_NONE, false>(plan, n_replicas, apart, d_to, d_tl, d_ef, beta, d_pairs, d_aux,
                                                      0.f, nullptr, 0, st);
    else
        launch_compress_batch<SPLC_QUANT_NONE, true>(plan, n_replicas, apart, d_to, d_tl, d_ef, beta, d_pairs, d_aux,
                                                     outer_lr, d_dbar, reset, st);
    return hipGetLastError() == hipSuccess ? SPLC_OK : SPLC_EHIP;
}

// Shared by sparseloco_aggregate and sparseloco_aggregate_update.
int aggregate_impl(const sparseloco_plan* plan, const sparseloco_messages* messages,
                   const sparseloco_tensors* delta_bar_out, const sparseloco_tensors* theta_outer, float outer_lr,
                   bool update, const sparseloco_tensors* reset, void* stream) {
    if (!plan) return SPLC_EINVAL;
    int rc = check_messages(plan, messages, 1);
    if (rc != SPLC_OK) return rc;
    if (update ? !theta_outer : !delta_bar_out) return SPLC_EINVAL;
    if (delta_bar_out && (rc = check_tensors(plan, delta_bar_out, SPLC_F32, 1)) != SPLC_OK) return rc;
    if (update && (rc = check_tensors(plan, theta_outer, SPLC_F32, 1)) != SPLC_OK) return rc;
    if (reset && (rc = check_tensors(plan, reset, SPLC_F32, 1)) != SPLC_OK) return rc;
    if ((delta_bar_out && delta_bar_out->n_sets != 1) || (update && theta_outer->n_sets != 1)) return SPLC_EINVAL;
    if (!finite(outer_lr)) return SPLC_EINVAL;
    if ((rc = current_device_is(plan->device)) != SPLC_OK) return rc;
    if (plan->n_chunks == 0) return SPLC_OK;

    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nr = messages->n_replicas;
    const uint16_t* const* dp = reinterpret_cast<const uint16_t* const*>(messages->d_table);
    const float* const* dx = reinterpret_cast<const float* const*>(messages->d_table + nr);
    float* const* dout = delta_bar_out ? set_table<float*>(delta_bar_out, 0) : nullptr;
    float* const* dth = update ? set_table<float*>(theta_outer, 0) : nullptr;
    float* const* dreset = reset ? set_table<float*>(reset, 0) : nullptr;
    const int n_reset = reset ? reset->n_sets : 0;
    const bool q2 = plan->quant == SPLC_QUANT_2BIT;
    if (q2 && !update)
        launch_aggregate<SPLC_QUANT_2BIT, 0>(plan, nr, dp, dx, dout, dth, outer_lr, 0, dreset, st);
    else if (q2)
        launch_aggregate<SPLC_QUANT_2BIT, 1>(plan, nr, dp, dx, dout, dth, outer_lr, n_reset, dreset, st);
    else if (!update)
        launch_aggregate<SPLC_QUANT_NONE, 0>(plan, nr, dp, dx, dout, dth, outer_lr, 0, dreset, st);
    else
        launch_aggregate<SPLC_QUANT_NONE, 1>(plan, nr, dp, dx, dout, dth, outer_lr, n_reset, dreset, st);
    return hipGetLastError() == hipSuccess ? SPLC_OK : SPLC_EHIP;
}

// Chunk table of one tensor.  rows == 1 (or flat layout): runs of 4096 elements; otherwise 64 x 64 tiles
// numbered row-major.
void append_chunks(std::vector<ChunkDesc>& table, uint32_t tensor, int64_t rows, int64_t cols, bool tiled) {
    if (rows * cols == 0) return;
    if (!tiled || rows == 1) {
        const int64_t numel = rows * cols;
        for (int64_t off = 0; off < numel; off += kChunk) {
            const int64_t n = (numel - off) < kChunk ? (numel - off) : kChunk;
            ChunkDesc cd = {};
            cd.tensor = tensor;
            cd.n_c = (uint32_t)n;
            cd.offset = (uint64_t)off;
            cd.stride = 64;
            cd.h = (uint8_t)((n + 63) / 64);
            cd.w = 64;
            cd.last_w = (uint8_t)(n - 64 * (cd.h - 1));
            cd.vec = n == kChunk ? 3 : 0;
            table.push_back(cd);
        }
        return;
    }
    for (int64_t r0 = 0; r0 < rows; r0 += 64) {
        for (int64_t c0 = 0; c0 < cols; c0 += 64) {
            const int64_t h = (rows - r0) < 64 ? (rows - r0) : 64, w = (cols - c0) < 64 ? (cols - c0) : 64;
            ChunkDesc cd = {};
            cd.tensor = tensor;
            cd.n_c = (uint32_t)(h * w);
            cd.offset = (uint64_t)(r0 * cols + c0);
            cd.stride = (uint32_t)cols;
            cd.h = (uint8_t)h;
            cd.w = (uint8_t)w;
            cd.last_w = (uint8_t)w;
            const bool full = h == 64 && w == 64;
            cd.vec = (uint8_t)((full ? 1 : 0) | ((full && cols % 2 == 0) ? 2 : 0));
            table.push_back(cd);
        }
    }
}

int chunk_class(const ChunkDesc& d) { return d.vec == 0 ? 0 : (d.vec == 1 ? 1 : 2); }

// Order in which workgroups take the entries: edge chunks first (they take a little longer and should not form the
// tail), then complete ones in matrices of odd row length, then the other complete ones (no kernel tells these two apart;
// it is the order that sparseloco_chunk_table answers).  For a tiled plan, inside each class every XCD gets a run of consecutive tiles:
// workgroups go to the eight XCDs round-robin by number, neighbouring tiles of a tile row continue each other's row
// segments (and share the cache lines on their common edge when the row length is no multiple of 32 floats), so
// neighbours should meet in one L2.  Only the order of processing changes: a chunk's number, and with it the place of
// its pairs in the message, is its `id`.
void order_for_launch(std::vector<ChunkDesc>& table, bool deal_to_xcds) {
    std::stable_sort(table.begin(), table.end(),
                     [](const ChunkDesc& a, const ChunkDesc& b) { return chunk_class(a) < chunk_class(b); });
    if (!deal_to_xcds) return;
    size_t start = 0;
    while (start < table.size()) {
        size_t end = start;
        while (end < table.size() && chunk_class(table[end]) == chunk_class(table[start])) ++end;
        const std::vector<ChunkDesc> seg(table.begin() + (ptrdiff_t)start, table.begin() + (ptrdiff_t)end);
        size_t next = 0;
        for (size_t r = 0; r < 8; ++r)
            for (size_t pos = start + (r + 8 - start % 8) % 8; pos < end; pos += 8) table[pos] = seg[next++];
        start = end;
    }
}

struct ChunkTables {
    int64_t n_chunks = 0, n_params = 0;
    std::vector<ChunkDesc> all;          // every chunk, launch order
    std::vector<ChunkDesc> rest;         // tiled plans: the chunks outside strips, launch order
    std::vector<ChunkDesc> strips;       // tiled plans: one entry per strip (its first tile), launch order
    std::vector<ChunkDesc> update;       // tiled plans: flat chunks for the element-wise update
};

// Validates the tensor list and counts its chunks; fills the tables if asked to.
int build_chunk_tables(int n_tensors, const int64_t* rows, const int64_t* cols, bool tiled, ChunkTables& t, bool fill) {
    if (n_tensors < 1 || !cols || (tiled && !rows)) return SPLC_EINVAL;
    int64_t n_chunks = 0, n_params = 0;
    for (int i = 0; i < n_tensors; ++i) {
        const int64_t r = tiled ? rows[i] : 1, c = cols[i];
        if (r < 0 || c < 0) return SPLC_EINVAL;
        if (r > 0 && c > (int64_t)0x7FFFFFFFFFFFFFFF / r) return SPLC_EINVAL;
        if (tiled && r > 1) {
            if (c >= (int64_t)1 << 24) return SPLC_EINVAL;        // byte offsets inside a tile must fit 32 bits
            n_chunks += ((r + 63) / 64) * ((c + 63) / 64);
        } else {
            n_chunks += (r * c + kChunk - 1) / kChunk;
        }
        n_params += r * c;
    }
    if (n_chunks > 0x7FFFFFFF) return SPLC_EINVAL;      // one workgroup per chunk in a 1-D grid
    t.n_chunks = n_chunks;
    t.n_params = n_params;
    if (!fill) return SPLC_OK;
    t.all.clear();
    t.all.reserve((size_t)n_chunks);
    for (int i = 0; i < n_tensors; ++i) append_chunks(t.all, (uint32_t)i, tiled ? rows[i] : 1, cols[i], tiled);
    for (size_t k = 0; k < t.all.size(); ++k) t.all[k].id = (uint32_t)k;
    t.rest.clear();
    t.strips.clear();
    t.update.clear();
    if (tiled) {
        // Strips: four complete tiles side by side, in matrices whose row length is no multiple of 32 floats (with
        // such a multiple a tile's 256-byte row segments are two whole cache lines already, and the one-tile
        // kernel, which needs no trip through LDS, is the faster one: measured 6.0 against 5.8 TB/s) but even (so
        // that rows of a bf16 source start on dword boundaries too).  Tiles of one tile row have consecutive numbers.
        size_t k = 0;
        for (int i = 0; i < n_tensors; ++i) {
            const int64_t r = rows[i], c = cols[i];
            if (r * c == 0) continue;
            if (r == 1) { k += (size_t)((c + kChunk - 1) / kChunk); continue; }
            const int64_t nbi = (r + 63) / 64, nbj = (c + 63) / 64, full_cols = c / 64;
            for (int64_t bi = 0; bi < nbi; ++bi, k += (size_t)nbj) {
                if (c % 32 == 0 || c % 2 != 0 || (bi + 1) * 64 > r) continue;
                for (int64_t s4 = 0; s4 + kStripTiles <= full_cols; s4 += kStripTiles)
                    for (int j = 0; j < kStripTiles; ++j) t.all[k + (size_t)(s4 + j)].reserved = 1u + (uint32_t)j;
            }
        }
        for (const ChunkDesc& cd : t.all) {
            if (cd.reserved == 0) t.rest.push_back(cd);
            else if (cd.reserved == 1) t.strips.push_back(cd);
        }
        order_for_launch(t.rest, true);
        // Strips of one tile row continue each other's rows: every XCD gets a run of consecutive strips.
        {
            const std::vector<ChunkDesc> seg(t.strips);
            size_t next = 0;
            for (size_t x = 0; x < 8; ++x)
                for (size_t pos = x; pos < seg.size(); pos += 8) t.strips[pos] = seg[next++];
        }
        for (int i = 0; i < n_tensors; ++i) append_chunks(t.update, (uint32_t)i, 1, rows[i] * cols[i], false);
        order_for_launch(t.update, false);
    }
    order_for_launch(t.all, tiled);
    return SPLC_OK;
}

int64_t count_class0(const std::vector<ChunkDesc>& v) {
    int64_t n = 0;
    for (const ChunkDesc& cd : v) n += cd.vec == 0;
    return n;
}

int plan_build(sparseloco_plan** out, int n_tensors, const int64_t* rows, const int64_t* cols, bool tiled, int chunk,
               int kappa, int quant_mode, void* stream) {
    if (!out) return SPLC_EINVAL;
    *out = nullptr;
    if (chunk != kChunk || kappa < 1 || kappa > kChunk) return SPLC_EINVAL;
    if (quant_mode != SPLC_QUANT_NONE && quant_mode != SPLC_QUANT_2BIT) return SPLC_EINVAL;
    ChunkTables t;
    int rc = build_chunk_tables(n_tensors, tiled ? rows : nullptr, cols, tiled, t, true);
    if (rc != SPLC_OK) return rc;
    sparseloco_plan* plan = new (std::nothrow) sparseloco_plan();
    if (!plan) return SPLC_ENOMEM;
    if (hipGetDevice(&plan->device) != hipSuccess) { delete plan; return SPLC_EHIP; }
    plan->n_tensors = n_tensors;
    plan->kappa = kappa;
    plan->quant = quant_mode;
    plan->layout = tiled ? SPLC_LAYOUT_TILE64 : SPLC_LAYOUT_FLAT;
    plan->n_chunks = t.n_chunks;
    plan->n_params = t.n_params;
    plan->numel.resize((size_t)n_tensors);
    for (int i = 0; i < n_tensors; ++i) plan->numel[(size_t)i] = (tiled ? rows[i] : 1) * cols[i];
    // (kept where a compression of this plan takes them: from some source they pay)
    const int64_t n_strips = (int64_t)t.strips.size();
    const bool with_strips = splc::strips_pay(n_strips, kappa, true) || splc::strips_pay(n_strips, kappa, false);
    if (!with_strips) t.strips.clear();
    const std::vector<ChunkDesc>& main_table = with_strips ? t.rest : t.all;
    plan->n_entries = (int64_t)main_table.size();
    plan->n_gen = count_class0(main_table);
    plan->n_strips = (int64_t)t.strips.size();
    plan->n_update = tiled ? (int64_t)t.update.size() : plan->n_entries;
    plan->n_update_gen = tiled ? count_class0(t.update) : plan->n_gen;
    plan->n_all_gen = count_class0(t.all);
    // device layout: [main table | strips | update table (tiled) | every chunk (with strips)]
    const size_t n_main = main_table.size(), n_str = t.strips.size(), n_upd = tiled ? t.update.size() : 0,
                 n_all = with_strips ? t.all.size() : 0, total = n_main + n_str + n_upd + n_all;
    if (total > 0) {
        const size_t bytes = total * sizeof(ChunkDesc);
        if (hipHostMalloc(reinterpret_cast<void**>(&plan->h_chunks), bytes, hipHostMallocDefault) != hipSuccess ||
            hipMalloc(reinterpret_cast<void**>(&plan->d_chunks), bytes) != hipSuccess) {
            rc = SPLC_ENOMEM;
        } else {
            std::copy(main_table.begin(), main_table.end(), plan->h_chunks);
            std::copy(t.strips.begin(), t.strips.end(), plan->h_chunks + n_main);
            if (tiled) std::copy(t.update.begin(), t.update.end(), plan->h_chunks + n_main + n_str);
            if (with_strips) std::copy(t.all.begin(), t.all.end(), plan->h_chunks + n_main + n_str + n_upd);
            plan->d_strips = plan->d_chunks + n_main;
            plan->d_update = tiled ? plan->d_chunks + n_main + n_str : plan->d_chunks;
            plan->d_all = with_strips ? plan->d_chunks + n_main + n_str + n_upd : plan->d_chunks;
            if (hipMemcpyAsync(plan->d_chunks, plan->h_chunks, bytes, hipMemcpyHostToDevice,
                               static_cast<hipStream_t>(stream)) != hipSuccess)
                rc = SPLC_EHIP;
        }
    }
    if (rc != SPLC_OK) {
        sparseloco_plan_destroy(plan);
        return rc;
    }
    *out = plan;
    return SPLC_OK;
}

}  // namespace

extern "C" {

int sparseloco_plan_create(sparseloco_plan** out, int n_tensors, const int64_t* numel, int chunk, int kappa,
                           int quant_mode, void* stream) {
    return plan_build(out, n_tensors, nullptr, numel, false, chunk, kappa, quant_mode, stream);
}

int sparseloco_plan_create_2d(sparseloco_plan** out, int n_tensors, const int64_t* rows, const int64_t* cols,
                              int chunk, int kappa, int quant_mode, void* stream) {
    return plan_build(out, n_tensors, rows, cols, true, chunk, kappa, quant_mode, stream);
}

void sparseloco_plan_destroy(sparseloco_plan* plan) {
    if (!plan) return;
    if (plan->d_chunks) (void)hipFree(plan->d_chunks);              // waits for the device; holds all tables
    if (plan->h_chunks) (void)hipHostFree(plan->h_chunks);
    delete plan;
}

int64_t sparseloco_plan_num_chunks(const sparseloco_plan* plan) { return plan ? plan->n_chunks : SPLC_EINVAL; }
int64_t sparseloco_plan_num_params(const sparseloco_plan* plan) { return plan ? plan->n_params : SPLC_EINVAL; }
int sparseloco_plan_num_tensors(const sparseloco_plan* plan) { return plan ? plan->n_tensors : SPLC_EINVAL; }
int sparseloco_plan_kappa(const sparseloco_plan* plan) { return plan ? plan->kappa : SPLC_EINVAL; }
int sparseloco_plan_quant_mode(const sparseloco_plan* plan) { return plan ? plan->quant : SPLC_EINVAL; }
int sparseloco_plan_layout(const sparseloco_plan* plan) { return plan ? plan->layout : SPLC_EINVAL; }

int sparseloco_plan_set_select(sparseloco_plan* plan, int select_mode) {
    if (!plan || (select_mode != SPLC_SELECT_AUTO && select_mode != SPLC_SELECT_RADIX)) return SPLC_EINVAL;
    plan->select = select_mode;
    return SPLC_OK;
}

int sparseloco_plan_set_radix_counter(sparseloco_plan* plan, uint32_t* device_counter) {
    if (!plan || !aligned(device_counter, 4)) return SPLC_EINVAL;
    plan->radix_counter = device_counter;
    return SPLC_OK;
}

int64_t sparseloco_chunk_table(int n_tensors, const int64_t* rows, const int64_t* cols, int layout, void* out,
                               int64_t capacity) {
    if (layout != SPLC_LAYOUT_FLAT && layout != SPLC_LAYOUT_TILE64) return SPLC_EINVAL;
    if (capacity < 0 || (capacity > 0 && !out)) return SPLC_EINVAL;
    const bool tiled = layout == SPLC_LAYOUT_TILE64;
    std::vector<int64_t> flat;
    if (!tiled && rows && cols && n_tensors >= 1) {               // flat layout: only the element counts matter
        flat.resize((size_t)n_tensors);
        for (int i = 0; i < n_tensors; ++i) {
            if (rows[i] < 0 || cols[i] < 0 || (rows[i] > 0 && cols[i] > (int64_t)0x7FFFFFFFFFFFFFFF / rows[i]))
                return SPLC_EINVAL;
            flat[(size_t)i] = rows[i] * cols[i];
        }
        cols = flat.data();
    }
    ChunkTables t;
    int rc = build_chunk_tables(n_tensors, tiled ? rows : nullptr, cols, tiled, t, out != nullptr);
    if (rc != SPLC_OK) return rc;
    if (out) {
        // the entries workgroups of the one-chunk kernels walk, then the members of the strips in strip order
        std::vector<ChunkDesc> view = t.strips.empty() ? t.all : t.rest;
        if (!t.strips.empty()) {
            std::vector<const ChunkDesc*> by_id(t.all.size());
            for (const ChunkDesc& cd : t.all) by_id[cd.id] = &cd;
            for (const ChunkDesc& first : t.strips)
                for (int j = 0; j < kStripTiles; ++j) view.push_back(*by_id[first.id + (uint32_t)j]);
        }
        const int64_t n = t.n_chunks < capacity ? t.n_chunks : capacity;
        std::copy(view.begin(), view.begin() + (ptrdiff_t)n, static_cast<ChunkDesc*>(out));
    }
    return t.n_chunks;
}

int sparseloco_tensors_bind(sparseloco_tensors** out, const sparseloco_plan* plan, int n_sets,
                            const void* const* ptrs, int dtype, void* stream) {
    if (!out) return SPLC_EINVAL;
    *out = nullptr;
    if (!plan || !ptrs || n_sets < 1 || n_sets > SPLC_MAX_REPLICAS) return SPLC_EINVAL;
    if (dtype != SPLC_F32 && dtype != SPLC_BF16) return SPLC_EINVAL;
    const size_t nt = (size_t)plan->n_tensors, n = nt * (size_t)n_sets;
    for (size_t i = 0; i < n; ++i) {
        if (plan->numel[i % nt] == 0) continue;
        if (!ptrs[i]) return SPLC_EINVAL;
        if (!aligned(ptrs[i], 4)) return SPLC_EALIGN;             // for bf16 it keeps vector rows dword aligned
    }
    int rc = current_device_is(plan->device);
    if (rc != SPLC_OK) return rc;
    sparseloco_tensors* t = new (std::nothrow) sparseloco_tensors();
    if (!t) return SPLC_ENOMEM;
    t->device = plan->device;
    t->n_tensors = plan->n_tensors;
    t->n_sets = n_sets;
    t->dtype = dtype;
    t->disjoint = n_sets == 1 || on_small_plan_disjoint(plan, [&](auto& ranges) {
        const uint64_t size = dtype == SPLC_BF16 ? 2 : 4;
        for (size_t i = 0; i < n; ++i)
            ranges.push_back(range_of(ptrs[i], (uint64_t)plan->numel[i % nt] * size));
    });
    if ((rc = upload_table(n, &t->h_table, &t->d_table)) == SPLC_OK) {
        for (size_t i = 0; i < n; ++i) t->h_table[i] = plan->numel[i % nt] == 0 ? nullptr : const_cast<void*>(ptrs[i]);
        if (hipMemcpyAsync(t->d_table, t->h_table, n * sizeof(void*), hipMemcpyHostToDevice,
                           static_cast<hipStream_t>(stream)) != hipSuccess)
            rc = SPLC_EHIP;
    }
    if (rc != SPLC_OK) {
        sparseloco_tensors_release(t);
        return rc;
    }
    *out = t;
    return SPLC_OK;
}

void sparseloco_tensors_release(sparseloco_tensors* t) {
    if (!t) return;
    if (t->d_table) (void)hipFree(t->d_table);                     // waits for the device
    if (t->h_table) (void)hipHostFree(t->h_table);
    delete t;
}

int sparseloco_messages_bind(sparseloco_messages** out, const sparseloco_plan* plan, int n_replicas,
                             uint16_t* const* pairs, float* const* aux, void* stream) {
    if (!out) return SPLC_EINVAL;
    *out = nullptr;
    if (!plan || !pairs || !aux || n_replicas < 1 || n_replicas > SPLC_MAX_REPLICAS) return SPLC_EINVAL;
    for (int r = 0; r < n_replicas; ++r) {
        if (plan->n_chunks == 0) continue;
        if (!pairs[r] || !aux[r]) return SPLC_EINVAL;
        if (!aligned(pairs[r], 2) || !aligned(aux[r], 4)) return SPLC_EALIGN;
    }
    int rc = current_device_is(plan->device);
    if (rc != SPLC_OK) return rc;
    sparseloco_messages* m = new (std::nothrow) sparseloco_messages();
    if (!m) return SPLC_ENOMEM;
    m->device = plan->device;
    m->n_replicas = n_replicas;
    m->quant = plan->quant;
    m->kappa = plan->kappa;
    m->n_chunks = plan->n_chunks;
    const size_t nr = (size_t)n_replicas;
    m->disjoint = n_replicas == 1 || on_small_plan_disjoint(plan, [&](auto& ranges) {
        const uint64_t slots = (uint64_t)plan->n_chunks * (uint64_t)plan->kappa;
        for (size_t r = 0; r < nr; ++r) {
            ranges.push_back(range_of(pairs[r], 2 * slots));
            ranges.push_back(range_of(aux[r], 4 * (plan->quant == SPLC_QUANT_2BIT ? 2 * (uint64_t)plan->n_chunks : slots)));
        }
    });
    if ((rc = upload_table(2 * nr, &m->h_table, &m->d_table)) == SPLC_OK) {
        for (size_t r = 0; r < nr; ++r) {
            m->h_table[r] = pairs[r];
            m->h_table[nr + r] = aux[r];
        }
        if (hipMemcpyAsync(m->d_table, m->h_table, 2 * nr * sizeof(void*), hipMemcpyHostToDevice,
                           static_cast<hipStream_t>(stream)) != hipSuccess)
            rc = SPLC_EHIP;
    }
    if (rc != SPLC_OK) {
        sparseloco_messages_release(m);
        return rc;
    }
    *out = m;
    return SPLC_OK;
}

void sparseloco_messages_release(sparseloco_messages* m) {
    if (!m) return;
    if (m->d_table) (void)hipFree(m->d_table);
    if (m->h_table) (void)hipHostFree(m->h_table);
    delete m;
}

int sparseloco_compress(const sparseloco_plan* plan, int delta_mode, const sparseloco_tensors* src_a,
                        const sparseloco_tensors* src_b, const sparseloco_tensors* ef, int replica, float beta,
                        uint16_t* pairs_out, float* aux_out, void* stream) {
    if (!plan || !src_a || !ef || !pairs_out || !aux_out || replica < 0) return SPLC_EINVAL;
    int mode, rc;
    if (delta_mode == SPLC_DELTA_FROM_PARAMS) {
        if (!src_b) return SPLC_EINVAL;
        if ((rc = check_tensors(plan, src_a, SPLC_F32, 1)) != SPLC_OK) return rc;
        if ((rc = check_tensors(plan, src_b, SPLC_F32, 1)) != SPLC_OK) return rc;
        mode = MODE_PARAMS_F32;
    } else if (delta_mode == SPLC_DELTA_DIRECT) {
        if (src_b) return SPLC_EINVAL;
        if ((rc = check_tensors(plan, src_a, src_a->dtype, 1)) != SPLC_OK) return rc;
        mode = src_a->dtype == SPLC_BF16 ? MODE_DIRECT_BF16 : MODE_DIRECT_F32;
    } else {
        return SPLC_EINVAL;
    }
    if ((rc = check_tensors(plan, ef, SPLC_F32, 1)) != SPLC_OK) return rc;
    for (const sparseloco_tensors* t : {src_a, src_b, ef})
        if (t && t->n_sets > 1 && replica >= t->n_sets) return SPLC_EINVAL;
    if (!finite(beta)) return SPLC_EINVAL;
    if (!aligned(pairs_out, 2) || !aligned(aux_out, 4)) return SPLC_EALIGN;
    if ((rc = current_device_is(plan->device)) != SPLC_OK) return rc;
    if (plan->n_chunks == 0) return SPLC_OK;

    hipStream_t st = static_cast<hipStream_t>(stream);
    const void* const* da = set_table<const void*>(src_a, replica);
    const void* const* db = src_b ? set_table<const void*>(src_b, replica) : nullptr;
    float* const* de = set_table<float*>(ef, replica);
    const bool q2 = plan->quant == SPLC_QUANT_2BIT;
    switch (mode) {
        case MODE_PARAMS_F32:
            if (q2) launch_compress<MODE_PARAMS_F32, SPLC_QUANT_2BIT>(plan, da, db, de, beta, pairs_out, aux_out, st);
            else launch_compress<MODE_PARAMS_F32, SPLC_QUANT_NONE>(plan, da, db, de, beta, pairs_out, aux_out, st);
            break;
        case MODE_DIRECT_F32:
            if (q2) launch_compress<MODE_DIRECT_F32, SPLC_QUANT_2BIT>(plan, da, db, de, beta, pairs_out, aux_out, st);
            else launch_compress<MODE_DIRECT_F32, SPLC_QUANT_NONE>(plan, da, db, de, beta, pairs_out, aux_out, st);
            break;
        default:
            if (q2) launch_compress<MODE_DIRECT_BF16, SPLC_QUANT_2BIT>(plan, da, db, de, beta, pairs_out, aux_out, st);
            else launch_compress<MODE_DIRECT_BF16, SPLC_QUANT_NONE>(plan, da, db, de, beta, pairs_out, aux_out, st);
            break;
    }
    return hipGetLastError() == hipSuccess ? SPLC_OK : SPLC_EHIP;
}

int sparseloco_compress_batch(const sparseloco_plan* plan, int n_replicas, const sparseloco_tensors* theta_outer,
                              const sparseloco_tensors* theta_local, const sparseloco_tensors* ef, float beta,
                              const sparseloco_messages* messages_out, void* stream) {
    return compress_batch_impl(plan, n_replicas, theta_outer, theta_local, ef, beta, messages_out, false, 0.f, nullptr, 0,
                               stream);
}

int sparseloco_outer_step_batch(const sparseloco_plan* plan, int n_replicas, const sparseloco_tensors* theta_outer,
                                const sparseloco_tensors* theta_local, const sparseloco_tensors* ef, float beta,
                                float outer_lr, const sparseloco_messages* messages_out,
                                const sparseloco_tensors* delta_bar_out, int reset_theta_local, void* stream) {
    return compress_batch_impl(plan, n_replicas, theta_outer, theta_local, ef, beta, messages_out, true, outer_lr,
                               delta_bar_out, reset_theta_local ? 1 : 0, stream);
}

int sparseloco_aggregate(const sparseloco_plan* plan, const sparseloco_messages* messages,
                         const sparseloco_tensors* delta_bar_out, void* stream) {
    return aggregate_impl(plan, messages, delta_bar_out, nullptr, 0.f, false, nullptr, stream);
}

int sparseloco_aggregate_update(const sparseloco_plan* plan, const sparseloco_messages* messages,
                                const sparseloco_tensors* theta_outer, float outer_lr,
                                const sparseloco_tensors* delta_bar_out, const sparseloco_tensors* theta_local_reset,
                                void* stream) {
    return aggregate_impl(plan, messages, delta_bar_out, theta_outer, outer_lr, true, theta_local_reset, stream);
}

int sparseloco_outer_update(const sparseloco_plan* plan, const sparseloco_tensors* theta_outer,
                            const sparseloco_tensors* delta_bar, float outer_lr, void* stream) {
    if (!plan) return SPLC_EINVAL;
    int rc;
    if ((rc = check_tensors(plan, theta_outer, SPLC_F32, 1)) != SPLC_OK) return rc;
    if ((rc = check_tensors(plan, delta_bar, SPLC_F32, 1)) != SPLC_OK) return rc;
    if (theta_outer->n_sets != 1 || delta_bar->n_sets != 1 || !finite(outer_lr)) return SPLC_EINVAL;
    if ((rc = current_device_is(plan->device)) != SPLC_OK) return rc;
    if (plan->n_chunks == 0) return SPLC_OK;
    hipLaunchKernelGGL(outer_update_kernel, dim3((unsigned)plan->n_update), dim3(kThreads),
                       plan->n_update >= splc::kFewStreamsUpdate ? reserve_lds(2, 0) : 0u, static_cast<hipStream_t>(stream),
                       plan->d_update, (unsigned)plan->n_update_gen,
                       set_table<float*>(theta_outer, 0), set_table<const float*>(delta_bar, 0), outer_lr);
    return hipGetLastError() == hipSuccess ? SPLC_OK : SPLC_EHIP;
}

const char* sparseloco_strerror(int status) {
    switch (status) {
        case SPLC_OK: return "ok";
        case SPLC_EINVAL: return "invalid argument";
        case SPLC_EALIGN: return "tensor pointer not sufficiently aligned";
        case SPLC_ENOMEM: return "allocation failed";
        case SPLC_EHIP: return "HIP runtime call failed";
        case SPLC_EPLAN: return "call does not match the plan or a binding";
        case SPLC_ETOOBIG: return "problem exceeds the fixed workspace of this call";
        default: return "unknown status";
    }
}

}  // extern "C"
