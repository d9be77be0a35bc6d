// common.hpp -- device-side descriptors and helpers shared by the gfx950
// kernels of the compression library.  Everything here is product code;
// nothing is shared with the CPU oracle.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bc {

// ---------------------------------------------------------------- geometry
// Streaming passes: one 256-thread workgroup (four wave64s) owns a chunk of
// 4096 consecutive elements of one tensor; thread j holds elements
// 1024*r + 4*j + q (r, q = 0..3) so every load instruction of a wave reads
// 1 KiB of fp32 contiguously.
constexpr int kBlock = 256;
constexpr int kChunk = 4096;
constexpr int kEpt = kChunk / kBlock;     // 16 elements per thread
constexpr int kRounds = 4;                // 4 rounds of 1024 elements
constexpr int kChunkWords = kChunk / 32;  // 128 sign words per chunk
constexpr int kBins0 = 2048;              // radix digit 0: key bits 30..20
constexpr int kBins12 = 1024;             // radix digits 1, 2: bits 19..10, 9..0

// ------------------------------------------------------------ descriptors
// One tensor of a compress or residual-update call (48 bytes).
struct TDesc {
    const void* grad;
    float* resid;       // nullptr: error feedback off
    uint32_t n;
    uint32_t dtype;     // 0 fp32, 1 fp16
    uint32_t tid;
    uint32_t k;         // sparse: k_t; sign: word count
    uint64_t off;       // payload offset of this tensor (entries or words)
    uint32_t chunk0;    // first global chunk index
    uint32_t nchunks;
};
static_assert(sizeof(TDesc) == 48, "TDesc layout");

// One tensor of a pack-part call (32 bytes): its payload offset and count
// (entries, or words for sign), the part's element range, and (sign) the
// part's word offset in the packed layout.
struct PDesc {
    uint64_t in_off;
    uint64_t out_off;
    uint32_t k;
    uint32_t lo, hi;
    uint32_t pad;
};
static_assert(sizeof(PDesc) == 32, "PDesc layout");

// Device pointers of one payload (the C-ABI bc_payload, without torch).
struct bc_payload_dev {
    uint32_t* idx;
    float* val;
    uint32_t* bits;
    float* scale;
};

// One tensor of an aggregate call (32 bytes).
struct ADesc {
    float* out;
    uint32_t n;
    uint32_t k;         // sparse: k_t; sign: word count
    uint64_t off;       // payload offset (same for every worker)
    uint32_t unit0;     // first global work unit (tile / wave chunk)
    uint32_t nunits;
};
static_assert(sizeof(ADesc) == 32, "ADesc layout");

// One worker's payload in an aggregate call.
// Worker table of the aggregate descriptor (pointers stored as uint64):
// a[Wp] (sparse: idx, sign: bits), then b[Wp] (sparse: val, sign: scale),
// then the unit -> tensor map; Wp = padded_workers(W) (below) and the
// slots past W repeat worker W-1.

// Largest t with d[t].chunk0 <= c (tensors without chunks share chunk0 with
// their successor, so the search lands on the tensor that owns chunk c).
template <typename D, uint32_t D::*Field>
__device__ __forceinline__ int find_owner(const D* __restrict__ d, int T, uint32_t c) {
    int lo = 0, hi = T - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (d[mid].*Field <= c) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The device descriptor table of a call is followed by a chunk -> tensor
// map (one uint32 per chunk), built on the host when the table is cached.
__device__ __forceinline__ int tensor_of_chunk(const TDesc* __restrict__ d, int T, uint32_t c) {
    return (int)reinterpret_cast<const uint32_t*>(d + T)[c];
}

// The chunk that workgroup b of a second pass over `chunks` chunks takes: the
// last ones first, whose v the first pass (in order) left in the last-level
// cache, but in groups of eight that keep their order, as workgroups are dealt
// to the eight compute dies in turn and a chunk's v may still be in the L2 of
// the die that wrote it (a sign call of 6 M elements 28 us, 32 backwards one
// by one).
__device__ __forceinline__ uint32_t backward_chunk(uint32_t b, uint32_t chunks) {
    const uint32_t groups = chunks / 8u;
    return b / 8u < groups ? 8u * (groups - 1u - b / 8u) + b % 8u : b;
}

// Pointers read from descriptor tables are generic; viewing them in the
// global address space lets the compiler use global (not flat) memory
// instructions with scalar base addresses.
#define BC_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ BC_GLOBAL T* gp(T* p) { return (BC_GLOBAL T*)p; }
template <typename T>
__device__ __forceinline__ const BC_GLOBAL T* gp(const T* p) { return (const BC_GLOBAL T*)p; }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// 16- and 8-byte global loads/stores (addresses aligned accordingly)
__device__ __forceinline__ f32x4 ldg4f(const float* p) { return *(const BC_GLOBAL f32x4*)p; }
__device__ __forceinline__ u32x4 ldg4u(const void* p) { return *(const BC_GLOBAL u32x4*)p; }
__device__ __forceinline__ u32x2 ldg2u(const void* p) { return *(const BC_GLOBAL u32x2*)p; }
__device__ __forceinline__ void stg4f(float* p, f32x4 v) { *(BC_GLOBAL f32x4*)p = v; }
// The same with the non-temporal hint when kNT: streaming passes over
// tensor sets larger than the last-level cache skip allocating their lines
// (measured: a two-read-one-write stream over 1.5 G elements moves 6.2 TB/s
// this way against 5.5 TB/s with cached accesses).
template <bool kNT>
__device__ __forceinline__ f32x4 ldg4f_s(const float* p) {
    if constexpr (kNT) return __builtin_nontemporal_load((const BC_GLOBAL f32x4*)p);
    else return *(const BC_GLOBAL f32x4*)p;
}
template <bool kNT>
__device__ __forceinline__ u32x2 ldg2u_s(const void* p) {
    if constexpr (kNT) return __builtin_nontemporal_load((const BC_GLOBAL u32x2*)p);
    else return *(const BC_GLOBAL u32x2*)p;
}
template <bool kNT>
__device__ __forceinline__ void stg4f_s(float* p, f32x4 v) {
    if constexpr (kNT) __builtin_nontemporal_store(v, (BC_GLOBAL f32x4*)p);
    else *(BC_GLOBAL f32x4*)p = v;
}

// ------------------------------------------------------------- bit helpers
__device__ __forceinline__ uint32_t f2u(float x) { return __float_as_uint(x); }
__device__ __forceinline__ float u2f(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ uint32_t key_of(float x) { return f2u(x) & 0x7FFFFFFFu; }

// IEEE binary16 bits -> fp32 (exact, subnormals included: v_cvt_f32_f16
// with fp16 denormals enabled, the HIP default).
__device__ __forceinline__ float h2f(uint32_t bits16) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }
__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// ----------------------------------------------------------- chunk loading
// Every chunk is read by the same straight-line code, which issues all of a
// thread's vector loads before it uses any of them, so that they are in
// flight together.  In a tensor's last chunk, groups of four that reach past
// the tensor's end read its last four elements instead (an address that may
// be aligned to an element only, which the hardware's vector loads take), and
// mend_tail puts what exists into place.  Only tensors of fewer than four
// elements are read one by one.  (A last chunk read element by element cost
// a list of 4096 tensors of 768 to 65536 elements, a quarter of whose
// chunks are last ones, 10 us of a 260 us sign step.)  The tests are
// uniform over the workgroup (one chunk, one tensor).
__device__ __forceinline__ bool whole_chunk(const TDesc& td, uint32_t j) {
    return (uint64_t)j * kChunk + kChunk <= td.n;
}

typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
// Four consecutive elements from element i of p on, any i.
template <bool kNT = false>
__device__ __forceinline__ f32x4 ldg4f_any(const float* p, uint32_t i) {
    const BC_GLOBAL f32x4_any* at = (const BC_GLOBAL f32x4_any*)((const BC_GLOBAL char*)p + 4u * i);
    if constexpr (kNT) return __builtin_nontemporal_load(at);
    else return *at;
}
template <bool kNT = false>
__device__ __forceinline__ u32x2 ldg4h_any(const uint16_t* p, uint32_t i) {
    const BC_GLOBAL u32x2_any* at = (const BC_GLOBAL u32x2_any*)((const BC_GLOBAL char*)p + 2u * i);
    if constexpr (kNT) return __builtin_nontemporal_load(at);
    else return *at;
}

// A thread's load of round r of chunk j covers its own group of four, or the
// tensor's last four elements (n >= 4): element load_base + load_at of the
// tensor.  The base is uniform (the group before the chunk, where a last
// chunk of fewer than four elements reaches back to) and the rest a small
// 32-bit offset, so that the loads need no 64-bit addresses per thread.
__device__ __forceinline__ size_t load_base(uint32_t j) { return j ? (size_t)j * kChunk - 4u : 0u; }
__device__ __forceinline__ uint32_t load_at(uint32_t n, uint32_t j, int r) {
    const uint32_t e = (j ? 4u : 0u) + 1024u * r + 4u * threadIdx.x;
    const uint32_t last = n - 4u - (uint32_t)load_base(j);
    return e < last ? e : last;
}

// Which of a thread's elements exist in chunk j of a tensor of n elements.
__device__ __forceinline__ uint32_t valid_of(uint32_t n, uint32_t j) {
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t e = j * (uint32_t)kChunk + 1024u * r + 4u * threadIdx.x;
        const uint32_t left = e < n ? n - e : 0u;
        m |= (left >= 4u ? 0xFu : (1u << left) - 1u) << (4 * r);
    }
    return m;
}

// v formed from a last chunk's loads: the group that straddles the tensor's
// end holds the last four elements and keeps those from its first on; the
// elements past the end become +0.0.
__device__ __forceinline__ void mend_tail(uint32_t n, uint32_t valid, float (&v)[kEpt]) {
    // elements of the straddling group (its first one is loaded last - rest);
    // a tensor of fewer than four elements is in place already
    const uint32_t rest = n >= 4u ? n & 3u : 0u;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t m = (valid >> (4 * r)) & 0xFu;
        const float x0 = v[4 * r], x1 = v[4 * r + 1], x2 = v[4 * r + 2], x3 = v[4 * r + 3];
        const bool cut = m != 0xFu;
        const float y0 = !cut || rest == 0u ? x0 : rest == 1u ? x3 : rest == 2u ? x2 : x1;
        const float y1 = !cut || rest == 0u ? x1 : rest == 2u ? x3 : x2;
        const float y2 = !cut || rest == 0u ? x2 : x3;
        v[4 * r] = m & 1u ? y0 : 0.f;
        v[4 * r + 1] = m & 2u ? y1 : 0.f;
        v[4 * r + 2] = m & 4u ? y2 : 0.f;
        v[4 * r + 3] = m & 8u ? x3 : 0.f;
    }
}

// Widened gradient element q (0..3) of a thread's round: fp32 bits, or the
// fp16 halves of two packed words.
template <int DT>
__device__ __forceinline__ float g_elem(const f32x4& gf, const u32x2& gh, int q) {
    if constexpr (DT == 0) return gf[q];
    else return h2f(((q < 2 ? gh.x : gh.y) >> (16 * (q & 1))) & 0xFFFFu);
}

// Elements 0, 1 and 2 of a tensor of fewer than four (the last again where
// there are fewer: mend_tail keeps what exists, in thread 0).
template <int DT>
__device__ __forceinline__ float tiny_elem(const TDesc& td, uint32_t q, bool use_resid) {
    const uint32_t i = q < td.n ? q : td.n - 1u;
    const float g = DT == 0 ? gp((const float*)td.grad)[i] : h2f(gp((const uint16_t*)td.grad)[i]);
    return use_resid ? g + gp(td.resid)[i] : g;
}
template <int DT>
__device__ __forceinline__ void load_tiny(const TDesc& td, bool use_resid, float (&v)[kEpt]) {
    v[0] = tiny_elem<DT>(td, 0, use_resid);
    v[1] = tiny_elem<DT>(td, 1, use_resid);
    v[2] = tiny_elem<DT>(td, 2, use_resid);
}

// Load the 16 elements a thread owns of chunk `j` of tensor `td`, forming
// v = widen(g) + e (e = 0 when there is no residual or `use_resid` is
// false).  Elements past the tensor's end read as +0.0 and are reported
// invalid through `valid` (bit 4*r + q).
template <int DT, bool kNT = false>
__device__ __forceinline__ void load_chunk(const TDesc& td, uint32_t j, bool use_resid,
                                           float (&v)[kEpt], uint32_t& valid) {
    const uint32_t n = td.n;
    if (n >= 4u) {
        f32x4 gf[kRounds];
        u32x2 gh[kRounds];
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            if constexpr (DT == 0) gf[r] = ldg4f_any<kNT>((const float*)td.grad + load_base(j), load_at(n, j, r));
            else gh[r] = ldg4h_any<kNT>((const uint16_t*)td.grad + load_base(j), load_at(n, j, r));
        }
        if (use_resid) {
            f32x4 ev[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r) ev[r] = ldg4f_any<kNT>(td.resid + load_base(j), load_at(n, j, r));
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[4 * r + q] = g_elem<DT>(gf[r], gh[r], q) + ev[r][q];
        } else {
#pragma unroll
            for (int r = 0; r < kRounds; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[4 * r + q] = g_elem<DT>(gf[r], gh[r], q);
        }
    } else {
#pragma unroll
        for (int i = 0; i < kEpt; ++i) v[i] = 0.f;
        load_tiny<DT>(td, use_resid, v);
    }
    valid = 0xFFFFu;
    if (!whole_chunk(td, j)) {
        valid = valid_of(n, j);
        mend_tail(n, valid, v);
    }
}

// Runtime dtype dispatch (uniform per workgroup: a chunk has one tensor).
template <bool kNT = false>
__device__ __forceinline__ void load_v(const TDesc& td, uint32_t j, bool use_resid, float (&v)[kEpt],
                                       uint32_t& valid) {
    if (td.dtype == 0) load_chunk<0, kNT>(td, j, use_resid, v, valid);
    else load_chunk<1, kNT>(td, j, use_resid, v, valid);
}

// Raw chunk data held in registers between issuing the loads and using
// them (lets a kernel prefetch its next chunk before a wait).  g[4r + q]
// holds element 4r + q's fp32 bits or, for fp16 gradients, g[4r] and
// g[4r + 1] hold round r's four elements as packed halves (low half
// first); e is written only when the residual is read.
struct RawChunk {
    uint32_t g[kEpt];
    float e[kEpt];
};

// The loads are non-temporal: the one-pass kernels, which use this, read
// every gradient and residual once and write the residual once.
// kDT: 0 every tensor of the call is fp32, 1 every tensor is fp16, 2 both
// occur (td.dtype decides).  A kernel that keeps loads in flight across
// iterations is instantiated per kDT so that the common single-dtype calls
// have one load sequence (no merge of two register sets that would make
// the compiler wait for the loads).  For the same reason tensors of fewer
// than four elements take it too, on their descriptor's first 16 bytes
// (dsc: any descriptor of the call); raw_to_v reads their elements.
template <int kDT>
__device__ __forceinline__ void load_raw(const TDesc* dsc, const TDesc& td, uint32_t j, bool use_resid, RawChunk& r) {
    if constexpr (kDT == 2) {
        if (td.dtype == 0) load_raw<0>(dsc, td, j, use_resid, r);
        else load_raw<1>(dsc, td, j, use_resid, r);
    } else {
        const bool tiny = td.n < 4u;
        const uint32_t n = tiny ? 4u : td.n;  // load_at: 0 for all
        const void* g = tiny ? (const void*)dsc : td.grad;
        const float* e = tiny ? (const float*)dsc : td.resid;
#pragma unroll
        for (int rr = 0; rr < kRounds; ++rr) {
            if constexpr (kDT == 0) {
                const f32x4 x = ldg4f_any<true>((const float*)g + load_base(j), load_at(n, j, rr));
#pragma unroll
                for (int q = 0; q < 4; ++q) r.g[4 * rr + q] = f2u(x[q]);
            } else {
                const u32x2 h = ldg4h_any<true>((const uint16_t*)g + load_base(j), load_at(n, j, rr));
                r.g[4 * rr] = h.x;
                r.g[4 * rr + 1] = h.y;
            }
        }
        if (use_resid) {
#pragma unroll
            for (int rr = 0; rr < kRounds; ++rr) {
                const f32x4 y = ldg4f_any<true>(e + load_base(j), load_at(n, j, rr));
#pragma unroll
                for (int q = 0; q < 4; ++q) r.e[4 * rr + q] = y[q];
            }
        }
    }
}

// v = widen(g) + e from a RawChunk (e = 0 without residual), exactly as
// load_v forms it; elements past the tensor's end read as +0.0.  Returns
// which exist.
template <int kDT>
__device__ __forceinline__ uint32_t raw_to_v(const TDesc& td, uint32_t j, bool use_resid, const RawChunk& r,
                                             float (&v)[kEpt]) {
    const bool f16 = kDT == 1 || (kDT == 2 && td.dtype != 0);
#pragma unroll
    for (int i = 0; i < kEpt; ++i) {
        const float g = f16 ? h2f((r.g[(i & ~3) + ((i >> 1) & 1)] >> (16 * (i & 1))) & 0xFFFFu) : u2f(r.g[i]);
        v[i] = use_resid ? g + r.e[i] : g;
    }
    if (whole_chunk(td, j)) return 0xFFFFu;
    if (td.n < 4u) {
        if (f16) load_tiny<1>(td, use_resid, v);
        else load_tiny<0>(td, use_resid, v);
    }
    const uint32_t valid = valid_of(td.n, j);
    mend_tail(td.n, valid, v);
    return valid;
}

// Load v that an earlier pass already stored (the residual buffer holds v),
// or recompute it from the gradient when error feedback is off.
__device__ __forceinline__ void load_stored_v(const TDesc& td, uint32_t j, float (&v)[kEpt],
                                              uint32_t& valid) {
    if (td.resid) {
        TDesc te = td;  // v as an fp32 tensor of its own
        te.grad = td.resid;
        load_chunk<0>(te, j, false, v, valid);
    } else if (td.dtype == 0) {
        load_chunk<0>(td, j, false, v, valid);
    } else {
        load_chunk<1>(td, j, false, v, valid);
    }
}

// Store 16 per-thread values back to a dense fp32 tensor (same pattern).
template <bool kNT = false>
__device__ __forceinline__ void store_chunk(float* dst, uint32_t n, uint32_t j, const float v[kEpt]) {
    const uint32_t base = j * (uint32_t)kChunk;
    if ((uint64_t)base + kChunk <= n) {
#pragma unroll
        for (int r = 0; r < kRounds; ++r)
            stg4f_s<kNT>(dst + base + 1024u * r + 4u * threadIdx.x,
                         f32x4{v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]});
        return;
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t e0 = base + 1024u * r + 4u * threadIdx.x;
        if (e0 + 3 < n) {
            stg4f_s<kNT>(dst + e0, f32x4{v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]});
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (e0 + q < n) gp(dst)[e0 + q] = v[4 * r + q];
        }
    }
}

// A unit of 4096 results, of which lane l of the workgroup holds elements
// 16 l .. 16 l + 15, on its way to coalesced stores through LDS: written so,
// every store instruction of the workgroup covers 4 KiB of the output
// without gaps (lane-wise 64-byte pieces left each instruction a quarter of
// every line).  The four 16-byte pieces of a lane are rotated by l / 4, so
// that neither side meets a bank conflict.
__device__ __forceinline__ uint32_t staged_at(uint32_t piece) {
    const uint32_t l = piece >> 2;
    return 16u * l + 4u * ((piece + (l >> 2)) & 3u);
}
__device__ __forceinline__ void stage_results(float* lds, const float (&res)[16]) {
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c)
        *reinterpret_cast<f32x4*>(lds + staged_at(4u * threadIdx.x + c)) =
            f32x4{res[4 * c], res[4 * c + 1], res[4 * c + 2], res[4 * c + 3]};
}
// After a barrier: piece k of this lane, elements 1024 k + 4 l .. + 3.
__device__ __forceinline__ f32x4 staged_piece(const float* lds, uint32_t k) {
    return *reinterpret_cast<const f32x4*>(lds + staged_at(256u * k + threadIdx.x));
}

// --------------------------------------------------------- block reductions
// Sum of a double over the 256 threads in a fixed tree (deterministic for a
// given block shape); every thread receives the total.
__device__ __forceinline__ double block_sum_f64(double x, double* sh /* >= 4 */) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane_id() == 0) sh[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return t;
}

// Exclusive prefix of a 64-bit value over the block (thread order), plus
// the block total.  `sh` needs 4 entries.
__device__ __forceinline__ uint64_t block_excl_scan_u64(uint64_t x, uint64_t* sh, uint64_t& total) {
    const int lane = lane_id();
    uint64_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint64_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[threadIdx.x >> 6] = inc;
    __syncthreads();
    const int w = threadIdx.x >> 6;
    uint64_t before = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) before += (q < w) ? sh[q] : 0;
    total = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return before + inc - x;
}

// ------------------------------------------------------- device atomics
__device__ __forceinline__ uint32_t atomic_add_agent(uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t atomic_load_acquire(uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_store_release(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_store_relaxed(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------- Philox
// Philox4x64-10 counter-based generator (Salmon et al., SC'11): ten rounds
// of two 64x64->128-bit multiplies on counter words 0 and 2, a fixed word
// permutation and xor with the remaining words and the key; the key is
// advanced by the two Weyl constants before every round but the first.
struct U64x4 { uint64_t v[4]; };

__host__ __device__ inline void mul_hilo64(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo) {
#if defined(__HIP_DEVICE_COMPILE__)
    // the 128-bit product from four 32x32+64-bit multiply-adds (v_mad_u64_u32),
    // sharing the partial products between the two halves; no sum overflows:
    // (2^32 - 1)^2 + (2^32 - 1) < 2^64
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
    const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
    const uint64_t p00 = (uint64_t)a0 * b0;
    const uint64_t p10 = (uint64_t)a1 * b0 + (p00 >> 32);
    const uint64_t p01 = (uint64_t)a0 * b1 + (uint32_t)p10;
    hi = (uint64_t)a1 * b1 + (p10 >> 32) + (p01 >> 32);
    lo = (p01 << 32) | (uint32_t)p00;
#else
    unsigned __int128 p = (unsigned __int128)a * b;
    hi = (uint64_t)(p >> 64);
    lo = (uint64_t)p;
#endif
}

__host__ __device__ inline U64x4 philox4x64_10(U64x4 c, uint64_t k0, uint64_t k1) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) { k0 += W0; k1 += W1; }
        uint64_t h0, l0, h1, l1;
        mul_hilo64(M0, c.v[0], h0, l0);
        mul_hilo64(M1, c.v[2], h1, l1);
        U64x4 o;
        o.v[0] = h1 ^ c.v[1] ^ k0;
        o.v[1] = l1;
        o.v[2] = h0 ^ c.v[3] ^ k1;
        o.v[3] = l0;
        c = o;
    }
    return c;
}

// Random-stream ids (second key word).
constexpr uint64_t kStreamRandk = 0;
constexpr uint64_t kStreamSample = 1;
constexpr uint64_t kStreamQuant = 2;

// Workspace header: failure flags reported by bytecomp_device_status.  No
// current kernel sets one: the one-pass compress kernels wait for other
// workgroups, but only for a bounded time, and a wait that runs out takes
// a path whose results are exact (the workgroup computes the missing
// partials itself), so it is no failure.

// --------------------------------------------- one-pass compress protocol
// A one-pass compress kernel defers each chunk's residual (and, for the
// quantizers, its codes) until its tensor's scale is known, which needs a
// published partial (a sum of |v|, or a largest |v|) of every chunk of the
// tensor.  A workgroup waits for missing partials only for a bounded time;
// then it computes each still-missing partial itself, from the chunk's
// gradient and residual, with exactly the owner's arithmetic (so the value
// is bit-identical), and publishes it by compare-and-swap from empty: if the
// owner published first, the owner's value stays.  The owner writes the
// chunk's residual only once its tensor's partials are all published, and a
// helper reads the chunk's residual only while its partial is still
// missing, so a helper's publication never rests on a residual the owner
// has already overwritten (had the owner begun, its partial would be
// published and the helper's swap would fail).  Every wait therefore ends
// after at most the limit plus the workgroup's own work, whatever the
// residency of the grid.

// ------------------------------------------------- aggregate worker table
// Worker descriptors in the aggregate table are padded to a multiple of 16.
__host__ __device__ constexpr int padded_workers(int W) { return (W + 15) & ~15; }

// The aggregate table is [ADesc x T][a x Wp][b x Wp][unit -> tensor map]
// with Wp = padded_workers(W); slots past W repeat worker W-1.
__device__ __forceinline__ const uint32_t* w_a(const uint64_t* __restrict__ wp, int w) {
    return (const uint32_t*)wp[w];
}
__device__ __forceinline__ const float* w_b(const uint64_t* __restrict__ wp, int W, int w) {
    return (const float*)wp[padded_workers(W) + w];
}
__device__ __forceinline__ int unit_owner(const uint64_t* __restrict__ wp, int W, uint32_t u) {
    return (int)reinterpret_cast<const uint32_t*>(wp + 2 * padded_workers(W))[u];
}

// Tensor whose payload entries hold flattened entry j: the last tensor
// with off <= j (tensors without entries share the next one's offset).
__device__ __forceinline__ int tensor_of_entry(const TDesc* __restrict__ d, int T, uint64_t j) {
    int lo = 0, hi = T - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (d[mid].off <= j) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// First position p in [0, k) with idx[p] >= x (k if none).
__device__ __forceinline__ uint32_t lower_bound_u32(const uint32_t* idx, uint32_t k, uint32_t x) {
    uint32_t lo = 0, hi = k;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (gp(idx)[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}


}  // namespace bc
