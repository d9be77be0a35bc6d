// kernels_part.hip -- the divisible scheme's packing step on gfx950 (paper
// Sec. 3.1, Reason #2, and the alltoall figure: a compressed tensor is
// partitioned into parts and node j receives part j from every node, then
// decompresses, aggregates and compresses it again).
//
// Parts are element ranges [lo, hi) of every tensor.  Packing part j of a
// sparse payload keeps, tensor by tensor, the entries whose index lies in
// the range, in payload order, with the index rebased to the range; a sign
// or quantizer payload (b bits per element) keeps the words that cover the
// range (lo is a multiple of 32, so the range starts on a word) and every
// tensor's scale.  part_off receives the packed offsets of the tensors:
// entries (sparse) or words (sign, quantizers), T + 1 values.
#include "launch.hpp"

namespace bc {

namespace {

// First positions in [0, k) with idx[p] >= x0 and >= x1 (k if none), found
// by a whole wave, both searches advancing together (their loads are in
// flight at once): each round probes 64 evenly spaced positions of the
// interval that holds the answer and keeps the one gap between a probe
// below x and the next, so a round divides the interval by 65.
__device__ __forceinline__ void wave_lower_bounds(const uint32_t* idx, uint32_t k, const uint32_t (&x)[2],
                                                  uint32_t (&at)[2]) {
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t lo[2] = {0, 0}, hi[2] = {k, k};  // the answers lie in [lo, hi]
    at[0] = at[1] = 0;
    if (k == 0) return;
    while (hi[0] - lo[0] > 64u || hi[1] - lo[1] > 64u) {
        uint64_t len[2];
        uint32_t y[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            len[q] = hi[q] - lo[q];
            const uint32_t pos = lo[q] + (uint32_t)((len[q] * (lane + 1u)) / 65u);
            y[q] = len[q] > 64u ? gp(idx)[pos] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t c = (uint32_t)__popcll(__ballot(y[q] < x[q]));
            if (len[q] <= 64u) continue;
            const uint32_t nlo = c ? lo[q] + (uint32_t)((len[q] * c) / 65u) + 1u : lo[q];
            const uint32_t nhi = c < 64u ? lo[q] + (uint32_t)((len[q] * (c + 1u)) / 65u) : hi[q];
            lo[q] = nlo;
            hi[q] = nhi;
        }
    }
    bool below[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        below[q] = lo[q] + lane < hi[q] && gp(idx)[lo[q] + lane < hi[q] ? lo[q] + lane : 0u] < x[q];
#pragma unroll
    for (int q = 0; q < 2; ++q) at[q] = lo[q] + (uint32_t)__popcll(__ballot(below[q]));
}

}  // namespace

// Sparse packing takes two launches (three for large parts, launch_pack_part).
// part_count leaves in part_off[t] the
// range's first entry of tensor t (high 32 bits) and its number of entries
// (low 32 bits) and clears part_off[T]; part_copy_sparse turns the counts
// into offsets in every workgroup, copies, and counts its finished
// workgroups in part_off[T]: the last one, when nobody reads the counts any
// more, writes the offsets over them.  Launches and dependent loads bound
// both (a BERT-base part is 137 thousand entries, 2.2 MB): with the scan in
// a launch of its own and each workgroup walking its tensors one by one,
// searching each again, a pack took 28 us.
__global__ __launch_bounds__(kBlock) void part_count(const PDesc* __restrict__ p, int T,
                                                     const uint32_t* __restrict__ idx,
                                                     uint64_t* __restrict__ part_off) {
    if (blockIdx.x == 0 && threadIdx.x == 0) part_off[T] = 0;
    const int t = (int)(blockIdx.x * (kBlock / 64) + wave_id());
    if (t >= T) return;
    const PDesc pd = p[t];
    const uint32_t x[2] = {pd.lo, pd.hi};
    uint32_t at[2];
    wave_lower_bounds(idx + pd.in_off, pd.k, x, at);
    if (lane_id() == 0) part_off[t] = (uint64_t)at[0] << 32 | (uint64_t)(at[1] - at[0]);
}

// Each workgroup copies spans of packed positions, whose sources every thread
// finds by itself: a search over the offsets of 256 runs of tensors in LDS,
// then a walk along the run (one tensor up to 256 tensors), from the thread's
// position before if that lies in the run too.  The grid follows the entries
// expected of the part: each workgroup reads every tensor's count and adds to
// one counter (512 workgroups for 134 spans: 11 us, 135: 7 us).  Spans are 1024
// positions, four per thread, or 4096 where the part holds more than the grid
// covers so (entries crowded into one part, high ratios: 5 M entries 55 us with
// the short spans).
constexpr uint32_t kPackSpan = 1024;

namespace {

// Packed positions b0 .. b0 + kPer * kBlock - 1, as far as below total.
template <uint32_t kPer>
__device__ __forceinline__ void copy_span(const PDesc* __restrict__ p, uint32_t per, const uint32_t* in_idx,
                                          const float* in_val, uint32_t* out_idx, float* out_val,
                                          const uint64_t* part_off, const uint64_t* run_off, uint64_t b0,
                                          uint64_t total) {
    const uint64_t m = total - b0 < kPer * (uint64_t)kBlock ? total - b0 : kPer * (uint64_t)kBlock;
    uint64_t src[kPer];
    uint32_t lo[kPer], ix[kPer];
    float va[kPer];
    // the tensor of this thread's position (its word, and the positions of it
    // that come before) and where its run of tensors ends
    uint64_t end = 0, left = 0, w = 0, at = 0, prev = 0;
    uint32_t t = 0, first = 0;
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint32_t i = r * (uint32_t)kBlock + threadIdx.x;
        const uint64_t o = b0 + (i < m ? i : (uint32_t)m - 1u);  // past the end: a position to read, not written
        bool moved = r == 0;
        if (o >= end) {
            uint32_t run = 0;  // the last run that starts at or before o
#pragma unroll
            for (uint32_t b = kBlock / 2; b >= 1; b >>= 1)
                if (run_off[run + b] <= o) run += b;
            end = run + 1u < (uint32_t)kBlock ? run_off[run + 1u] : total;
            t = run * per;
            left = o - run_off[run];
            w = part_off[t];
            moved = true;
        } else {
            left += o - prev;
        }
        while (left >= (uint32_t)w) {
            left -= (uint32_t)w;
            w = part_off[++t];
            moved = true;
        }
        if (moved) {
            at = p[t].in_off + (w >> 32);
            first = p[t].lo;
        }
        src[r] = at + left;
        lo[r] = first;
        prev = o;
    }
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        ix[r] = gp(in_idx)[src[r]];
        va[r] = gp(in_val)[src[r]];
    }
#pragma unroll
    for (uint32_t r = 0; r < kPer; ++r) {
        const uint32_t i = r * (uint32_t)kBlock + threadIdx.x;
        if (i < m) {
            gp(out_idx)[b0 + i] = ix[r] - lo[r];
            gp(out_val)[b0 + i] = va[r];
        }
    }
}

}  // namespace

namespace {
// This thread's run of tensors, and the entries before it and of the part,
// from the counts in part_off.
struct Run {
    uint32_t per, t0, t1;
    uint64_t before, total;
};
__device__ __forceinline__ Run scan_counts(int T, const uint64_t* part_off, uint64_t* sh) {
    Run r;
    r.per = ((uint32_t)T + kBlock - 1u) / (uint32_t)kBlock;
    r.t0 = threadIdx.x * r.per < (uint32_t)T ? threadIdx.x * r.per : (uint32_t)T;
    r.t1 = r.t0 + r.per < (uint32_t)T ? r.t0 + r.per : (uint32_t)T;
    uint64_t mine = 0;
    for (uint32_t t = r.t0; t < r.t1; ++t) mine += (uint32_t)part_off[t];
    r.before = block_excl_scan_u64(mine, sh, r.total);
    return r;
}
// Offsets over the counts.
__device__ __forceinline__ void put_offsets(int T, const Run& r, uint64_t* part_off) {
    uint64_t run = r.before;
    for (uint32_t t = r.t0; t < r.t1; ++t) {
        const uint32_t c = (uint32_t)part_off[t];
        part_off[t] = run;
        run += c;
    }
    if (threadIdx.x == 0) part_off[T] = r.total;
}
}  // namespace

// kLarge: no counting of finished workgroups; part_offsets follows.
template <bool kLarge>
__global__ __launch_bounds__(kBlock) void part_copy_sparse(const PDesc* __restrict__ p, int T,
                                                           const uint32_t* __restrict__ in_idx,
                                                           const float* __restrict__ in_val,
                                                           uint32_t* __restrict__ out_idx,
                                                           float* __restrict__ out_val, uint64_t* part_off) {
    __shared__ uint64_t run_off[kBlock];
    __shared__ uint64_t sh[4];
    __shared__ int last_sh;
    const Run r = scan_counts(T, part_off, sh);
    run_off[threadIdx.x] = r.before;
    __syncthreads();
    if (r.total <= (uint64_t)gridDim.x * kPackSpan) {
        const uint64_t b0 = (uint64_t)blockIdx.x * kPackSpan;
        if (b0 < r.total)
            copy_span<kPackSpan / kBlock>(p, r.per, in_idx, in_val, out_idx, out_val, part_off, run_off, b0, r.total);
    } else {
        const uint64_t step = (uint64_t)gridDim.x * 4 * kPackSpan;
        for (uint64_t b0 = (uint64_t)blockIdx.x * 4 * kPackSpan; b0 < r.total; b0 += step)
            copy_span<4 * kPackSpan / kBlock>(p, r.per, in_idx, in_val, out_idx, out_val, part_off, run_off, b0,
                                              r.total);
    }
    if (kLarge) return;
    // done with the counts; the last workgroup replaces them.  Only reads
    // come before this point that it could overtake, and the barrier waits
    // for their data, so the addition needs no release (which would write
    // back the L2: 9 us of the kernel's 14)
    __syncthreads();
    if (threadIdx.x == 0)
        last_sh = __hip_atomic_fetch_add((unsigned long long*)part_off + T, 1ull, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) == (unsigned long long)gridDim.x - 1ull;
    __syncthreads();
    if (last_sh) put_offsets(T, r, part_off);
}

__global__ __launch_bounds__(kBlock) void part_offsets(int T, uint64_t* part_off) {
    __shared__ uint64_t sh[4];
    put_offsets(T, scan_counts(T, part_off, sh), part_off);
}

// Sign and quantizers (`bits` per element): copy tensor t's range words
// and its scale; part_off gets the (host-computed) word offsets.  kLong (some
// range is longer than kPackWords words): the workgroups of a column share a
// tensor in pieces of as many, eight loads in flight per thread (one
// workgroup for BERT-base's embedding, 2.9 MB of 8-bit codes, would run on
// alone long after the others).  Otherwise no more loads than words: 4096
// tensors of up to 2048 words 30 us, 38 with the piece loop.
constexpr uint32_t kPackWords = 2048;

template <bool kLong>
__global__ __launch_bounds__(kBlock) void part_copy_words(const PDesc* __restrict__ p, int T, uint32_t bits,
                                                          const uint32_t* __restrict__ in_bits,
                                                          const float* __restrict__ in_scale,
                                                          uint32_t* __restrict__ out_bits,
                                                          float* __restrict__ out_scale,
                                                          uint64_t* __restrict__ part_off, uint64_t total) {
    for (int t = blockIdx.x; t < T; t += gridDim.x) {
        const PDesc pd = p[t];
        // bits per element: the range starts on a word (lo is a multiple of 32)
        const uint32_t nw = (uint32_t)(((uint64_t)(pd.hi - pd.lo) * bits + 31u) / 32u);
        const uint64_t src = pd.in_off + (uint64_t)pd.lo / 32u * bits;
        if constexpr (kLong) {
            for (uint64_t b = (uint64_t)blockIdx.y * kPackWords; b < nw; b += (uint64_t)gridDim.y * kPackWords) {
                uint32_t x[kPackWords / kBlock];
#pragma unroll
                for (uint32_t r = 0; r < kPackWords / kBlock; ++r) {
                    const uint64_t i = b + r * (uint32_t)kBlock + threadIdx.x;
                    x[r] = gp(in_bits)[src + (i < nw ? i : b)];
                }
#pragma unroll
                for (uint32_t r = 0; r < kPackWords / kBlock; ++r) {
                    const uint64_t i = b + r * (uint32_t)kBlock + threadIdx.x;
                    if (i < nw) gp(out_bits)[pd.out_off + i] = x[r];
                }
            }
        } else {
            for (uint32_t i = threadIdx.x; i < nw; i += kBlock) out_bits[pd.out_off + i] = gp(in_bits)[src + i];
        }
        if ((!kLong || blockIdx.y == 0) && threadIdx.x == 0) {
            out_scale[t] = gp(in_scale)[t];
            part_off[t] = pd.out_off;
            if (t == 0) part_off[T] = total;
        }
    }
}

hipError_t launch_pack_part(int word_bits, const PDesc* p, int T, bc_payload_dev in, bc_payload_dev out,
                            uint64_t* part_off, uint64_t words, uint64_t max_words, uint64_t expected, int cus,
                            hipStream_t s) {
    if (T <= 0) return hipSuccess;
    const uint32_t grid = (uint32_t)(T < 4 * cus ? T : 4 * cus);
    if (word_bits) {
        // pieces of the longest range, while the grid (mostly idle where the
        // other tensors are short) stays under 64 workgroups per compute unit
        uint64_t pieces = (max_words + kPackWords - 1) / kPackWords;
        if (pieces > 64u * (uint64_t)cus / grid) pieces = 64u * (uint64_t)cus / grid;
        if (pieces > 1)
            hipLaunchKernelGGL(part_copy_words<true>, dim3(grid, (uint32_t)pieces), dim3(kBlock), 0, s, p, T,
                               (uint32_t)word_bits, in.bits, in.scale, out.bits, out.scale, part_off, words);
        else
            hipLaunchKernelGGL(part_copy_words<false>, dim3(grid), dim3(kBlock), 0, s, p, T, (uint32_t)word_bits,
                               in.bits, in.scale, out.bits, out.scale, part_off, words);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(part_count, dim3((T + 3) / 4), dim3(kBlock), 0, s, p, T, in.idx, part_off);
    // above one short span per compute unit (262 thousand entries) as many
    // workgroups as long spans, and a third launch in place of their additions
    // to one counter: 500 thousand entries 20 us, 22 with the counter, 5 M 30
    // and 55; a BERT-base part's 137 thousand 16 with the counter
    uint64_t blocks = expected / kPackSpan + 1;
    if (blocks <= (uint64_t)cus) {
        hipLaunchKernelGGL(part_copy_sparse<false>, dim3((uint32_t)blocks), dim3(kBlock), 0, s, p, T, in.idx, in.val,
                           out.idx, out.val, part_off);
    } else {
        blocks = expected / (4 * kPackSpan) + 1;
        if (blocks > 16u * (uint64_t)cus) blocks = 16u * (uint64_t)cus;
        hipLaunchKernelGGL(part_copy_sparse<true>, dim3((uint32_t)blocks), dim3(kBlock), 0, s, p, T, in.idx, in.val,
                           out.idx, out.val, part_off);
        hipLaunchKernelGGL(part_offsets, dim3(1), dim3(kBlock), 0, s, T, part_off);
    }
    return hipGetLastError();
}

}  // namespace bc
