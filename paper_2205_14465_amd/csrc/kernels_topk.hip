// kernels_topk.hip -- top-k sparsification with error feedback on gfx950:
// exact top-k and the DGC-style sampled-threshold variant (paper Sec. 2.3,
// sparsification; Sec. 5.1, DGC at a 1% rate with error feedback).
//
// Result (both kinds): the k_t entries of v = g + e_old with the largest
// |v| (keys = magnitude bits), ties to the lower index, emitted with
// ascending indices and values v[idx]; residual e_new = v with the chosen
// entries set to +0.0.
//
// Pipeline (all tensors of a call advance together, one launch per step):
//   exact:    stream pass 1 writes e_new = v and a 2048-bin histogram of
//             key bits 30..20 per tensor -> exact bin of the k-th key ->
//             stream pass 2 re-reads v and compacts the candidates (keys at
//             or above that bin) per 4096-element chunk, in index order.
//   sampled:  one workgroup per tensor draws a seeded sample (up to 16384
//             elements in runs of 16) and takes a threshold with a margin
//             from it, to 2^-13 of the value -> ONE stream pass writes e_new
//             and compacts candidates.  Tensors of fewer than 16384 elements
//             are read whole instead and go by their exact threshold.  If a
//             tensor ends with fewer than k candidates, the exact histogram
//             path runs for that tensor only; if its k-th key lies above the
//             range the sample promised, its candidates are binned again.
//   both:     the pass that compacts the candidates also histograms them in
//             2048 bins of 2^s keys counted from the threshold; the k-th
//             candidate's bin A follows, then one pass over the candidates
//             counts those above bin A in each chunk and histograms the few
//             inside it by their low s bits, and one workgroup per tensor
//             finds the k-th key tau from those and places every chunk's
//             winners (a scan over the chunks); the emit pass writes the
//             payload and zeroes e_new at the winners.  Keys counted from the
//             threshold need one pass over the candidates where fixed digits
//             (11, 10, 10 bits) took three.
// The sampled stream pass writes +0.0 into e_new already at the candidates
// far enough above the threshold to be winners (a lower estimate of how many
// keys lie above still says so): scattered 4-byte stores are what the emit
// pass is bound by, and up to three quarters of them fall away.  Should such
// a candidate lose after all, the emit pass writes its v back.
// BERT-base at 1% (199 tensors, 109.5 M elements): seven launches instead of
// sixteen, 286 instead of 423 us a call, of which the stream pass, at the
// memory's rate (6.3 TB/s), takes 208, the threshold 19, the emit pass 15 (51
// before; 22 instead of 102 under DGC), placing 12, counting 9, the bin search
// 5 and the fallback 4.5 where no tensor needs it.  In 3000 such calls on new
// gradients 12 had one tensor of fewer than k candidates: mean 280.9, median
// 280.3, longest 336 us.  The margin of a quarter and 16 is about 4.5 standard
// deviations of the sample's count; a fallback now costs a fifth of a call, so
// a wider one would save less than 0.3 us a call.
// Trimming or topping up to exactly k in the selection order makes the
// sampled kind return the same entries as the exact kind.
//
// A DGC step (Sec. 5.1) runs inside the same passes: the pass that forms v
// (the exact path's histogram pass, the sampled path's stream pass; the
// sample reads the same values) first takes the velocity step
// u <- fl32(fl32(m * u) + fl32(c * g)) and writes u, then v = fl32(u + e);
// the emit pass writes +0.0 into u as well as e_new at the winners.  The
// call's table then holds u in the gradient's place; the gradients come
// from a second table of the same tensors.
#include "launch.hpp"

namespace bc {

namespace {

// A tensor's threshold word (t_thr): the threshold key, whose low 10 bits
// are zero, with the shift s of the candidates' bins in bits 4..0.  t_zero
// holds the key from which the stream pass writes e_new = +0.0 at once
// (kNoEarlyZero: nowhere).
constexpr uint32_t kNoEarlyZero = 0xFFFFFFFFu;
constexpr uint32_t kExactShift = 10;  // bins of 2^10 keys: bits 30..20 of an exact threshold in 1024 of them
__device__ __forceinline__ uint32_t thr_key(uint32_t w) { return w & ~0x3FFu; }
__device__ __forceinline__ uint32_t thr_shift(uint32_t w) { return w & 31u; }
// Whether a listed key is at or above the threshold (a tensor that find_bin
// gave a higher threshold keeps its list), and the bin of one that is: the
// last bin takes everything past the range.
__device__ __forceinline__ bool cand_in(uint32_t key, uint32_t w) { return key >= thr_key(w); }
__device__ __forceinline__ uint32_t cand_bin(uint32_t key, uint32_t w) {
    const uint32_t b = (key - thr_key(w)) >> thr_shift(w);
    return b < (uint32_t)kBins0 ? b : (uint32_t)kBins0 - 1u;
}

// Place of a chunk's candidate r (of m) in the chunk's slot of kChunk
// entries.  Slots are 32 KiB apart, so equal places of all chunks would lie
// on the same few memory channels; a start that moves on by 256 bytes per
// chunk spreads the short lists over all of them.  Lists of up to half a
// slot leave the other half alone (cand_vel).
__device__ __forceinline__ uint32_t cand_at(uint32_t c, uint32_t m, uint32_t r) {
    return m <= kChunk / 2 ? (r + 32u * c) & (kChunk / 2 - 1u) : r;
}
// A DGC step keeps candidate r's velocity u in the slot's second half, where
// it has written u = +0.0 early (in chunks of up to kListMax candidates).
constexpr uint32_t kListMax = 512;  // candidates of a chunk listed in LDS at a time
__device__ __forceinline__ float* cand_vel(const Ws& ws, uint32_t c, uint32_t r) {
    return (float*)(ws.t_cand + (size_t)c * kChunk + kChunk / 2) + ((r + 64u * c) & (kChunk / 2 - 1u));
}

// A tensor's fallback word (t_fb): what find_bin could not settle, and
// whether its new threshold is there.
constexpr uint32_t kFbFew = 1;   // fewer than k candidates: the whole tensor again
constexpr uint32_t kFbPast = 2;  // the k-th past the bins' range: the candidates again
constexpr uint32_t kFbReady = 4;

constexpr uint32_t kWholeBelow = 4u * kChunk;  // shorter tensors are read whole, not sampled

// The DGC velocity step of a chunk: td holds u (as the fp32 gradient) and
// e, tg the step's gradient; u receives fl32(fl32(m * u) + fl32(c * g))
// (c the clipping factor, or g as widened without clipping) and v fl32(u + e),
// +0.0 past the tensor's end.
template <bool kNT>
__device__ __forceinline__ void load_v_dgc(const TDesc& td, const TDesc& tg, uint32_t j, const DgcFuse& f,
                                           float (&u)[kEpt], float (&v)[kEpt], uint32_t& valid) {
    float g[kEpt], e[kEpt];
    load_v<kNT>(tg, j, false, g, valid);
    load_v<kNT>(td, j, false, u, valid);
    TDesc te = td;
    te.grad = td.resid;
    load_v<kNT>(te, j, false, e, valid);
    if (f.clip) {
        const float cf = *f.clip;
#pragma unroll
        for (int i = 0; i < kEpt; ++i) g[i] = cf * g[i];
    }
#pragma unroll
    for (int i = 0; i < kEpt; ++i) {
        const float mu = f.m * u[i];
        u[i] = mu + g[i];
        v[i] = u[i] + e[i];
    }
}

__device__ __forceinline__ float* vel_of(const TDesc& td) { return (float*)const_cast<void*>(td.grad); }

// Add the keys of a thread's valid elements to a block's LDS histogram of
// bits 30..20.  Zeros (most of a sparse aggregate, which the divisible
// scheme compresses again; untouched rows of an embedding) are counted per
// thread: as atomic additions they would all meet in one bin (13.7 M
// elements, 92% zeros: 53 us, against 12.5 us counted apart).
__device__ __forceinline__ void add_keys(uint32_t* lh, const float (&v)[kEpt], uint32_t valid) {
    uint32_t zeros = 0;
#pragma unroll
    for (int i = 0; i < kEpt; ++i) {
        const uint32_t key = key_of(v[i]);
        if ((valid >> i) & 1u) {
            if (key != 0u) atomicAdd(&lh[key >> 20], 1u);
            else ++zeros;
        }
    }
    if (__ballot(zeros != 0u)) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) zeros += (uint32_t)__shfl_xor((int)zeros, o, 64);
        if (lane_id() == 0) atomicAdd(&lh[0], zeros);
    }
}

// Flush a block's LDS histogram into the tensor's global histogram.
__device__ __forceinline__ void flush_hist(const uint32_t* lh, uint32_t* gh, int bins) {
    for (int b = threadIdx.x; b < bins; b += kBlock) {
        const uint32_t x = lh[b];
        if (x) atomicAdd(gh + b, x);
    }
}

}  // namespace

// Stream pass of the exact path: e_new = v (kDGC: after the velocity step)
// and the histogram of key bits 30..20.
template <bool kDGC>
__global__ __launch_bounds__(kBlock) void topk_hist_pass(const TDesc* __restrict__ d, int T, uint32_t C, Ws ws,
                                                         uint64_t* __restrict__ clear_status, int copies,
                                                         DgcFuse f) {
    __shared__ uint32_t lh[kBins0];
    const uint32_t c = blockIdx.x;
    if (clear_status && threadIdx.x == 0) clear_status[c] = 0ull;
    const int t = tensor_of_chunk(d, T, c);
    const TDesc td = d[t];
    const uint32_t j = c - td.chunk0;
    for (int b = threadIdx.x; b < kBins0; b += kBlock) lh[b] = 0;
    float v[kEpt];
    uint32_t valid;
    if constexpr (kDGC) {
        float u[kEpt];
        load_v_dgc<false>(td, f.dg[t], j, f, u, v, valid);
        store_chunk(vel_of(td), td.n, j, u);
        store_chunk(td.resid, td.n, j, v);
    } else {
        load_v(td, j, td.resid != nullptr, v, valid);
        if (td.resid) store_chunk(td.resid, td.n, j, v);
    }
    __syncthreads();
    add_keys(lh, v, valid);
    __syncthreads();
    flush_hist(lh, ws.t_hist + ((size_t)t * copies + c % (uint32_t)copies) * kBins0, kBins0);
}

// Thresholds of the sampled kind: one workgroup per tensor looks at up to
// 16384 elements, kept as keys in registers (16 a thread), and takes from
// them the threshold and the early-zero key, first to key bits 30..20, then
// to bits 30..10, with two LDS histograms.  A tensor of fewer than 16384
// elements is read whole: its threshold is exact to those bits.  A longer one
// gives 2% of its elements, at least 4096 and at most 16384, in runs of 16
// (64 bytes of fp32), one at a Philox-drawn place in each of as many equal
// strata.  (With a histogram of bits 30..20 alone the threshold falls up to
// an eighth of an octave low; error feedback holds the top 1% of a steady
// gradient within a few percent of the k-th, so that seven to nine times k
// entries became candidates, against 1.3 to 2.3 times now.)  The LDS
// additions bound it, about a cycle each, so four times the elements took
// twice the time for a margin that the sample does not need.  Also clears the
// tensor's histograms and, first of all kernels of a call, the fallback's
// words.
// Workgroups of 1024 threads (this kernel and topk_place); of 256 for calls
// of more than 256 tensors, which fill the GPU by their number, and in which
// a wide workgroup's barriers and idle waves are what short tensors wait for.
// A call with 1024 against 256 threads: 16 tensors of 1 M elements 73 and
// 80 us, BERT-base's 199 285 and 328, 300 of 100 thousand 114 and 110, 1000
// of 9 thousand 103 and 77, 40000 of 400 2123 and 935 (with two histogram
// copies in the first).
constexpr int kWideBlock = 1024, kNarrowBlock = kBlock;
constexpr int kWideTensors = 256;
constexpr uint32_t kRun = 16;
constexpr uint32_t kRunsMin = 4096 / kRun, kRunsMax = kWholeBelow / kRun;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;
static_assert(kRunsMax <= 4 * kNarrowBlock && kWholeBelow / 4 / kRunsMin >= kRun / 4, "sampling geometry");

namespace {

// One element as the stream pass will form it.
template <bool kDGC>
__device__ __forceinline__ float form_v(float g, float u, float e, bool resid, const DgcFuse& f, float clip) {
    if constexpr (kDGC) {
        if (f.clip) g = clip * g;
        const float mu = f.m * u;
        g = mu + g;
    }
    return resid ? g + e : g;
}

// Keys of kN groups of 4 elements (first elements at[]), whose loads are all
// in flight together: kDT and kResid keep them free of branches.
template <bool kDGC, int kDT, bool kResid, uint32_t kN>
__device__ __forceinline__ void group_keys(const TDesc& td, const TDesc& tg, const DgcFuse& f, const uint32_t* at,
                                           uint32_t* key) {
    const void* grad = kDGC ? tg.grad : td.grad;
    f32x4 g[kN], e[kN], u[kN];
    u32x2 h[kN];
#pragma unroll
    for (uint32_t q = 0; q < kN; ++q) {
        if constexpr (kDT == 0) g[q] = ldg4f((const float*)grad + at[q]);
        else h[q] = ldg2u((const uint16_t*)grad + at[q]);
        if constexpr (kResid) e[q] = ldg4f(td.resid + at[q]);
        if constexpr (kDGC) u[q] = ldg4f((const float*)td.grad + at[q]);
    }
    const float clip = kDGC && f.clip ? *f.clip : 1.f;
#pragma unroll
    for (uint32_t q = 0; q < kN; ++q)
#pragma unroll
        for (int p = 0; p < 4; ++p)
            key[4 * q + p] = key_of(form_v<kDGC>(g_elem<kDT>(g[q], h[q], p), kDGC ? u[q][p] : 0.f,
                                                 kResid ? e[q][p] : 0.f, kResid, f, clip));
}

template <bool kDGC, uint32_t kN>
__device__ __forceinline__ void group_keys(const TDesc& td, const TDesc& tg, const DgcFuse& f, const uint32_t* at,
                                           uint32_t* key) {
    const uint32_t dtype = kDGC ? tg.dtype : td.dtype;
    if (kDGC || td.resid) {  // a DGC step has residuals
        if (dtype == 0) group_keys<kDGC, 0, true, kN>(td, tg, f, at, key);
        else group_keys<kDGC, 1, true, kN>(td, tg, f, at, key);
    } else {
        if (dtype == 0) group_keys<kDGC, 0, false, kN>(td, tg, f, at, key);
        else group_keys<kDGC, 1, false, kN>(td, tg, f, at, key);
    }
}

// Exclusive prefix over the kThreads threads; sh: one entry per wave, not
// used by the scan before.
template <int kThreads>
__device__ __forceinline__ uint32_t wide_scan(uint32_t x, uint32_t* sh) {
    const int lane = lane_id(), w = threadIdx.x >> 6;
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int q = 0; q < kThreads / 64; ++q) before += q < w ? sh[q] : 0u;
    return before + inc - x;
}

}  // namespace

template <bool kDGC, int kThreads>
__global__ __launch_bounds__(kThreads) void topk_threshold(const TDesc* __restrict__ d, double ratio, uint64_t seed,
                                                           int copies, uint32_t max_shift, Ws ws, DgcFuse f) {
    constexpr uint32_t kGroups = kWholeBelow / 4 / kThreads;  // groups of 4 elements a thread holds
    constexpr uint32_t kLh = kThreads == kWideBlock ? 4 : 1;  // copies of a histogram (lane mod kLh)
    __shared__ uint32_t lh[kLh * kBins0];  // of one, later of two with 1024 bins
    __shared__ uint32_t start[kRunsMax];  // first group of 4 of each run
    __shared__ uint32_t sh[3][kThreads / 64];
    __shared__ uint32_t found[5];
    const int t = blockIdx.x;
    const TDesc td = d[t];
    if (t == 0 && threadIdx.x < kAnyWords) ws.t_any[threadIdx.x] = 0u;
    {
        u32x4* gh = (u32x4*)(ws.t_hist + (size_t)t * copies * kBins0);
        for (int b = threadIdx.x; b < copies * kBins0 / 4; b += kThreads) gh[b] = u32x4{0u, 0u, 0u, 0u};
    }
    if (td.k == 0) return;
    const TDesc tg = kDGC ? f.dg[t] : td;
    const bool whole = td.n < kWholeBelow;
    const uint32_t units = td.n / 4;
    uint32_t runs = 0;
    if (!whole) {
        runs = td.n / (50u * kRun);
        runs = runs < kRunsMin ? kRunsMin : runs > kRunsMax ? kRunsMax : runs;
        const uint64_t step = ((uint64_t)units << 16) / runs;  // a stratum, in units of 2^-16 groups
        if (4u * threadIdx.x < runs) {
            const U64x4 ctr = {{(uint64_t)td.tid, (uint64_t)threadIdx.x, 0, 0}};
            const U64x4 r = philox4x64_10(ctr, seed, kStreamSample);
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t i = 4u * threadIdx.x + q;
                const uint32_t a = (uint32_t)(step * i >> 16);
                const uint32_t len = (uint32_t)(step * (i + 1) >> 16) - a;  // at least 16, and a + len <= units
                if (i < runs) start[i] = a + (uint32_t)(((r.v[q] >> 32) * (len - (kRun / 4 - 1))) >> 32);
            }
        }
    }
    for (int b = threadIdx.x; b < (int)kLh * kBins0; b += kThreads) lh[b] = 0;
    if (threadIdx.x < 5) found[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t groups = whole ? units : runs * (kRun / 4);
    const uint32_t total = whole ? td.n : runs * kRun;
    uint32_t key[4 * kGroups + 1];  // kNoKey: none
    constexpr uint32_t kBatch = kDGC ? 2 : 4;  // groups loaded together
#pragma unroll
    for (uint32_t q0 = 0; q0 < kGroups; q0 += kBatch) {
        uint32_t at[kBatch];
        if (q0 * kThreads < groups) {  // places past the last group read it again
#pragma unroll
            for (uint32_t q = 0; q < kBatch; ++q) {
                uint32_t i = (q0 + q) * kThreads + threadIdx.x;
                i = i < groups ? i : groups - 1u;
                at[q] = whole ? 4u * i : 4u * (start[i / 4] + i % 4);
            }
            group_keys<kDGC, kBatch>(td, tg, f, at, key + 4 * q0);
        }
#pragma unroll
        for (uint32_t q = 0; q < kBatch; ++q)
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if ((q0 + q) * kThreads + threadIdx.x >= groups) key[4 * (q0 + q) + p] = kNoKey;
    }
    key[4 * kGroups] = kNoKey;
    if (whole && threadIdx.x < td.n % 4) {  // past the last whole group
        const uint32_t i = 4u * units + threadIdx.x;
        const TDesc& src = kDGC ? tg : td;
        const float g = src.dtype == 0 ? gp((const float*)src.grad)[i] : h2f(gp((const uint16_t*)src.grad)[i]);
        const float u = kDGC ? gp((const float*)td.grad)[i] : 0.f;
        const float e = td.resid ? gp(td.resid)[i] : 0.f;
        key[4 * kGroups] =
            key_of(form_v<kDGC>(g, u, e, td.resid != nullptr, f, kDGC && f.clip ? *f.clip : 1.f));
    }
    uint32_t zeros = 0;  // counted apart: they would all meet in one bin
    uint32_t* mine = lh + (threadIdx.x & (kLh - 1));
#pragma unroll
    for (uint32_t q = 0; q <= 4 * kGroups; ++q) {
        if (q < 4 * kGroups && q / 4 * kThreads >= groups) continue;  // nobody's (uniform)
        if (key[q] == 0u) ++zeros;
        else if (key[q] != kNoKey) atomicAdd(mine + kLh * (key[q] >> 20), 1u);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) zeros += (uint32_t)__shfl_xor((int)zeros, o, 64);
    if (lane_id() == 0 && zeros) {
        atomicAdd(lh, zeros);
        atomicAdd(&found[4], zeros);
    }
    __syncthreads();
    // the threshold's place among the keys, and a place that the k-th key
    // hardly ever lies above: the k rule on the sample's size with margins
    uint32_t target = td.k, early = 0;
    uint32_t ks = 0;
    if (!whole) {
        const uint64_t ppm = (uint64_t)llround(ratio * 1e6);
        ks = (uint32_t)(((uint64_t)total * ppm + 999999u) / 1000000u);
        if (ks < 1) ks = 1;
        const uint32_t tg2 = ks + ks / 4 + 16;
        target = tg2 < total ? tg2 : total;
        // no early zeros where the whole sample falls short of the margin: the
        // exact path, which all but certainly follows, would put them back
        early = tg2 < total && ks - ks / 4 > 8 ? ks - ks / 4 - 8 : 0u;
    }
    {
        // thread i owns the i-th kPer bins from the top
        constexpr uint32_t kPer = kBins0 / kThreads;
        const uint32_t top = (uint32_t)kBins0 - 1u - kPer * threadIdx.x;
        uint32_t h[kPer], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            h[q] = 0;
#pragma unroll
            for (uint32_t p = 0; p < kLh; ++p) h[q] += lh[kLh * (top - q) + p];
            sum += h[q];
        }
        uint32_t above = wide_scan<kThreads>(sum, sh[0]);
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            if (above < target && target <= above + h[q]) {
                found[0] = top - q;
                found[1] = above;
            }
            if (early && above < early && early <= above + h[q]) {
                found[2] = top - q;
                found[3] = above;
            }
            if (!early && above == 0 && h[q]) found[2] = top - q;  // the highest bin with keys
            above += h[q];
        }
    }
    __syncthreads();
    const uint32_t b0 = found[0], above0 = found[1], b1 = found[2], above1 = found[3], nz = found[4];
    for (int b = threadIdx.x; b < (int)kLh * kBins0; b += kThreads) lh[b] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q <= 4 * kGroups; ++q) {
        if (q < 4 * kGroups && q / 4 * kThreads >= groups) continue;
        if (key[q] == 0u) continue;
        const uint32_t b = key[q] >> 20, x = kLh * (key[q] >> 10 & 1023u);
        if (b == b0) atomicAdd(mine + x, 1u);
        if (early && b == b1) atomicAdd(mine + kLh * kBins12 + x, 1u);
    }
    if (threadIdx.x == 0 && nz) {
        if (b0 == 0) atomicAdd(lh, nz);
        if (early && b1 == 0) atomicAdd(lh + kLh * kBins12, nz);
    }
    if (threadIdx.x < 4) found[threadIdx.x] = 0u;
    __syncthreads();
    {
        constexpr uint32_t kPer = kBins12 / kThreads;
        const uint32_t top = (uint32_t)kBins12 - 1u - kPer * threadIdx.x;
        uint32_t h[2][kPer], sum[2] = {0, 0};
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q)
#pragma unroll
            for (uint32_t x = 0; x < 2; ++x) {
                h[x][q] = 0;
#pragma unroll
                for (uint32_t p = 0; p < kLh; ++p) h[x][q] += lh[kLh * (x * kBins12 + top - q) + p];
                sum[x] += h[x][q];
            }
        uint32_t a0 = above0 + wide_scan<kThreads>(sum[0], sh[1]);
        uint32_t a1 = above1 + wide_scan<kThreads>(sum[1], sh[2]);
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            if (a0 < target && target <= a0 + h[0][q]) found[0] = top - q;
            if (early && a1 < early && early <= a1 + h[1][q]) found[1] = top - q;
            a0 += h[0][q];
            a1 += h[1][q];
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    uint32_t thr = b0 << 20 | found[0] << 10;
    // fewer non-zeros in the sample than its margin asks for, but its k: only
    // zeros stay out (with threshold 0 every element becomes a candidate: 16
    // tensors of 1 M elements with 1.15 k non-zeros 276 us, 110 so)
    if (!whole && thr == 0u && total - nz >= ks) thr = 1024u;
    uint32_t zero = kNoEarlyZero, span;
    if (whole) {  // every key past the k-th's 2^10 wins
        zero = thr + 1024u;
        span = 1024u;
    } else if (early) {
        zero = (b1 << 20 | found[1] << 10) + 1024u;
        span = 2u * (zero - thr) + 4096u;  // reaches well past the k-th key's likely place
    } else {
        span = ((b1 + 2u) << 20) - thr;
    }
    uint32_t s = 4;
    while (s < max_shift && span > ((uint32_t)(kBins0 - 1) << s)) ++s;
    ws.t_thr[t] = thr | s;
    ws.t_zero[td.chunk0] = zero;
}

// Stores and a wait by which a workgroup hands data to others of the same
// kernel: the stores go through to where every compute die sees them, so the
// hand-over needs no release (which writes back the die's whole L2 cache,
// about 9 us, one workgroup after another).
__device__ __forceinline__ void put_agent(uint32_t* p, uint32_t x) {
    __hip_atomic_store((BC_GLOBAL uint32_t*)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// Loads that follow see what other workgroups handed over.
__device__ __forceinline__ void acquire_agent() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

// Read (and clear) the eight bins under `hi` of a tensor's histogram, all
// copies added, highest bin first.  Whole vectors: with single words, lanes
// 32 bytes apart, the clearing stores bound a find (12 us at T = 199).
// kInPass: the histogram is used again by other workgroups of the same kernel.
template <bool kInPass>
__device__ __forceinline__ void take_bins(uint32_t* gh, int hi, int copies, uint32_t (&h)[8]) {
    constexpr int stride = kBins0, kMax = kGeneralCopiesMax;
    u32x4 a[kMax], b[kMax];
#pragma unroll
    for (int r = 0; r < kMax; ++r) {
        a[r] = b[r] = u32x4{0u, 0u, 0u, 0u};
        if (r < copies) {
            a[r] = ldg4u(gh + r * stride + hi - 4);
            b[r] = ldg4u(gh + r * stride + hi - 8);
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) h[q] = 0;
#pragma unroll
    for (int r = 0; r < kMax; ++r) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            h[q] += a[r][3 - q];
            h[4 + q] += b[r][3 - q];
        }
        if (r < copies) {
            if constexpr (kInPass) {
#pragma unroll
                for (int q = 1; q <= 8; ++q) put_agent(gh + r * stride + hi - q, 0u);
            } else {
                *(BC_GLOBAL u32x4*)(gh + r * stride + hi - 4) = u32x4{0u, 0u, 0u, 0u};
                *(BC_GLOBAL u32x4*)(gh + r * stride + hi - 8) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    }
}

// The exact candidate threshold of a tensor, the bin of the k-th key in its
// histogram of key bits 30..20, by a whole workgroup.
// keep_zero: of the tensor's candidates, whose early zeros stay as they are.
template <bool kInPass>
__device__ __forceinline__ void find_thr(const TDesc& td, int t, int copies, const Ws& ws, uint64_t* sh,
                                         bool keep_zero) {
    const int hi = kBins0 - threadIdx.x * 8;  // thread i owns the i-th eight bins from the top
    uint32_t h[8];
    take_bins<kInPass>(ws.t_hist + (size_t)t * copies * kBins0, hi, copies, h);
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) mine += h[q];
    uint64_t total;
    uint32_t above = (uint32_t)block_excl_scan_u64(mine, sh, total);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (above < td.k && td.k <= above + h[q]) {
            const uint32_t thr = (uint32_t)(hi - 1 - q) << 20 | kExactShift;
            if constexpr (kInPass) {
                put_agent(ws.t_thr + t, thr);
                if (!keep_zero) put_agent(ws.t_zero + td.chunk0, kNoEarlyZero);
            } else {
                ws.t_thr[t] = thr;
                ws.t_zero[td.chunk0] = kNoEarlyZero;  // e_new is already written
            }
        }
        above += h[q];
    }
}

// The bin of the k-th candidate of a tensor, by a whole workgroup; otherwise
// kFbFew, or kFbPast for the k-th in the last bin (which has no upper edge).
// An exact threshold meets neither.
__device__ __forceinline__ uint32_t find_bin(const TDesc& td, int t, int copies, const Ws& ws, uint64_t* sh,
                                         uint32_t* found) {
    const int hi = kBins0 - threadIdx.x * 8;
    uint32_t h[8];
    take_bins<false>(ws.t_hist + (size_t)t * copies * kBins0, hi, copies, h);
    if (threadIdx.x == 0) found[0] = (uint32_t)kBins0 - 1u;
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) mine += h[q];
    uint64_t total;
    uint32_t above = (uint32_t)block_excl_scan_u64(mine, sh, total);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (above < td.k && td.k <= above + h[q]) {
            found[0] = (uint32_t)(hi - 1 - q);
            found[1] = above;
        }
        above += h[q];
    }
    __syncthreads();
    if (found[0] == (uint32_t)kBins0 - 1u) return total < td.k ? kFbFew : kFbPast;
    if (threadIdx.x == 0) {
        ws.t_prefix[t] = found[0];
        ws.t_krem[t] = td.k - found[1];
    }
    return 0u;
}

__global__ __launch_bounds__(kBlock) void topk_find_thr(const TDesc* __restrict__ d, int copies, Ws ws) {
    __shared__ uint64_t sh[4];
    const TDesc td = d[blockIdx.x];
    if (td.k) find_thr<false>(td, (int)blockIdx.x, copies, ws, sh, false);
}

__global__ __launch_bounds__(kBlock) void topk_find_bin(const TDesc* __restrict__ d, int copies, Ws ws) {
    __shared__ uint64_t sh[4];
    __shared__ uint32_t found[2];
    const int t = blockIdx.x;
    const TDesc td = d[t];
    if (td.k == 0) return;
    const uint32_t fb = find_bin(td, t, copies, ws, sh, found);
    if (threadIdx.x != 0) return;
    ws.t_fb[t] = fb;  // bytecomp_topk_stats counts kFbFew
    if (fb == 0u) return;
    // one entry of the fallback's list: the tensor, and how many chunks the
    // entries before it have (t_krem and t_prefix count its finished chunks)
    ws.t_krem[t] = ws.t_prefix[t] = 0u;
    const unsigned long long at = atomicAdd((unsigned long long*)ws.t_any, 1ull << 32 | td.nchunks);
    ws.t_off[at >> 32] = (uint64_t)t << 32 | (uint32_t)at;
}

// Candidate compaction.  kStream (sampled main pass): v = g + e,
// e_new = v written back (kDGC: after the velocity step, u written back),
// +0.0 at the candidates at or above the threshold word's early-zero key.
// Re-read mode: v from the residual (or g).  Candidates = valid entries
// with key at or above the threshold, compacted in index order into the
// chunk's slot of t_cand; also the LDS histogram of their bins.  They pass
// through a list in LDS, kListMax at a time, so that they are stored side by
// side and one thread each instead of one of a thread's 16 elements after
// another.
struct CompactLds {
    uint32_t lh[kBins0];
    uint64_t sh[4];
    uint2 list[kListMax];
};

template <bool kNT, bool kDGC, bool kStream>
__device__ __forceinline__ void compact_chunk(const TDesc& td, int t, uint32_t c, int copies, const Ws& ws,
                                              const DgcFuse& f, CompactLds& l, float* list_u) {
    uint32_t* lh = l.lh;
    uint64_t* sh = l.sh;
    uint2* list = l.list;
    const uint32_t j = c - td.chunk0;
    const uint32_t w = ws.t_thr[t], zero = ws.t_zero[td.chunk0];
    const uint32_t thr = thr_key(w);
    for (int b = threadIdx.x; b < kBins0; b += kBlock) lh[b] = 0;
    float v[kEpt], u[kEpt];
    uint32_t valid;
    if constexpr (kDGC && kStream) {
        load_v_dgc<kNT>(td, f.dg[t], j, f, u, v, valid);
    } else if constexpr (kStream) {
        load_v<kNT>(td, j, td.resid != nullptr, v, valid);
        if (td.resid) {
            float e[kEpt];
#pragma unroll
            for (int i = 0; i < kEpt; ++i) e[i] = key_of(v[i]) >= zero ? 0.f : v[i];
            store_chunk<kNT>(td.resid, td.n, j, e);
        }
    } else {
        load_stored_v(td, j, v, valid);
    }
    uint32_t pm = 0;
#pragma unroll
    for (int i = 0; i < kEpt; ++i)
        if (((valid >> i) & 1u) && key_of(v[i]) >= thr) pm |= 1u << i;
    uint64_t packed = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) packed |= (uint64_t)__popc((pm >> (4 * r)) & 0xFu) << (16 * r);
    uint64_t tot;
    const uint64_t pre = block_excl_scan_u64(packed, sh, tot);
    const uint32_t m = (uint32_t)(tot & 0xFFFFu) + (uint32_t)(tot >> 16 & 0xFFFFu) +
                       (uint32_t)(tot >> 32 & 0xFFFFu) + (uint32_t)(tot >> 48);
    const bool keep_u = kDGC && kStream && m <= kListMax;
    uint2* out = ws.t_cand + (size_t)c * kChunk;
    if constexpr (kDGC && kStream) {
        if (keep_u) {
            uint32_t base = 0;
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                uint32_t at = base + (uint32_t)((pre >> (16 * r)) & 0xFFFFu);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if ((pm >> (4 * r + q)) & 1u) list_u[at++] = u[4 * r + q];
                base += (uint32_t)((tot >> (16 * r)) & 0xFFFFu);
            }
        }
        float e[kEpt];
#pragma unroll
        for (int i = 0; i < kEpt; ++i) {
            const bool z = keep_u && key_of(v[i]) >= zero;
            u[i] = z ? 0.f : u[i];
            e[i] = z ? 0.f : v[i];
        }
        store_chunk<kNT>(vel_of(td), td.n, j, u);
        store_chunk<kNT>(td.resid, td.n, j, e);
    }
    if ((kDGC && kStream) || m <= kListMax) {
        for (uint32_t w0 = 0; w0 < m; w0 += kListMax) {  // once for all but dense chunks
            uint32_t base = 0;
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                uint32_t at = base + (uint32_t)((pre >> (16 * r)) & 0xFFFFu) - w0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = 4 * r + q;
                    if ((pm >> i) & 1u) {
                        if (at < kListMax)
                            list[at] = make_uint2(j * (uint32_t)kChunk + 1024u * r + 4u * threadIdx.x + q, f2u(v[i]));
                        ++at;
                    }
                }
                base += (uint32_t)((tot >> (16 * r)) & 0xFFFFu);
            }
            __syncthreads();
            const uint32_t nl = m - w0 < kListMax ? m - w0 : kListMax;
            for (uint32_t i = threadIdx.x; i < nl; i += kBlock) {
                const uint2 e = list[i];
                const uint32_t key = e.y & 0x7FFFFFFFu;
                out[cand_at(c, m, w0 + i)] = e;
                if constexpr (kDGC) {
                    if (keep_u && key >= zero) *cand_vel(ws, c, w0 + i) = list_u[i];
                }
                atomicAdd(&lh[cand_bin(key, w)], 1u);
            }
            __syncthreads();
        }
    } else {
        // dense: straight from the registers (20 M elements that are all
        // candidates: 94 us, 120 through the list; in the DGC pass the code
        // costs the sparse case registers and 18 us of 470)
        uint32_t base = 0;
        __syncthreads();  // the histogram is clear
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            uint32_t at = base + (uint32_t)((pre >> (16 * r)) & 0xFFFFu);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * r + q;
                if ((pm >> i) & 1u) {
                    out[cand_at(c, m, at++)] =
                        make_uint2(j * (uint32_t)kChunk + 1024u * r + 4u * threadIdx.x + q, f2u(v[i]));
                    atomicAdd(&lh[cand_bin(key_of(v[i]), w)], 1u);
                }
            }
            base += (uint32_t)((tot >> (16 * r)) & 0xFFFFu);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) ws.t_ccount[c] = m;
    if (m == 0) return;  // uniform; the histogram is untouched
    flush_hist(lh, ws.t_hist + ((size_t)t * copies + c % (uint32_t)copies) * kBins0, kBins0);
}

template <bool kNT, bool kDGC, bool kStream>
__global__ __launch_bounds__(kBlock) void topk_compact(
    const TDesc* __restrict__ d, int T, int copies, Ws ws, DgcFuse f) {
    __shared__ CompactLds l;
    __shared__ float list_u[kDGC && kStream ? kListMax : 1];
    const int t = tensor_of_chunk(d, T, blockIdx.x);
    const TDesc td = d[t];
    compact_chunk<kNT, kDGC, kStream>(td, t, blockIdx.x, copies, ws, f, l, list_u);
}

// The tensors that find_bin listed, in one launch that ends at once when there
// are none (the usual case).  kFbFew: the exact path over the whole tensor.
// kFbPast (most values zero and k near the number of the others, or values
// over many octaves between the sample's threshold and the k-th): the k-th is
// among the candidates, so the two passes go over those and only give them a
// threshold, the k-th's bits 30..20, whose bins reach; list and early zeros
// stay.  Only the listed tensors' chunks are visited.  Workgroups claim batches of consecutive ones, first
// all batches of the first pass, then all of the second: in the first the
// chunks get back what the stream pass zeroed early and add their keys to
// their tensor's histogram of bits 30..20, and whoever finishes a tensor's
// last chunk finds its exact threshold; in the second they are compacted
// again, and whoever finishes the last finds the bin.  A workgroup waits only
// in the second pass, for a threshold whose chunks are all claimed by
// workgroups that run and wait for nothing, so the wait ends whatever part of
// the grid is resident.  The two counters are paid once per batch and tensor,
// and what other workgroups read goes out by put_agent (one listed tensor of
// BERT-base cost 3.3 ms when all chunks of the call were visited one by one
// with a release each).
namespace {

constexpr uint32_t kAllBins = 20;  // a threshold word that bins keys by their bits 30..20

// Histogram of the candidates of chunks [c0, c1) in the bins of threshold
// word w, a wave per chunk at a time.
__device__ __forceinline__ void rebin_chunks(const Ws& ws, uint32_t c0, uint32_t c1, uint32_t w, uint32_t* lh) {
    constexpr uint32_t kU = 8;  // a lane's loads in flight together
    uint32_t zeros = 0;         // counted apart: they would all meet in one bin
    for (uint32_t c = c0 + (uint32_t)wave_id(); c < c1; c += kBlock / 64) {
        const uint32_t m = ws.t_ccount[c];
        const uint2* cand = ws.t_cand + (size_t)c * kChunk;
        for (uint32_t i0 = (uint32_t)lane_id(); i0 < m; i0 += 64 * kU) {
            uint32_t key[kU];
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u)
                key[u] = i0 + 64 * u < m ? cand[cand_at(c, m, i0 + 64 * u)].y & 0x7FFFFFFFu : kNoKey;
#pragma unroll
            for (uint32_t u = 0; u < kU; ++u) {
                if (key[u] == kNoKey || !cand_in(key[u], w)) continue;
                if (key[u] == 0u) ++zeros;
                else atomicAdd(&lh[cand_bin(key[u], w)], 1u);
            }
        }
    }
    if (zeros) atomicAdd(&lh[0], zeros);
}

}  // namespace

template <bool kDGC>
__global__ __launch_bounds__(kBlock) void topk_fallback(const TDesc* __restrict__ d, int copies, Ws ws) {
    __shared__ CompactLds l;
    __shared__ uint32_t word, found[2];
    const uint64_t any = *(const uint64_t*)ws.t_any;  // listed tensors, and their chunks
    if (any == 0) return;
    const uint32_t listed = (uint32_t)(any >> 32), F = (uint32_t)any;
    const uint32_t batch = (F + gridDim.x - 1u) / gridDim.x;
    const uint32_t batches = (F + batch - 1u) / batch;
    const DgcFuse none{nullptr, 0.f, nullptr};
    for (;;) {
        __syncthreads();  // every thread has read `word`
        if (threadIdx.x == 0) word = atomicAdd(ws.t_any + 2, 1u);
        __syncthreads();
        const uint32_t q = word;
        if (q >= 2u * batches) return;
        const bool second = q >= batches;
        uint32_t f = (second ? q - batches : q) * batch;
        const uint32_t f1 = f + batch < F ? f + batch : F;
        uint32_t i = 0, hi = listed - 1u;  // the last entry that starts at or before chunk f of the list
        while (i < hi) {
            const uint32_t mid = (i + hi + 1u) >> 1;
            if ((uint32_t)ws.t_off[mid] <= f) i = mid; else hi = mid - 1u;
        }
        for (; f < f1; ++i) {
            const int t = (int)(ws.t_off[i] >> 32);
            const TDesc td = d[t];
            const uint32_t j0 = f - (uint32_t)ws.t_off[i];
            const uint32_t j1 = j0 + (f1 - f) < td.nchunks ? j0 + (f1 - f) : td.nchunks;
            f += j1 - j0;
            if (second) {
                if (threadIdx.x == 0)
                    while (!(__hip_atomic_load(ws.t_fb + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFbReady))
                        __builtin_amdgcn_s_sleep(8);
                __syncthreads();
                acquire_agent();  // threshold and restored values written elsewhere
            }
            const bool past = ws.t_fb[t] & kFbPast;
            if (past) {
                for (int b = threadIdx.x; b < kBins0; b += kBlock) l.lh[b] = 0;
                __syncthreads();
                rebin_chunks(ws, td.chunk0 + j0, td.chunk0 + j1, second ? ws.t_thr[t] : kAllBins, l.lh);
                __syncthreads();
                flush_hist(l.lh, ws.t_hist + ((size_t)t * copies + f % (uint32_t)copies) * kBins0, kBins0);
            } else if (!second) {
                for (int b = threadIdx.x; b < kBins0; b += kBlock) l.lh[b] = 0;
                const uint32_t zero = ws.t_zero[td.chunk0];
                for (uint32_t c = td.chunk0 + j0; c < td.chunk0 + j1; ++c) {
                    const uint32_t m = ws.t_ccount[c];
                    if (td.resid && zero != kNoEarlyZero && (!kDGC || m <= kListMax)) {
                        const uint2* cand = ws.t_cand + (size_t)c * kChunk;
                        constexpr uint32_t kU = 4;  // a thread's loads in flight together
                        for (uint32_t r0 = threadIdx.x; r0 < m; r0 += kU * kBlock) {
                            uint2 e[kU];
#pragma unroll
                            for (uint32_t u = 0; u < kU; ++u) {
                                const uint32_t r = r0 + u * kBlock;
                                e[u] = r < m ? cand[cand_at(c, m, r)] : make_uint2(0, 0);
                            }
#pragma unroll
                            for (uint32_t u = 0; u < kU; ++u) {
                                const uint32_t r = r0 + u * kBlock;
                                if (r >= m || (e[u].y & 0x7FFFFFFFu) < zero) continue;
                                put_agent((uint32_t*)td.resid + e[u].x, e[u].y);
                                if constexpr (kDGC) put_agent((uint32_t*)vel_of(td) + e[u].x, f2u(*cand_vel(ws, c, r)));
                            }
                        }
                    }
                    stores_done();
                    __syncthreads();  // this workgroup re-reads the chunk
                    float v[kEpt];
                    uint32_t valid;
                    load_stored_v(td, c - td.chunk0, v, valid);
                    add_keys(l.lh, v, valid);
                }
                __syncthreads();
                flush_hist(l.lh, ws.t_hist + ((size_t)t * copies + f % (uint32_t)copies) * kBins0, kBins0);
            } else {
                for (uint32_t c = td.chunk0 + j0; c < td.chunk0 + j1; ++c) {
                    compact_chunk<false, false, false>(td, t, c, copies, ws, none, l, nullptr);
                    __syncthreads();  // the next one clears the histogram
                }
            }
            stores_done();  // before the chunks count as done
            __syncthreads();
            if (threadIdx.x == 0) word = atomicAdd(second ? ws.t_prefix + t : ws.t_krem + t, j1 - j0) + (j1 - j0);
            __syncthreads();
            if (word != td.nchunks) continue;
            acquire_agent();  // the others' histograms
            if (second) {
                (void)find_bin(td, t, copies, ws, l.sh, found);
            } else {
                find_thr<true>(td, t, copies, ws, l.sh, past);
                stores_done();
                __syncthreads();
                if (threadIdx.x == 0) put_agent(ws.t_fb + t, (past ? kFbPast : kFbFew) | kFbReady);
            }
        }
    }
}

// Candidates inside the k-th key's bin (a chunk rarely has more than one or
// two) as one word per chunk: bit 63 set, every one has the low bits in bits
// 13..0; otherwise up to four of them, 14 bits each.  More, and different
// ones: the reader goes through the chunk's candidates again.
constexpr uint32_t kLowsMax = 4;
constexpr uint64_t kLowsSame = 1ull << 63;

// Per chunk: candidates above the k-th key's bin, and those inside it, which
// also go into the tensor's histogram of their low s bits.  Each wave takes
// kCountChunks consecutive chunks, whose loads it issues together (one
// chunk per wave for calls of few chunks, where the wave count matters
// more).  Entries with equal low bits are added together, so that a tensor
// of equal keys costs an addition per chunk and not one per entry.
constexpr uint32_t kCountBatchFrom = 4096;  // chunks

template <uint32_t kCountChunks>
__global__ __launch_bounds__(kBlock) void topk_cand_count(const TDesc* __restrict__ d, int T, uint32_t C,
                                                          int copies, Ws ws) {
    const int lane = lane_id();
    const uint32_t c0 = (blockIdx.x * (kBlock / 64) + wave_id()) * kCountChunks;
    uint32_t m[kCountChunks], w[kCountChunks], bin[kCountChunks], key[kCountChunks];
    int tt[kCountChunks];
#pragma unroll
    for (uint32_t u = 0; u < kCountChunks; ++u) {
        m[u] = c0 + u < C ? ws.t_ccount[c0 + u] : 0u;
        tt[u] = c0 + u < C ? tensor_of_chunk(d, T, c0 + u) : 0;
    }
#pragma unroll
    for (uint32_t u = 0; u < kCountChunks; ++u) {
        w[u] = ws.t_thr[tt[u]];
        bin[u] = ws.t_prefix[tt[u]];
        key[u] = (uint32_t)lane < m[u]
                     ? ws.t_cand[(size_t)(c0 + u) * kChunk + cand_at(c0 + u, m[u], (uint32_t)lane)].y & 0x7FFFFFFFu
                     : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < kCountChunks; ++u) {
        const uint32_t c = c0 + u;
        if (c >= C) break;
        const uint2* cand = ws.t_cand + (size_t)c * kChunk;
        uint32_t* gh = ws.t_hist + (size_t)tt[u] * copies * kBins0;
        const uint32_t low_mask = (1u << thr_shift(w[u])) - 1u;
        uint32_t gt = 0, nb = 0;
        uint32_t cur = 0, cur_n = 0;  // additions to bin `cur` not yet made
        uint32_t first = 0;
        bool same = true;
        uint64_t lows = 0;
        for (uint32_t i0 = 0; i0 < m[u]; i0 += 64) {
            const uint32_t i = i0 + (uint32_t)lane;
            bool in = i < m[u];
            uint32_t k = key[u];
            if (i0) k = in ? cand[cand_at(c, m[u], i)].y & 0x7FFFFFFFu : 0u;
            in = in && cand_in(k, w[u]);
            const uint32_t b = cand_bin(k, w[u]);
            gt += (uint32_t)__popcll(__ballot(in && b > bin[u]));
            const bool inside = in && b == bin[u];
            const uint32_t low = (k - thr_key(w[u])) & low_mask;
            uint64_t rest = __ballot(inside);
            for (int round = 0; rest; ++round) {
                if (round == 4) {  // many different ones: an addition per entry
                    if ((rest >> lane) & 1u) atomicAdd(gh + low, 1u);
                    nb += (uint32_t)__popcll(rest);
                    same = false;
                    break;
                }
                const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)low, (int)__builtin_ctzll(rest));
                const uint64_t eq = __ballot(inside && low == x) & rest;
                const uint32_t n = (uint32_t)__popcll(eq);
                rest &= ~eq;
                if (nb == 0) first = x;
                same = same && x == first;
                for (uint32_t q = nb; q < kLowsMax && q < nb + n; ++q) lows |= (uint64_t)x << (14u * q);
                nb += n;
                if (cur_n && x != cur) {
                    if (lane == 0) atomicAdd(gh + cur, cur_n);
                    cur_n = 0;
                }
                cur = x;
                cur_n += n;
            }
        }
        if (lane == 0) {
            if (cur_n) atomicAdd(gh + cur, cur_n);
            ws.t_gt[c] = gt;
            ws.t_eq[c] = nb;
            ws.t_off[c] = nb > kLowsMax && same ? kLowsSame | first : lows;
        }
    }
}

// One workgroup per tensor: the k-th key tau from the histogram of low bits,
// then every chunk's place.  eqb[c] = number of tau-equal candidates in
// earlier chunks; a chunk keeps its tau-equal candidates while the running
// count stays below the number needed.  Thread i walks a contiguous run of
// the tensor's chunks; two block scans over the runs' totals give every
// chunk its prefix.  Runs of up to kPlaceRegs chunks (tensors of up to
// kThreads * kPlaceRegs chunks) keep their counts in registers; longer runs are
// gone through three times.
constexpr uint32_t kPlaceRegs = 8;

namespace {

// Whether a chunk's word does not hold its candidates inside the k-th key's bin.
__device__ __forceinline__ bool chunk_again(uint32_t nb, uint64_t lows) {
    return nb > kLowsMax && !(lows & kLowsSame);
}

// Candidates above and equal to the k-th key, whose low bits are `tau_low`,
// from a chunk's counts and word.
__device__ __forceinline__ void chunk_counts(uint32_t gt0, uint32_t nb, uint64_t lows, uint32_t tau_low,
                                             uint32_t& gt, uint32_t& eq) {
    gt = gt0;
    eq = 0;
    if (nb == 0) return;
    if (lows & kLowsSame) {
        const uint32_t x = (uint32_t)lows;
        if (x > tau_low) gt += nb;
        else if (x == tau_low) eq = nb;
        return;
    }
#pragma unroll
    for (uint32_t q = 0; q < kLowsMax; ++q) {
        const uint32_t x = (uint32_t)(lows >> (14u * q)) & 0x3FFFu;
        gt += q < nb && x > tau_low ? 1u : 0u;
        eq += q < nb && x == tau_low ? 1u : 0u;
    }
}

// The same for a chunk whose candidates have to be read again, by a whole
// wave, left in the chunk's counts and word: `gt` above, and `eq` with the
// low bits tau_low.
__device__ __forceinline__ void recount_chunk(const Ws& ws, uint32_t c, uint32_t w, uint32_t bin,
                                              uint32_t tau_low, uint32_t& gt, uint32_t& eq) {
    const uint32_t m = ws.t_ccount[c];
    const uint2* cand = ws.t_cand + (size_t)c * kChunk;
    const uint32_t low_mask = (1u << thr_shift(w)) - 1u;
    gt = ws.t_gt[c];
    eq = 0;
    constexpr uint32_t kU = 4;
    for (uint32_t i0 = 0; i0 < m; i0 += 64 * kU) {
        uint32_t key[kU];
#pragma unroll
        for (uint32_t q = 0; q < kU; ++q) {
            const uint32_t i = i0 + 64 * q + (uint32_t)lane_id();
            key[q] = i < m ? cand[cand_at(c, m, i)].y & 0x7FFFFFFFu : 0u;
        }
#pragma unroll
        for (uint32_t q = 0; q < kU; ++q) {
            const bool inside = i0 + 64 * q + (uint32_t)lane_id() < m && cand_in(key[q], w) && cand_bin(key[q], w) == bin;
            const uint32_t x = (key[q] - thr_key(w)) & low_mask;
            gt += (uint32_t)__popcll(__ballot(inside && x > tau_low));
            eq += (uint32_t)__popcll(__ballot(inside && x == tau_low));
        }
    }
    if (lane_id() == 0) {
        ws.t_gt[c] = gt;
        ws.t_eq[c] = eq;
        ws.t_off[c] = kLowsSame | tau_low;
    }
}

// Winners of one chunk given the tau-equal candidates before it.
__device__ __forceinline__ uint32_t chunk_winners(uint32_t gt, uint32_t eq, uint32_t eq_before, uint32_t need) {
    const uint32_t left = eq_before < need ? need - eq_before : 0;
    return gt + (left < eq ? left : eq);
}

}  // namespace

template <int kThreads>
__global__ __launch_bounds__(kThreads) void topk_place(const TDesc* __restrict__ d, int copies, Ws ws) {
    __shared__ uint32_t sh[3][kThreads / 64];
    __shared__ uint32_t found[2];
    const int t = blockIdx.x;
    const TDesc td = d[t];
    if (td.k == 0 || td.nchunks == 0) return;
    const uint32_t w = ws.t_thr[t], bin = ws.t_prefix[t], krem = ws.t_krem[t];
    const uint32_t per = (td.nchunks + kThreads - 1) / kThreads;
    const uint32_t lo = threadIdx.x * per;
    const uint32_t hi = lo + per < td.nchunks ? lo + per : td.nchunks;
    uint32_t* eqp = ws.t_eq + td.chunk0;
    uint32_t* gtp = ws.t_gt + td.chunk0;
    uint64_t* offp = ws.t_off + td.chunk0;
    uint32_t gt[kPlaceRegs], eq[kPlaceRegs];
    uint64_t lows[kPlaceRegs];
    const bool regs = per <= kPlaceRegs;
    if (regs) {  // in flight during the search for tau
#pragma unroll
        for (uint32_t u = 0; u < kPlaceRegs; ++u) {
            const bool in = lo + u < hi;
            gt[u] = in ? gtp[lo + u] : 0u;
            eq[u] = in ? eqp[lo + u] : 0u;
            lows[u] = in ? offp[lo + u] : 0u;
        }
    }
    // the krem-th largest of the low bits: thread i owns the i-th run of
    // max(1, 2^s / kThreads) bins from the top
    const uint32_t bins = 1u << thr_shift(w), run = bins <= (uint32_t)kThreads ? 1u : bins / kThreads;
    const bool owns = threadIdx.x * run < bins;
    const uint32_t* gh = ws.t_hist + (size_t)t * copies * kBins0 + (owns ? bins - threadIdx.x * run : run);
    uint32_t mine = 0;
    for (uint32_t q = 1; owns && q <= run; ++q) mine += *(gh - q);
    uint32_t above = wide_scan<kThreads>(mine, sh[0]);
    if (owns && above < krem && krem <= above + mine) {
        uint32_t q = 1, x = *(gh - 1);
        while (krem > above + x) {
            above += x;
            x = *(gh - ++q);
        }
        found[0] = bins - threadIdx.x * run - q;
        found[1] = above;
    }
    __syncthreads();
    const uint32_t tau_low = found[0];
    const uint32_t need = krem - found[1];
    if (threadIdx.x == 0) {
        ws.t_prefix[t] = thr_key(w) + (bin << thr_shift(w) | tau_low);
        ws.t_krem[t] = need;
    }
    // chunks to read again (more candidates in the k-th key's bin than a word
    // holds): the wave takes those of its lanes' runs one by one
    bool any_again = !regs;
    if (regs) {
#pragma unroll
        for (uint32_t q = 0; q < kPlaceRegs; ++q) any_again = any_again || chunk_again(eq[q], lows[q]);
    }
    for (uint32_t u = 0; __ballot(any_again) && u < per; ++u) {
        const bool in = lo + u < hi;
        uint32_t nb = 0;
        uint64_t word = 0;
        if (regs) {
#pragma unroll
            for (uint32_t q = 0; q < kPlaceRegs; ++q)
                if (q == u) {
                    nb = eq[q];
                    word = lows[q];
                }
        } else if (in) {
            nb = eqp[lo + u];
            word = offp[lo + u];
        }
        uint64_t again = __ballot(chunk_again(nb, word));
        while (again) {
            const int l = (int)__builtin_ctzll(again);
            again &= again - 1;
            uint32_t g, e;
            recount_chunk(ws, td.chunk0 + (uint32_t)__builtin_amdgcn_readlane((int)(lo + u), l), w, bin, tau_low, g,
                          e);
            if (regs && lane_id() == l) {
#pragma unroll
                for (uint32_t q = 0; q < kPlaceRegs; ++q)
                    if (q == u) {
                        gt[q] = g;
                        eq[q] = e;
                        lows[q] = kLowsSame | tau_low;
                    }
            }
        }
    }
    __syncthreads();  // counts and words written by other lanes
    uint32_t eq_run = 0;
    if (regs) {
#pragma unroll
        for (uint32_t u = 0; u < kPlaceRegs; ++u) {
            if (__ballot(eq[u] != 0u)) {
                chunk_counts(gt[u], eq[u], lows[u], tau_low, gt[u], eq[u]);
                eq_run += eq[u];
            }
        }
    } else {
        for (uint32_t q = lo; q < hi; ++q) {
            uint32_t g, e;
            chunk_counts(gtp[q], eqp[q], offp[q], tau_low, g, e);
            eq_run += e;
        }
    }
    // tau-equal candidates before each run, then winners before each run
    const uint32_t eqb0 = wide_scan<kThreads>(eq_run, sh[1]);
    uint32_t sel_run = 0, e = eqb0;
    if (regs) {
#pragma unroll
        for (uint32_t u = 0; u < kPlaceRegs; ++u) {
            sel_run += chunk_winners(gt[u], eq[u], e, need);
            e += eq[u];
        }
    } else {
        for (uint32_t q = lo; q < hi; ++q) {
            uint32_t g, x;
            chunk_counts(gtp[q], eqp[q], offp[q], tau_low, g, x);
            sel_run += chunk_winners(g, x, e, need);
            e += x;
        }
    }
    uint64_t pos = td.off + wide_scan<kThreads>(sel_run, sh[2]);
    e = eqb0;
    if (regs) {
#pragma unroll
        for (uint32_t u = 0; u < kPlaceRegs; ++u) {
            if (lo + u < hi) {
                offp[lo + u] = pos;
                ws.t_eqb[td.chunk0 + lo + u] = e;
                pos += chunk_winners(gt[u], eq[u], e, need);
                e += eq[u];
            }
        }
    } else {
        for (uint32_t q = lo; q < hi; ++q) {
            uint32_t g, x;
            chunk_counts(gtp[q], eqp[q], offp[q], tau_low, g, x);
            offp[q] = pos;
            ws.t_eqb[td.chunk0 + q] = e;
            pos += chunk_winners(g, x, e, need);
            e += x;
        }
    }
}

// Emit the winners of a chunk in index order and clear them in e_new (kDGC:
// and in u) unless the stream pass has; candidates it cleared that lose get
// their values back.  One wave per chunk; ranks come from ballots.
template <bool kDGC>
__global__ __launch_bounds__(kBlock) void topk_emit(const TDesc* __restrict__ d, int T, uint32_t C,
                                                    uint32_t* __restrict__ idx,
                                                    float* __restrict__ val, Ws ws) {
    const int lane = lane_id();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;  // lanes under this one
    const uint32_t c = blockIdx.x * (kBlock / 64) + wave_id();
    const uint32_t m = c < C ? ws.t_ccount[c] : 0u;
    if (m > 0) {
        const int t = tensor_of_chunk(d, T, c);
        float* resid = d[t].resid;
        const uint64_t end = d[t].off + d[t].k;
        const uint32_t tau = ws.t_prefix[t];
        const uint64_t need = ws.t_krem[t];
        const uint32_t zero = kDGC && m > kListMax ? kNoEarlyZero : ws.t_zero[d[t].chunk0];
        const uint2* cand = ws.t_cand + (size_t)c * kChunk;
        uint64_t eq_seen = ws.t_eqb[c];
        uint64_t pos = ws.t_off[c];
        for (uint32_t i0 = 0; i0 < m; i0 += 64) {
            const uint32_t i = i0 + lane;
            uint2 e = make_uint2(0, 0);
            uint32_t key = 0;
            if (i < m) {
                e = cand[cand_at(c, m, i)];
                key = e.y & 0x7FFFFFFFu;
            }
            const bool is_eq = i < m && key == tau;
            const uint64_t meq = __ballot(is_eq);
            const uint64_t eq_rank = eq_seen + (uint64_t)__popcll(meq & below);
            const bool sel = i < m && (key > tau || (is_eq && eq_rank < need));
            const uint64_t msel = __ballot(sel);
            const uint64_t at = pos + (uint64_t)__popcll(msel & below);
            if (sel && at < end) {
                idx[at] = e.x;
                val[at] = u2f(e.y);
                if (key < zero) {
                    if (resid) gp(resid)[e.x] = 0.f;
                    if constexpr (kDGC) gp(vel_of(d[t]))[e.x] = 0.f;
                }
            } else if (i < m && key >= zero) {
                if (resid) gp(resid)[e.x] = u2f(e.y);
                if constexpr (kDGC) gp(vel_of(d[t]))[e.x] = *cand_vel(ws, c, i);
            }
            eq_seen += (uint64_t)__popcll(meq);
            pos += (uint64_t)__popcll(msel);
        }
    }
}

// ------------------------------------------------- few-chunk exact path
// Calls of at most topk_few_chunks_limit() chunks (2048 unless set lower)
// take a path of five launches (the
// general pipeline's per-step launches cost more than the passes themselves
// at these sizes): clear, the histogram pass, then three kernels that each
// redo the previous radix step's bin search from the global histogram in
// every workgroup instead of in a launch of its own:
//   compact:  bin b of the k-th key (digit 0) -> candidates (keys at or
//             above bin b) per chunk, index order; histogram of digit 1
//             among the candidates in bin b;
//   digit 2:  digit 1 -> histogram of digit 2 among the candidates whose
//             digits 0 and 1 match;
//   emit:     digit 2 gives the k-th key tau and how many tau-equal entries
//             to keep; each wave takes one chunk, counts its candidates
//             above and equal to tau, and finds the counts of all earlier
//             chunks of its tensor by looking back over their published
//             counts (decoupled look-back, Merrill and Garland 2016): a
//             chunk's wave publishes its own counts, then its running
//             totals; a wave that finds an earlier chunk unpublished
//             counts that chunk's candidates itself, so no wave waits for
//             another and the pass needs no particular residency.
// Histogram regions: digit 0 in `copies` copies (chunk c adds to copy
// c % copies, which spreads the atomic additions to the busiest bins over
// several addresses; readers add the copies) at t_hist[(t * copies + r) * 2048],
// then digit 1 at t_hist[copies * T * 2048 + t * 1024] and digit 2 at
// t_hist[copies * T * 2048 + T * 1024 + t * 1024].
// Look-back words (t_off, cleared by the histogram pass): bit 62 counts
// published, bit 63 running totals published, bits 61..31 entries above
// tau, bits 30..0 entries equal to tau (chunk counts, or totals over the
// tensor's chunks up to and including this one).
constexpr uint64_t kLbCounts = 1ull << 62, kLbTotals = 1ull << 63;
constexpr int kLbPolls = 16;  // re-reads of unpublished look-back words before counting them
constexpr int kFewCopiesMax = 4;
// digit-0 histogram copies of a few-chunk call of T tensors
inline int few_copies(int T) { return T <= 16 ? kFewCopiesMax : 1; }

namespace {

// Bin holding the target-th largest entry of a global histogram, searched
// by the whole workgroup (thread i owns the i-th run of bins from the top);
// *above receives the entries in higher bins.  Needs 1 <= target <= total.
__device__ uint32_t block_hist_select(const uint32_t* __restrict__ gh, int bins, uint32_t target, uint64_t* sh,
                                      uint32_t* res_sh, uint32_t* above, int copies = 1,
                                      size_t copy_stride = 0) {
    const int per = bins / kBlock;  // 8 or 4
    const int hi = bins - (int)threadIdx.x * per;
    uint32_t h[8];
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) h[q] = q < per ? gh[hi - 1 - q] : 0u;
    for (int r = 1; r < copies; ++r)
#pragma unroll
        for (int q = 0; q < 8; ++q) h[q] += q < per ? gh[r * copy_stride + hi - 1 - q] : 0u;
#pragma unroll
    for (int q = 0; q < 8; ++q) mine += h[q];
    uint64_t tot;
    uint32_t a = (uint32_t)block_excl_scan_u64(mine, sh, tot);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (q < per && a < target && target <= a + h[q]) {
            res_sh[0] = (uint32_t)(hi - 1 - q);
            res_sh[1] = a;
        }
        a += h[q];
    }
    __syncthreads();
    const uint32_t b = res_sh[0];
    *above = res_sh[1];
    __syncthreads();
    return b;
}

// The same over 1024 bins by one wave (lane i owns the i-th run of 16
// bins from the top).
__device__ uint32_t wave_hist_select(const uint32_t* __restrict__ gh, uint32_t target, uint32_t* above) {
    const int lane = lane_id();
    const int hi = kBins12 - lane * 16;
    uint32_t h[16];
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        h[q] = gh[hi - 1 - q];
        mine += h[q];
    }
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    uint32_t a = inc - mine;
    int found = -1;
    uint32_t fa = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        if (found < 0 && a < target && target <= a + h[q]) {
            found = hi - 1 - q;
            fa = a;
        }
        a += h[q];
    }
    const uint64_t m = __ballot(found >= 0);
    const int src = m ? (int)__builtin_ctzll(m) : 0;
    *above = (uint32_t)__shfl(fa, src, 64);
    return (uint32_t)__shfl(found, src, 64);
}

__device__ __forceinline__ uint64_t lb_load(const uint64_t* p) {
    return __hip_atomic_load((unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void lb_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store((unsigned long long*)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t lb_word(uint64_t flag, uint32_t gt, uint32_t eq) {
    return flag | (uint64_t)gt << 31 | (uint64_t)eq;
}

// Candidates of chunk c above and equal to tau, counted by one wave.
__device__ __forceinline__ void wave_count_chunk(const Ws& ws, uint32_t c, uint32_t tau, uint32_t& gt,
                                                 uint32_t& eq) {
    const int lane = lane_id();
    const uint32_t m = ws.t_ccount[c];
    const uint2* cand = ws.t_cand + (size_t)c * kChunk;
    gt = 0;
    eq = 0;
    for (uint32_t i0 = 0; i0 < m; i0 += 64) {
        const uint32_t i = i0 + (uint32_t)lane;
        const uint32_t key = i < m ? cand[i].y & 0x7FFFFFFFu : 0u;
        gt += (uint32_t)__popcll(__ballot(i < m && key > tau));
        eq += (uint32_t)__popcll(__ballot(i < m && key == tau));
    }
}

}  // namespace

// Digit 0 from the histogram pass's counts, then candidate compaction
// (v re-read from the stored e_new, or from g without error feedback) and
// the digit-1 histogram of the candidates in bin b.
__global__ __launch_bounds__(kBlock) void topk_fast_compact(const TDesc* __restrict__ d, int T, uint32_t C,
                                                            int copies, Ws ws) {
    __shared__ uint32_t lh[kBins12];
    __shared__ uint64_t sh[4];
    __shared__ uint32_t res_sh[2];
    const uint32_t c = blockIdx.x;
    const int t = tensor_of_chunk(d, T, c);
    const TDesc td = d[t];
    const uint32_t j = c - td.chunk0;
    float v[kEpt];
    uint32_t valid;
    load_stored_v(td, j, v, valid);  // in flight during the bin search
    for (int b = threadIdx.x; b < kBins12; b += kBlock) lh[b] = 0;
    uint32_t above;
    const uint32_t b0 = block_hist_select(ws.t_hist + (size_t)t * copies * kBins0, kBins0, td.k, sh, res_sh, &above,
                                          copies, kBins0);
    if (j == 0 && threadIdx.x == 0) {
        ws.t_thr[t] = b0 << 20;
        ws.t_fb[t] = td.k - above;  // entries still to select inside bin b
    }
    const uint32_t thr = b0 << 20;
    uint32_t pm = 0;
#pragma unroll
    for (int i = 0; i < kEpt; ++i)
        if (((valid >> i) & 1u) && key_of(v[i]) >= thr) pm |= 1u << i;
    uint64_t packed = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) packed |= (uint64_t)__popc((pm >> (4 * r)) & 0xFu) << (16 * r);
    uint64_t tot;
    const uint64_t pre = block_excl_scan_u64(packed, sh, tot);
    uint2* out = ws.t_cand + (size_t)c * kChunk;
    uint32_t base = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        uint32_t rank = base + (uint32_t)((pre >> (16 * r)) & 0xFFFFu);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 4 * r + q;
            if ((pm >> i) & 1u) {
                const uint32_t e = j * (uint32_t)kChunk + 1024u * r + 4u * threadIdx.x + q;
                const uint32_t key = key_of(v[i]);
                out[rank++] = make_uint2(e, f2u(v[i]));
                if ((key >> 20) == b0) atomicAdd(&lh[(key >> 10) & (kBins12 - 1)], 1u);
            }
        }
        base += (uint32_t)((tot >> (16 * r)) & 0xFFFFu);
    }
    if (threadIdx.x == 0) ws.t_ccount[c] = base;
    __syncthreads();
    flush_hist(lh, ws.t_hist + (size_t)copies * T * kBins0 + (size_t)t * kBins12, kBins12);
}

// Digit 1, then the digit-2 histogram of the candidates whose digits 0 and
// 1 match.
__global__ __launch_bounds__(kBlock) void topk_fast_digit2(const TDesc* __restrict__ d, int T, int copies, Ws ws) {
    __shared__ uint32_t lh[kBins12];
    __shared__ uint64_t sh[4];
    __shared__ uint32_t res_sh[2];
    const uint32_t c = blockIdx.x;
    const int t = tensor_of_chunk(d, T, c);
    const TDesc td = d[t];
    const uint32_t j = c - td.chunk0;
    uint32_t* h1 = ws.t_hist + (size_t)copies * T * kBins0;
    // the chunk's count and first candidates, in flight during the bin search
    // (a slot holds kChunk entries, so the first kBlock are always in bounds)
    const uint32_t m = ws.t_ccount[c];
    const uint2* cand = ws.t_cand + (size_t)c * kChunk;
    const uint32_t key0 = cand[threadIdx.x].y & 0x7FFFFFFFu;
    for (int b = threadIdx.x; b < kBins12; b += kBlock) lh[b] = 0;
    const uint32_t thr = ws.t_thr[t], r0 = ws.t_fb[t];
    uint32_t above;
    const uint32_t d1 = block_hist_select(h1 + (size_t)t * kBins12, kBins12, r0, sh, res_sh, &above);
    const uint32_t prefix = thr | d1 << 10;
    if (j == 0 && threadIdx.x == 0) {
        ws.t_prefix[t] = prefix;
        ws.t_krem[t] = r0 - above;
    }
    if (threadIdx.x < m && (key0 >> 10) == (prefix >> 10)) atomicAdd(&lh[key0 & (kBins12 - 1)], 1u);
    for (uint32_t i = threadIdx.x + kBlock; i < m; i += kBlock) {
        const uint32_t key = cand[i].y & 0x7FFFFFFFu;
        if ((key >> 10) == (prefix >> 10)) atomicAdd(&lh[key & (kBins12 - 1)], 1u);
    }
    __syncthreads();
    flush_hist(lh, h1 + (size_t)T * kBins12 + (size_t)t * kBins12, kBins12);
}

// Digit 2 gives tau; one wave per chunk counts, looks back, and emits its
// winners in index order (clearing them in e_new; kDGC: and in u).
template <bool kDGC>
__global__ __launch_bounds__(kBlock) void topk_fast_emit(const TDesc* __restrict__ d, int T, uint32_t C, int copies,
                                                         uint32_t* __restrict__ idx, float* __restrict__ val,
                                                         Ws ws) {
    const int lane = lane_id();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t c = blockIdx.x * (kBlock / 64) + wave_id();
    if (c >= C) return;
    const int t = tensor_of_chunk(d, T, c);
    const TDesc td = d[t];
    // the chunk's count and first 64 candidates, in flight during the bin
    // search (always inside the chunk's slot)
    const uint32_t m = ws.t_ccount[c];
    const uint2* cand = ws.t_cand + (size_t)c * kChunk;
    const uint2 first = cand[lane];
    const uint32_t prefix = ws.t_prefix[t], r1 = ws.t_krem[t];
    uint32_t above;
    const uint32_t d2 =
        wave_hist_select(ws.t_hist + (size_t)copies * T * kBins0 + (size_t)(T + t) * kBins12, r1, &above);
    const uint32_t tau = prefix | d2;
    const uint32_t need = r1 - above;  // tau-equal entries to keep, lowest indices first
    uint32_t gt, eq;
    {
        const uint32_t key = (uint32_t)lane < m ? first.y & 0x7FFFFFFFu : 0u;
        gt = (uint32_t)__popcll(__ballot((uint32_t)lane < m && key > tau));
        eq = (uint32_t)__popcll(__ballot((uint32_t)lane < m && key == tau));
        for (uint32_t i0 = 64; i0 < m; i0 += 64) {
            const uint32_t i = i0 + (uint32_t)lane;
            const uint32_t k2 = i < m ? cand[i].y & 0x7FFFFFFFu : 0u;
            gt += (uint32_t)__popcll(__ballot(i < m && k2 > tau));
            eq += (uint32_t)__popcll(__ballot(i < m && k2 == tau));
        }
    }
    uint64_t* lb = ws.t_off;
    if (lane == 0) lb_store(lb + c, lb_word(kLbCounts, gt, eq));
    // totals of the earlier chunks of the tensor
    uint32_t gt_b = 0, eq_b = 0;
    for (int64_t q0 = (int64_t)c - 1; q0 >= (int64_t)td.chunk0; q0 -= 64) {
        const int64_t q = q0 - lane;
        const bool in = q >= (int64_t)td.chunk0;
        uint64_t w = in ? lb_load(lb + q) : 0ull;
        uint64_t tot_m;
        int lim;
        // chunks whose waves run alongside this one publish within a few
        // load latencies: poll those still unpublished a bounded number of
        // times before counting them here
        for (int spin = 0;; ++spin) {
            tot_m = __ballot(in && (w & kLbTotals));
            lim = tot_m ? (int)__builtin_ctzll(tot_m) : 63;  // up to the nearest chunk with totals
            const bool pend = in && lane <= lim && w == 0ull;
            if (!__ballot(pend) || spin == kLbPolls) break;
            __builtin_amdgcn_s_sleep(4);
            if (pend) w = lb_load(lb + q);
        }
        const bool use = in && lane <= lim;
        // unpublished chunks: count them here, one at a time with the whole wave
        uint64_t help = __ballot(use && w == 0ull);
        while (help) {
            const int l = (int)__builtin_ctzll(help);
            help &= help - 1;
            uint32_t hg, he;
            wave_count_chunk(ws, (uint32_t)(q0 - l), tau, hg, he);
            if (lane == l) w = lb_word(kLbCounts, hg, he);
        }
        uint32_t g = use ? (uint32_t)(w >> 31) & 0x7FFFFFFFu : 0u;
        uint32_t e = use ? (uint32_t)w & 0x7FFFFFFFu : 0u;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            g += __shfl_xor(g, o, 64);
            e += __shfl_xor(e, o, 64);
        }
        gt_b += g;
        eq_b += e;
        if (tot_m) break;
    }
    if (lane == 0) lb_store(lb + c, lb_word(kLbCounts | kLbTotals, gt_b + gt, eq_b + eq));
    // emit
    if (m == 0) return;
    float* resid = td.resid;
    const uint64_t end = td.off + td.k;
    uint64_t eq_seen = eq_b;
    uint64_t pos = td.off + gt_b + (eq_b < need ? eq_b : need);
    for (uint32_t i0 = 0; i0 < m; i0 += 64) {
        const uint32_t i = i0 + lane;
        uint2 e = make_uint2(0, 0);
        uint32_t key = 0;
        if (i < m) {
            e = i0 == 0 ? first : cand[i];
            key = e.y & 0x7FFFFFFFu;
        }
        const bool is_eq = i < m && key == tau;
        const uint64_t meq = __ballot(is_eq);
        const uint64_t eq_rank = eq_seen + (uint64_t)__popcll(meq & below);
        const bool sel = i < m && (key > tau || (is_eq && eq_rank < need));
        const uint64_t msel = __ballot(sel);
        const uint64_t at = pos + (uint64_t)__popcll(msel & below);
        if (sel && at < end) {
            idx[at] = e.x;
            val[at] = u2f(e.y);
            if (resid) gp(resid)[e.x] = 0.f;
            if constexpr (kDGC) gp(vel_of(td))[e.x] = 0.f;
        }
        eq_seen += (uint64_t)__popcll(meq);
        pos += (uint64_t)__popcll(msel);
    }
}

// Clear the tensors' histograms (T * 2048 words, a multiple of 4) and the
// fallback flag at the start of a call.
__global__ void topk_zero_hist(uint32_t* h, uint64_t n, uint32_t* any) {
    const uint64_t n4 = n / 4;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (uint64_t)gridDim.x * blockDim.x)
        reinterpret_cast<u32x4*>(h)[i] = u32x4{0u, 0u, 0u, 0u};
    if (blockIdx.x == 0 && threadIdx.x == 0) any[0] = 0u;
}

namespace {

template <bool kDGC>
hipError_t launch_topk_t(int kind, double ratio, uint64_t seed, const TDesc* d, int T, uint32_t C,
                         uint32_t* idx, float* val, const Ws& ws, hipStream_t s, const DgcFuse& f) {
    const dim3 blk(kBlock);
    const DgcFuse none{nullptr, 0.f, nullptr};
    if (C <= topk_few_chunks_limit()) {  // few chunks: the five-launch exact path (both kinds: same result)
        const int copies = few_copies(T);
        const uint64_t hn = (uint64_t)T * ((uint64_t)copies * kBins0 + 2 * kBins12);
        uint32_t zb = (uint32_t)((hn / 4 + 255) / 256);
        if (zb > 4096) zb = 4096;
        hipLaunchKernelGGL(topk_zero_hist, dim3(zb), dim3(256), 0, s, ws.t_hist, hn, ws.t_any);
        (void)launch_timed(kTimedTopkHist, topk_hist_pass<kDGC>, dim3(C), blk, 0, s, d, T, C, ws, ws.t_off, copies, f);
        hipLaunchKernelGGL(topk_fast_compact, dim3(C), blk, 0, s, d, T, C, copies, ws);
        hipLaunchKernelGGL(topk_fast_digit2, dim3(C), blk, 0, s, d, T, copies, ws);
        hipLaunchKernelGGL(topk_fast_emit<kDGC>, dim3((C + kBlock / 64 - 1) / (kBlock / 64)), blk, 0, s, d, T, C,
                           copies, idx, val, ws);
        return hipGetLastError();
    }
    const int R = topk_general_copies(T);
    if (kind == 0) {  // exact
        const uint64_t hn = (uint64_t)T * R * kBins0;
        uint32_t zb = (uint32_t)((hn / 4 + 255) / 256);
        if (zb > 4096) zb = 4096;
        hipLaunchKernelGGL(topk_zero_hist, dim3(zb), dim3(256), 0, s, ws.t_hist, hn, ws.t_any);
        hipLaunchKernelGGL(topk_hist_pass<kDGC>, dim3(C), blk, 0, s, d, T, C, ws, (uint64_t*)nullptr, R, f);
        hipLaunchKernelGGL(topk_find_thr, dim3(T), blk, 0, s, d, R, ws);
        (void)launch_timed(kTimedTopkCompact, topk_compact<false, false, false>, dim3(C), blk, 0, s, d, T, R, ws, none);
        hipLaunchKernelGGL(topk_find_bin, dim3(T), blk, 0, s, d, R, ws);
    } else {  // sampled threshold, exact fallback per tensor
        if (T > kWideTensors)
            hipLaunchKernelGGL((topk_threshold<kDGC, kNarrowBlock>), dim3(T), dim3(kNarrowBlock), 0, s, d, ratio, seed,
                               R, topk_max_shift(R), ws, f);
        else
            hipLaunchKernelGGL((topk_threshold<kDGC, kWideBlock>), dim3(T), dim3(kWideBlock), 0, s, d, ratio, seed, R,
                               topk_max_shift(R), ws, f);
        if (C > kNtChunks)
            (void)launch_timed(kTimedTopkCompact, topk_compact<true, kDGC, true>, dim3(C), blk, 0, s, d, T, R, ws, f);
        else
            (void)launch_timed(kTimedTopkCompact, topk_compact<false, kDGC, true>, dim3(C), blk, 0, s, d, T, R, ws,
                               f);
        hipLaunchKernelGGL(topk_find_bin, dim3(T), blk, 0, s, d, R, ws);
        hipLaunchKernelGGL(topk_fallback<kDGC>, dim3(C < 1024u ? C : 1024u), blk, 0, s, d, R, ws);
    }
    if (C >= kCountBatchFrom)
        hipLaunchKernelGGL(topk_cand_count<4>, dim3((C + 15) / 16), blk, 0, s, d, T, C, R, ws);
    else
        hipLaunchKernelGGL(topk_cand_count<1>, dim3((C + 3) / 4), blk, 0, s, d, T, C, R, ws);
    if (T > kWideTensors)
        hipLaunchKernelGGL(topk_place<kNarrowBlock>, dim3(T), dim3(kNarrowBlock), 0, s, d, R, ws);
    else
        hipLaunchKernelGGL(topk_place<kWideBlock>, dim3(T), dim3(kWideBlock), 0, s, d, R, ws);
    hipLaunchKernelGGL(topk_emit<kDGC>, dim3((C + kBlock / 64 - 1) / (kBlock / 64)), blk, 0, s, d, T, C, idx, val,
                       ws);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_topk(int kind, double ratio, uint64_t seed, const TDesc* d, int T, uint32_t C,
                       bool, bool, uint32_t* idx, float* val, const Ws& ws, hipStream_t s, const DgcFuse* dgc) {
    if (C == 0) return hipSuccess;
    if (dgc) return launch_topk_t<true>(kind, ratio, seed, d, T, C, idx, val, ws, s, *dgc);
    return launch_topk_t<false>(kind, ratio, seed, d, T, C, idx, val, ws, s, DgcFuse{nullptr, 0.f, nullptr});
}

}  // namespace bc
