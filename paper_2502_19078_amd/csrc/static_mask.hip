// Prefix-static masks (arXiv 2502.19078): (i) the generation-phase line of the algorithm "CLADA
// Inference" read literally -- the mask is regenerated by thresholding the prefill magnitudes
// A_j of the neuron-activation equation (section 3.2.1) with tau_final, so it only changes when
// the indicator pattern does; (ii) a hard top-k on a prefix aggregate, which is how section 4
// characterises the Griffin baseline.  Both produce an ascending neuron list for
// clada_static_ffn_decode.  The lists are rebuilt rarely (at most once per decode step), F is at
// most 2^18: one workgroup does the whole job, all integer work after the compare.
#include "clada_internal.h"

namespace {

constexpr int NT = 1024;

// Exclusive prefix sum of one int per thread over the workgroup; *total gets the sum.
__device__ __forceinline__ int block_excl_scan(int v, int *s_wave, int *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    __syncthreads();                       // s_wave may still be read from a previous scan
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    int base = 0, all = 0;
    for (int w = 0; w < NT / 64; ++w) {
        const int c = s_wave[w];
        if (w < wave) base += c;
        all += c;
    }
    *total = all;
    return base + inc - v;
}

// Thread t owns the contiguous neurons [t*per, min(F, (t+1)*per)): writes those whose flag is set,
// ascending, behind the flagged neurons of the threads before it.
template <typename Flag>
__device__ __forceinline__ void compact(int F, int per, Flag flag, int *s_wave, int *idx_out, int *n_out)
{
    const int j0 = min(F, (int)threadIdx.x * per), j1 = min(F, j0 + per);
    int c = 0;
    for (int j = j0; j < j1; ++j) c += flag(j) ? 1 : 0;
    int total;
    int pos = block_excl_scan(c, s_wave, &total);
    for (int j = j0; j < j1; ++j)
        if (flag(j)) idx_out[pos++] = j;
    if (threadIdx.x == 0) *n_out = total;
}

__global__ void __launch_bounds__(NT)
k_mask_threshold(const float *__restrict__ A, int F, const float *__restrict__ tau, int *__restrict__ idx_out,
                 int *__restrict__ n_out)
{
    __shared__ int s_wave[NT / 64];
    const float t = tau[0];
    const int per = (F + NT - 1) / NT;
    compact(F, per, [&](int j) { return A[j] >= t; }, s_wave, idx_out, n_out);     // NaN compares false: cut
}

// Unsigned key that orders like the float (larger score -> larger key); -0 and +0 share a key,
// NaN gets the smallest key of all.
__device__ __forceinline__ unsigned int order_key(float f)
{
    if (f != f) return 0u;
    if (f == 0.0f) f = 0.0f;
    const unsigned int u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The k largest scores, ties at the k-th value going to the lower indices.  Radix select of the k-th largest key in three
// passes of 11, 11 and 10 bits, then one ordered compaction.
//
// What bounds it: latency, in one workgroup.  The scores of a 7B layer (44 KB) took 46 us with four 8-bit passes (a wave's
// lanes met in a handful of bins), one thread walking the bins, and a contiguous piece of the scores per thread in the
// compaction; wide digits, a parallel descent and coalesced tiles, the keys held in registers up to 16384 of them, take 13.
constexpr int DIGIT_BINS = 2048, HELD = 16;
__global__ void __launch_bounds__(NT)
k_mask_topk(const float *__restrict__ score, int F, int k, int *__restrict__ idx_out, int *__restrict__ n_out)
{
    constexpr int NWAVE = NT / 64;
    __shared__ int s_hist[DIGIT_BINS];
    __shared__ int s_wave[NWAVE], s_wave2[NWAVE];
    __shared__ unsigned int s_prefix;
    __shared__ int s_remaining;
    __shared__ int s_gt[CLADA_MAX_DFF / 64], s_eq[CLADA_MAX_DFF / 64];       // per tile of 64 scores
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (k <= 0) {
        if (tid == 0) *n_out = 0;
        return;
    }
    if (k > F) k = F;
    unsigned int held[HELD];                                 // key of score i NT + tid
#pragma unroll
    for (int i = 0; i < HELD; ++i) {
        const int j = i * NT + tid;
        held[i] = j < F ? order_key(score[j]) : 0u;
    }
    // f(i, key, valid) for the scores i NT + tid, all threads of a wave together
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < HELD; ++i)
            if (i * NT < F) f(i, held[i], i * NT + tid < F);
        for (int i = HELD; i * NT < F; ++i) {
            const int j = i * NT + tid;
            f(i, j < F ? order_key(score[j]) : 0u, j < F);
        }
    };
    if (tid == 0) { s_prefix = 0u; s_remaining = k; }
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0, bits = pass == 2 ? 10 : 11;
        for (int i = tid; i < DIGIT_BINS; i += NT) s_hist[i] = 0;
        __syncthreads();
        const unsigned int prefix = s_prefix;
        const int rem = s_remaining;
        const unsigned int himask = pass == 0 ? 0u : 0xffffffffu << (shift + bits), dmask = (1u << bits) - 1u;
        each([&](int, unsigned int key, bool valid) {
            if (valid && (key & himask) == prefix) atomicAdd(&s_hist[(key >> shift) & dmask], 1);
        });
        __syncthreads();
        // thread t holds the bins from the largest digit down: 2047 - 2 t and the one below
        const int hi = s_hist[DIGIT_BINS - 1 - 2 * tid], lo = s_hist[DIGIT_BINS - 2 - 2 * tid];
        int all;
        const int before = block_excl_scan(hi + lo, s_wave, &all);
        if (before < rem && before + hi + lo >= rem) {       // exactly one thread: the bin with the rem-th largest
            const bool second = before + hi < rem;
            s_prefix = prefix | ((unsigned int)(DIGIT_BINS - 1 - 2 * tid - (second ? 1 : 0)) << shift);
            s_remaining = rem - before - (second ? hi : 0);  // still to take among keys with this digit
        }
        __syncthreads();
    }
    const unsigned int kth = s_prefix;                       // key of the k-th largest score
    const int need = s_remaining;                            // how many of the scores equal to it are taken
    each([&](int i, unsigned int key, bool valid) {
        const unsigned long long g = __ballot(valid && key > kth), e = __ballot(valid && key == kth);
        if (lane == 0 && i * NT + wave * 64 < F) { s_gt[i * NWAVE + wave] = __popcll(g); s_eq[i * NWAVE + wave] = __popcll(e); }
    });
    __syncthreads();
    // tiles dealt to the threads in order: equal scores before each tile, then the position its first taken one gets
    const int tiles = (F + 63) / 64, per = (tiles + NT - 1) / NT;
    const int t0 = min(tiles, tid * per), t1 = min(tiles, t0 + per);
    int ceq = 0;
    for (int t = t0; t < t1; ++t) ceq += s_eq[t];
    int total;
    int eq = block_excl_scan(ceq, s_wave, &total);
    int c = 0;
    {
        int r = eq;
        for (int t = t0; t < t1; ++t) { c += s_gt[t] + max(0, min(need - r, s_eq[t])); r += s_eq[t]; }
    }
    int pos = block_excl_scan(c, s_wave2, &total);
    for (int t = t0; t < t1; ++t) {
        const int g = s_gt[t], e = s_eq[t];
        s_gt[t] = pos;
        s_eq[t] = eq;
        pos += g + max(0, min(need - eq, e));
        eq += e;
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    each([&](int i, unsigned int key, bool valid) {
        const unsigned long long e = __ballot(valid && key == kth);
        const int t = min(i * NWAVE + wave, tiles - 1);      // (a tile past the end takes nothing)
        const bool take = valid && (key > kth || (key == kth && s_eq[t] + __popcll(e & below) < need));
        const unsigned long long m = __ballot(take);
        if (take) idx_out[s_gt[t] + __popcll(m & below)] = i * NT + tid;
    });
    if (tid == 0) *n_out = total;
}

// Packed storage of a mask: bit j % 32 of word j / 32 is set iff neuron j is kept -- d_ff / 8 bytes
// instead of 4 bytes per kept neuron (the memory the paper's limitations paragraph worries about).
__global__ void __launch_bounds__(NT)
k_mask_pack(const int *__restrict__ idx, const int *__restrict__ n_in, int F, unsigned int *__restrict__ bits)
{
    const int words = (F + 31) / 32;
    for (int w = threadIdx.x; w < words; w += NT) bits[w] = 0u;
    __syncthreads();                                 // one workgroup: its own zeroes are visible to its atomics
    const int n = min(max(n_in[0], 0), F);
    for (int e = threadIdx.x; e < n; e += NT) {
        const int j = idx[e];
        if (j >= 0 && j < F) atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
}

__global__ void __launch_bounds__(NT)
k_mask_unpack(const unsigned int *__restrict__ bits, int F, int *__restrict__ idx_out, int *__restrict__ n_out)
{
    __shared__ int s_wave[NT / 64];
    const int words = (F + 31) / 32;
    const int per = (words + NT - 1) / NT;
    const int w0 = min(words, (int)threadIdx.x * per), w1 = min(words, w0 + per);
    auto word = [&](int w) {                         // bits past d_ff are ignored
        unsigned int v = bits[w];
        if (w == words - 1 && (F & 31)) v &= (1u << (F & 31)) - 1u;
        return v;
    };
    int c = 0;
    for (int w = w0; w < w1; ++w) c += __popc(word(w));
    int total;
    int pos = block_excl_scan(c, s_wave, &total);
    for (int w = w0; w < w1; ++w) {
        unsigned int v = word(w);
        while (v) {
            const int b = __ffs(v) - 1;
            idx_out[pos++] = 32 * w + b;
            v &= v - 1u;
        }
    }
    if (threadIdx.x == 0) *n_out = total;
}

clada_status check_args(clada_ctx *ctx, const void *src, int32_t F, const void *idx_out, const void *n_out)
{
    if (!ctx) return CLADA_ERR_NULL;
    if (!src || !idx_out || !n_out) return clada_fail(ctx, CLADA_ERR_NULL, "an array pointer is NULL");
    if (F < 1 || F > CLADA_MAX_DFF) return clada_fail(ctx, CLADA_ERR_SHAPE, "d_ff=%d outside [1,%d]", F, CLADA_MAX_DFF);
    if (!ctx->ws) return clada_fail(ctx, CLADA_ERR_WORKSPACE, "the context has no workspace (no device)");
    return CLADA_OK;
}

}  // namespace

extern "C" clada_status clada_static_mask_threshold(clada_ctx *ctx, const float *A, int32_t d_ff,
                                                    const float *tau_final, int32_t *active_idx,
                                                    int32_t *n_active, void *hip_stream)
{
    clada_status st = check_args(ctx, A, d_ff, active_idx, n_active);
    if (st != CLADA_OK) return st;
    if (!tau_final) return clada_fail(ctx, CLADA_ERR_NULL, "tau_final is NULL");
    hipLaunchKernelGGL(k_mask_threshold, dim3(1), dim3(NT), 0, (hipStream_t)hip_stream, A, d_ff, tau_final,
                       active_idx, n_active);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}

extern "C" clada_status clada_static_mask_topk(clada_ctx *ctx, const float *score, int32_t d_ff, int32_t k,
                                               int32_t *active_idx, int32_t *n_active, void *hip_stream)
{
    if (ctx && d_ff >= 1 && (k < 0 || k > d_ff)) return clada_fail(ctx, CLADA_ERR_VALUE, "k=%d outside [0,%d]", k, d_ff);
    clada_status st = check_args(ctx, score, d_ff, active_idx, n_active);
    if (st != CLADA_OK) return st;
    hipLaunchKernelGGL(k_mask_topk, dim3(1), dim3(NT), 0, (hipStream_t)hip_stream, score, d_ff, k, active_idx,
                       n_active);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}

extern "C" clada_status clada_mask_pack(clada_ctx *ctx, const int32_t *active_idx, const int32_t *n_active,
                                        int32_t d_ff, uint32_t *mask_bits, void *hip_stream)
{
    clada_status st = check_args(ctx, active_idx, d_ff, mask_bits, n_active);
    if (st != CLADA_OK) return st;
    hipLaunchKernelGGL(k_mask_pack, dim3(1), dim3(NT), 0, (hipStream_t)hip_stream, active_idx, n_active, d_ff,
                       mask_bits);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}

extern "C" clada_status clada_mask_unpack(clada_ctx *ctx, const uint32_t *mask_bits, int32_t d_ff,
                                          int32_t *active_idx, int32_t *n_active, void *hip_stream)
{
    clada_status st = check_args(ctx, mask_bits, d_ff, active_idx, n_active);
    if (st != CLADA_OK) return st;
    hipLaunchKernelGGL(k_mask_unpack, dim3(1), dim3(NT), 0, (hipStream_t)hip_stream, mask_bits, d_ff, active_idx,
                       n_active);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}
