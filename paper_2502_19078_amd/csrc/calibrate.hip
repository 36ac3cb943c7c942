// Base-threshold calibration: exact nearest-rank quantile of the pooled prefix
// magnitudes (the percentile stand-in for the error-bounded search of section
// 3.2.2) by radix select on the fp32 bit patterns.  Non-negative floats order
// like their unsigned bit patterns, so two histogram passes, over bits [30:16]
// and [15:0], pin down the k-th smallest value exactly.  All integer work;
// integer atomics commute, so the result does not depend on scheduling.
//
// What bounds it: two reads of the pool, and for short prefixes the launches.  Three passes of 2048 bins with a select kernel
// after each took 54 us on a pool of 22 MB (7 launches) and 140 us on one of 235 MB; wide histograms in LDS save a pass, the
// second pass descends into the first one's histogram itself (every workgroup alike), and the histograms are kept zero
// between calls, in a part of the workspace that no other call uses (35 and 112 us; 31 and 110 with the histogram cleared by 16 bytes
// and read eight words at a time).
#include <math.h>

#include "clada_internal.h"

namespace {

constexpr int BINS1 = 1 << 15, BINS2 = 1 << 16;      // bits [30:16] and [15:0]
constexpr int COARSE = 256;                          // the leading eight bits of either, so that a descent reads 256 + 256 counts

struct CalibState {
    unsigned long long fine1[BINS1], coarse1[COARSE];        // zero between calls (cleared by k_calib_finish)
    unsigned long long fine2[BINS2], coarse2[COARSE];        // cleared by the first pass of a call
    unsigned long long k2;                                   // remaining 1-based rank inside the prefix
    unsigned int prefix;                                     // bits [30:16] of the result
};
static_assert(sizeof(CalibState) <= CALIB_BYTES, "the header's part for the histograms");

constexpr int CALIB_THREADS = 1024;
constexpr int CHUNK4 = 4 * CALIB_THREADS;            // 16-byte groups a workgroup takes at a time

// Index of the entry of cnt[0..256) that holds the 1-based rank *k, which becomes the rank inside it.  Wave 0 only.
__device__ __forceinline__ int descend256(const unsigned long long *cnt, unsigned long long *k)
{
    const int lane = threadIdx.x & 63;
    unsigned long long c[4], sum = 0ull;
#pragma unroll
    for (int e = 0; e < 4; ++e) { c[e] = cnt[4 * lane + e]; sum += c[e]; }
    unsigned long long inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    unsigned long long run = inc - sum;
    int bin = -1;
    unsigned long long left = 0ull;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (bin < 0 && run < *k && run + c[e] >= *k) { bin = 4 * lane + e; left = *k - run; }
        run += c[e];
    }
    const unsigned long long who = __ballot(bin >= 0);
    const int src = who ? __ffsll((long long)who) - 1 : 63;  // (the counts add up to n >= k: somebody holds it)
    *k = __shfl(left, src);
    return __shfl(bin, src);
}

// One pass.  The magnitudes of a layer crowd into a few hundred of the 2^15 bins, so that a handful of a wave's lanes meet at
// an address; exact zeros (half of a ReLU's) would all meet and are counted apart, in registers.
// One workgroup per compute unit, the next chunk on its way while one is counted.  The second pass counts in 16 bits (two
// bins a word): a wave that may have counted 4095 values since it last did so moves the whole histogram to the result (with
// an exchange per word, so that no count is moved twice); 16 waves cannot overflow a bin in between.
template <int PASS>
__global__ void __launch_bounds__(CALIB_THREADS)
k_calib_hist(const float *__restrict__ pool, long long n, unsigned long long k, CalibState *st)
{
    __shared__ __align__(16) unsigned int s_hist[BINS1];                   // 128 KiB: 2^15 words, or 2^16 half words
    __shared__ unsigned int s_coarse[COARSE];
    __shared__ unsigned int s_prefix, s_zero;
    const int tid = threadIdx.x, lane = tid & 63;
    const long long n4 = n >> 2, n_chunk = (n4 + CHUNK4 - 1) / CHUNK4;
    const u32x4 *p4 = reinterpret_cast<const u32x4 *>(pool);
    auto ask = [&](u32x4 (&v)[4], long long ch) {            // past the end: the pool's first group, not counted
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long long i = ch * CHUNK4 + r * CALIB_THREADS + tid;
            v[r] = n4 > 0 ? __builtin_nontemporal_load(p4 + (i < n4 ? i : 0)) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    u32x4 v[2][4];
    ask(v[0], blockIdx.x);
    for (int i = tid; i < BINS1 / 4; i += CALIB_THREADS) reinterpret_cast<u32x4 *>(s_hist)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid < COARSE) s_coarse[tid] = 0u;
    if (tid == 0) s_zero = 0u;
    if (PASS == 1) {
        unsigned long long *z = st->fine2;                   // fine2 and coarse2 lie side by side
        for (int i = blockIdx.x * CALIB_THREADS + tid; i < BINS2 + COARSE; i += gridDim.x * CALIB_THREADS) z[i] = 0ull;
    } else if (tid < 64) {
        const int c = descend256(st->coarse1, &k);
        unsigned int f = 0u;                                 // 128 bins per coarse one: two per lane
        const unsigned long long a = st->fine1[c * 128 + 2 * lane], b = st->fine1[c * 128 + 2 * lane + 1];
        unsigned long long inc = a + b;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long t = __shfl_up(inc, o);
            if (lane >= o) inc += t;
        }
        const unsigned long long run = inc - a - b;
        const bool mine = run < k && inc >= k;
        const unsigned long long who = __ballot(mine);
        const int src = who ? __ffsll((long long)who) - 1 : 63;
        const bool second = run + a < k;
        const unsigned long long left = k - run - (second ? a : 0ull);
        f = (unsigned int)(c * 128 + 2 * lane + (second ? 1 : 0));
        f = __shfl(f, src);
        const unsigned long long k2 = __shfl(left, src);
        if (lane == 0) s_prefix = f;
        if (blockIdx.x == 0 && lane == 0) { st->prefix = f << 16; st->k2 = k2; }
    }
    __syncthreads();
    const unsigned int prefix = PASS == 2 ? s_prefix : 0u;
    unsigned int zeros = 0u;
    // moves the counts of the words first, first + step, .. to the result: eight words read at a time, neighbouring ones by
    // neighbouring lanes (four in a row per lane, whose occupied words then lie with few lanes: 13.1 -> 27.6 us a pass)
    auto carry = [&](int first, int step) {
        for (int w0 = first; w0 < BINS1; w0 += 8 * step) {   // (BINS1 is a multiple of 8 step)
            unsigned int g[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = s_hist[w0 + e * step];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (!g[e]) continue;
                const int w = w0 + e * step;
                if (PASS == 1) {
                    atomicAdd(&st->fine1[w], (unsigned long long)g[e]);
                    atomicAdd(&s_coarse[w >> 7], g[e]);
                } else {
                    const unsigned int c = atomicExch(&s_hist[w], 0u);
                    if (c & 0xffffu) atomicAdd(&st->fine2[2 * w], (unsigned long long)(c & 0xffffu));
                    if (c >> 16) atomicAdd(&st->fine2[2 * w + 1], (unsigned long long)(c >> 16));
                    atomicAdd(&s_coarse[w >> 7], (c & 0xffffu) + (c >> 16));
                }
            }
        }
    };
    unsigned int took = 0u;                                  // values this lane has counted in the running chunk
    int bound = 0;                                           // at most so many by this wave since its last carry
    auto count = [&](unsigned int u) {
        u &= 0x7fffffffu;
        zeros += u == 0u ? 1u : 0u;
        if (PASS == 1) {
            if (u != 0u) atomicAdd(&s_hist[u >> 16], 1u);
        } else if ((u >> 16) == prefix && u != 0u) {
            atomicAdd(&s_hist[(u & 0xffffu) >> 1], (u & 1u) ? 0x10000u : 1u);
            took = 1u;
        }
    };
    auto count_chunk = [&](const u32x4 (&w)[4], long long ch) {
        took = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (ch * CHUNK4 + r * CALIB_THREADS + tid < n4) {
#pragma unroll
                for (int e = 0; e < 4; ++e) count(w[r][e]);
            }
        }
        if (PASS == 2) {
            bound += 16 * __popcll(__ballot(took != 0u));
            if (bound + 1024 > 4095 - 3) { carry(lane, 64); bound = 0; }
        }
    };
    for (long long ch = blockIdx.x; ch < n_chunk; ch += 2 * (long long)gridDim.x) {
        const long long c1 = ch + gridDim.x, c2 = c1 + gridDim.x;
        if (c1 < n_chunk) ask(v[1], c1);
        count_chunk(v[0], ch);
        if (c2 < n_chunk) ask(v[0], c2);
        if (c1 < n_chunk) count_chunk(v[1], c1);
    }
    if (blockIdx.x == 0) {                                   // the last n % 4 values
        const unsigned int *p1 = reinterpret_cast<const unsigned int *>(pool);
        if ((n4 << 2) + tid < n) count(p1[(n4 << 2) + tid]);
    }
    if (zeros) atomicAdd(&s_zero, zeros);                    // (a workgroup sees fewer than 2^32 values)
    __syncthreads();
    carry(tid, CALIB_THREADS);
    __syncthreads();
    if (tid == 0 && s_zero && (PASS == 1 || prefix == 0u)) {
        atomicAdd(PASS == 1 ? &st->fine1[0] : &st->fine2[0], (unsigned long long)s_zero);
        atomicAdd(&s_coarse[0], s_zero);
    }
    __syncthreads();
    if (tid < COARSE && s_coarse[tid]) atomicAdd(PASS == 1 ? &st->coarse1[tid] : &st->coarse2[tid], (unsigned long long)s_coarse[tid]);
}

// Workgroup 0 descends into the second histogram; all of them clear the first one for the next call.
__global__ void __launch_bounds__(256) k_calib_finish(CalibState *st, float *tau_out)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < BINS1 + COARSE; i += gridDim.x * 256) st->fine1[i] = 0ull;   // (coarse1 follows fine1)
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        unsigned long long k = st->k2;
        const int c = descend256(st->coarse2, &k);
        const int f = descend256(st->fine2 + c * 256, &k);
        if (threadIdx.x == 0) *tau_out = __uint_as_float(st->prefix | (unsigned int)(c * 256 + f));
    }
}

__global__ void __launch_bounds__(256) k_calib_clear(CalibState *st)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < BINS1 + COARSE; i += gridDim.x * 256) st->fine1[i] = 0ull;
}

}  // namespace

size_t clada_ws_calibrate(void) { return 256; }      // (the histograms are in the header)

extern "C" clada_status clada_threshold_calibrate(clada_ctx *ctx, const float *abs_act_pool, int64_t n,
                                                  float target_sparsity, float *tau_base_out,
                                                  void *hip_stream)
{
    if (!ctx) return CLADA_ERR_NULL;
    if (!abs_act_pool || !tau_base_out) return clada_fail(ctx, CLADA_ERR_NULL, "pool or output is NULL");
    if (n < 1) return clada_fail(ctx, CLADA_ERR_SHAPE, "n=%lld must be >= 1", (long long)n);
    if (!(target_sparsity >= 0.0f) || !(target_sparsity < 1.0f))
        return clada_fail(ctx, CLADA_ERR_VALUE, "target_sparsity=%g outside [0,1)", (double)target_sparsity);
    if (!aligned16(abs_act_pool)) return clada_fail(ctx, CLADA_ERR_ALIGN, "pool must be 16-byte aligned");
    const size_t need = CLADA_WS_HEADER + clada_ws_calibrate();
    if (ctx->ws_bytes < need)
        return clada_fail(ctx, CLADA_ERR_WORKSPACE, "workspace %zu < %zu bytes needed", ctx->ws_bytes, need);
    // nearest rank, taken in fp64 on the fp32 value of q
    long long k = (long long)ceil((double)target_sparsity * (double)n);
    if (k < 1) k = 1;
    if (k > n) k = n;
    CalibState *st = reinterpret_cast<CalibState *>(ctx->ws + CALIB_STATE);
    hipStream_t stream = (hipStream_t)hip_stream;
    const long long want = ((n >> 2) + CHUNK4 - 1) / CHUNK4;
    const int cap = ctx->num_cu;
    const int blocks = (int)(want < 1 ? 1 : (want > cap ? cap : want));
    // The first histogram is zero between calls because the last kernel clears it.  A call that a refused launch cut short
    // may leave it filled: the next one clears it first.  (Recorded into a graph, that clearing has not run yet: the mark stays.)
    hipStreamCaptureStatus cap_status = hipStreamCaptureStatusNone;
    if (ctx->calib_dirty) {
        CLADA_CHECK_HIP(ctx, hipStreamIsCapturing(stream, &cap_status));
        hipLaunchKernelGGL(k_calib_clear, dim3(32), dim3(256), 0, stream, st);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
    }
    const int mark = cap_status != hipStreamCaptureStatusNone;
    ctx->calib_dirty = 1;
    hipLaunchKernelGGL(k_calib_hist<1>, dim3(blocks), dim3(CALIB_THREADS), 0, stream, abs_act_pool, (long long)n, (unsigned long long)k, st);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL(k_calib_hist<2>, dim3(blocks), dim3(CALIB_THREADS), 0, stream, abs_act_pool, (long long)n, (unsigned long long)k, st);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL(k_calib_finish, dim3(32), dim3(256), 0, stream, st, tau_base_out);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    ctx->calib_dirty = mark;
    return CLADA_OK;
}
