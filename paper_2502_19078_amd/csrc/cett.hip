// Error-bounded base-threshold search (arXiv 2502.19078, section 3.2.2, base-threshold equation):
//     tau_base = max eps  s.t.  mean over validation tokens of CETT(x; eps) <= bound,
//     CETT(x; eps) = || sum_{j : |a_j(x)| < eps} h_j(x) W_down[j,:] ||_2 / || MLP(x) ||_2.
//
// The gate/up GEMM runs once (|a| pool and h stay in the workspace), the dense down projection
// gives the denominators, and every probe of eps is one masking pass over h plus one down
// projection whose epilogue reduces the output rows to sums of squares.  The search is a
// bisection on the bit pattern of the non-negative float eps (monotone in eps), with the bracket
// kept on the device: lo always satisfies the bound, hi never does, 31 probes resolve the float.
#include <type_traits>

#include "clada_internal.h"

namespace {

struct CettState {
    unsigned int lo, hi, mid;     // float bit patterns; the probe in flight is `mid`
    float mean_lo, mean_mid;      // mean CETT at lo / at the last probe
    // the large search (see k_cett_next): what has been measured so far, and the running sum's state
    int skip;                     // no further dense probe is needed
    int done;                     // the bisection has ended
    unsigned int known_lo, known_hi;      // largest feasible / smallest infeasible bit pattern measured
    float known_mean;             // mean CETT at known_lo
    int xlo, xhi, x, side;        // their places in the sorted sample, the probe's, which side moved last
    int same;                     // probes since the start while only one side has been measured
    float glo, ghi;               // mean - bound there (one is halved while the other side keeps moving)
    unsigned int base;            // the cut sums in buffer `sel` hold the neurons below this bit pattern
    int sel;
    int listed;                   // the neurons inside the first bracket are listed (no token had too many)
    // the search over a table (see k_cett_ladder)
    int kept;                     // the cut sums in buffer `sel` are those at `base`
    unsigned int edge, cut;       // the table's window: the magnitudes from known_lo up to here; up to where every token's fit
    int at, xt;                   // places of the expected answer (-1: none) and of `edge`
    int arrive;                   // workgroups of k_cett_curve that are done
};
static_assert(2 * sizeof(CettState) <= 256, "two of them in their place in the workspace");

// den[t] = || MLP(x_t) ||_2 from the per-column-tile sums of squares (ascending tile order);
// thread 0 of block 0 sets up the bracket, or the single probe of an evaluation call.
__global__ void __launch_bounds__(256)
k_cett_begin(CettState *st, const float *__restrict__ rowsq, int n_tn, int T, float *__restrict__ den,
             int search, float eps)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < T && rowsq) {                 // (the non-gated family's denominators come from k_cett_row_norm)
        float s = 0.0f;
#pragma unroll 8
        for (int i = 0; i < n_tn; ++i) s += rowsq[(size_t)i * T + t];
        den[t] = sqrtf(s);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->lo = 0u;                      // eps = 0 cuts nothing: CETT = 0
        st->hi = 0x7f800000u;             // eps = +inf cuts everything: CETT = 1 > bound
        st->mid = search ? (0x7f800000u >> 1) : __float_as_uint(eps);
        st->mean_lo = 0.0f;
        st->mean_mid = 0.0f;
    }
}

// den[t] = || y[t,:] ||_2 of a stored output (layer dtype): the denominators of the non-gated family, whose
// output carries the bias b_out that no neuron owns (the projection's own epilogue adds it to y; the row-norm
// epilogues do not know about it).  One wave per token: lane-strided sums of squares, then a fixed butterfly.
template <int ES>
__global__ void __launch_bounds__(256)
k_cett_row_norm(const char *__restrict__ y, int T, int d, float *__restrict__ den)
{
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T) return;
    const char *row = y + (size_t)t * d * ES;
    float s = 0.0f;
    for (int i = lane; i < d; i += 64) {
        const float v = ES == 4 ? reinterpret_cast<const float *>(row)[i]
                                : __uint_as_float((unsigned int)reinterpret_cast<const unsigned short *>(row)[i] << 16);
        s = fmaf(v, v, s);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) den[t] = sqrtf(s);
}

// hcut = h where |a| < eps (strict, NaN never cut), 0 elsewhere; eps = the probe in the state.
// One thread per 8 neurons when the rows allow 16-byte accesses, else per neuron.
template <int ES>
__global__ void __launch_bounds__(256)
k_cett_mask(const CettState *__restrict__ st, const float *__restrict__ pool, const char *__restrict__ h,
            char *__restrict__ hcut, int T, int F, int Fp, int may_skip)
{
    if (may_skip == 1 && st->skip) return;
    if (may_skip == 2 && st->kept) return;
    const float eps = __uint_as_float(st->mid);
    const size_t groups = (size_t)Fp / 8;
    const size_t total = (size_t)T * groups;
    for (size_t g = (size_t)blockIdx.x * 256 + threadIdx.x; g < total; g += (size_t)gridDim.x * 256) {
        const size_t t = g / groups;
        const int j0 = (int)(g % groups) * 8;
        const float *pr = pool + t * (size_t)F;
        const char *hr = h + (t * (size_t)Fp + j0) * ES;
        char *dr = hcut + (t * (size_t)Fp + j0) * ES;
        bool cut[8];
        if (F % 4 == 0 && j0 + 8 <= F) {
            const float4 p0 = *reinterpret_cast<const float4 *>(pr + j0);
            const float4 p1 = *reinterpret_cast<const float4 *>(pr + j0 + 4);
            cut[0] = p0.x < eps; cut[1] = p0.y < eps; cut[2] = p0.z < eps; cut[3] = p0.w < eps;
            cut[4] = p1.x < eps; cut[5] = p1.y < eps; cut[6] = p1.z < eps; cut[7] = p1.w < eps;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) cut[e] = (j0 + e < F) && (pr[j0 + e] < eps);
        }
        if (ES == 2) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(hr);
            u32x4 o;
            o.x = (cut[0] ? v.x & 0x0000ffffu : 0u) | (cut[1] ? v.x & 0xffff0000u : 0u);
            o.y = (cut[2] ? v.y & 0x0000ffffu : 0u) | (cut[3] ? v.y & 0xffff0000u : 0u);
            o.z = (cut[4] ? v.z & 0x0000ffffu : 0u) | (cut[5] ? v.z & 0xffff0000u : 0u);
            o.w = (cut[6] ? v.w & 0x0000ffffu : 0u) | (cut[7] ? v.w & 0xffff0000u : 0u);
            *reinterpret_cast<u32x4 *>(dr) = o;
        } else {
            const u32x4 v0 = *reinterpret_cast<const u32x4 *>(hr), v1 = *reinterpret_cast<const u32x4 *>(hr + 16);
            u32x4 o0, o1;
            o0.x = cut[0] ? v0.x : 0u; o0.y = cut[1] ? v0.y : 0u; o0.z = cut[2] ? v0.z : 0u; o0.w = cut[3] ? v0.w : 0u;
            o1.x = cut[4] ? v1.x : 0u; o1.y = cut[5] ? v1.y : 0u; o1.z = cut[6] ? v1.z : 0u; o1.w = cut[7] ? v1.w : 0u;
            *reinterpret_cast<u32x4 *>(dr) = o0;
            *reinterpret_cast<u32x4 *>(dr + 16) = o1;
        }
    }
}

// One workgroup: per-token CETT of the probe, their mean in a fixed order (thread i sums tokens
// i, i+1024, ...; then a tree over the threads), and the bisection step.
__global__ void __launch_bounds__(1024)
k_cett_update(CettState *st, const float *__restrict__ rowsq, int n_tn, int T, const float *__restrict__ den,
              float bound, int search, float *__restrict__ cett_out, float *__restrict__ mean_out)
{
    __shared__ float s_sum[1024];
    const int tid = threadIdx.x;
    float acc = 0.0f;
    for (int t = tid; t < T; t += 1024) {
        float s = 0.0f;
        for (int i = 0; i < n_tn; ++i) s += rowsq[(size_t)i * T + t];
        const float dn = den[t];
        const float c = dn > 0.0f ? sqrtf(s) / dn : 0.0f;       // a zero dense output has nothing to lose
        if (cett_out) cett_out[t] = c;
        acc += c;
    }
    s_sum[tid] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) s_sum[tid] += s_sum[tid + w];
        __syncthreads();
    }
    if (tid == 0) {
        const float mean = s_sum[0] / (float)T;
        st->mean_mid = mean;
        if (mean_out) *mean_out = mean;
        if (search) {
            unsigned int lo = st->lo, hi = st->hi;
            const unsigned int mid = st->mid;
            if (mean <= bound) { lo = mid; st->mean_lo = mean; }     // NaN fails the test: treated as over the bound
            else hi = mid;
            st->lo = lo;
            st->hi = hi;
            st->mid = lo + ((hi - lo) >> 1);
        }
    }
}

__global__ void k_cett_finish(const CettState *st, float *tau_out, float *mean_out)
{
    if (threadIdx.x == 0) {
        *tau_out = __uint_as_float(st->lo);
        if (mean_out) *mean_out = st->mean_lo;
    }
}

// ---------------------------------------------------------------------------------------------------------------------
// The large search.  A dense probe costs a masked projection (80 us for 512 tokens of a 7B layer), and bisecting the bit
// pattern from 0 .. +inf spends 31 of them, most on thresholds whose answer is known from a neighbour.  Here
//   (1) some dense probes close a bracket around the answer, at thresholds taken from a sorted sample of the pool: as a
//       function of the rank the mean is smooth (as one of the threshold it is not: SiLU's minimum piles the magnitudes up).
//       The curve of sqrt(sum of the cut h^2 / sum of all h^2) over a few tokens -- what the mean would be if the rows of W_down
//       were orthogonal and of one length -- says where to probe first and, scaled through a measured point, second; from then
//       on false position with the Illinois rule.  Three or four probes leave about forty magnitudes per token (without the
//       curve six or seven);
//   (2) the last feasible probe leaves the cut sums at the bracket's lower end in fp32;
//   (3) up to 1024 tokens the first or second probe is near enough: a table of every token's CETT at the few dozen magnitudes
//       above it answers the rest of the bisection (k_cett_ladder, k_cett_bisect).  Where the answer lies past the table, two
//       more probes close the bracket, and a second table follows;
//   (4) what that leaves open (thousands of equal magnitudes), and searches over more tokens: the plain bisection; a probe
//       outside the bracket is answered by it, one inside adds the rows of the neurons between the sums' threshold and
//       the probe to the sums, token by token, for the next few probes at a time.
// us (plain bisection / without the table / so): 512 tokens of 4096 x 11008 2370 / 470 - 580 / 330 - 390, 80 of 3584 x 9728 - / 296 - 340 / 214 - 229,
// 64 of 1024 x 4096 - / 244 - 287 / 176 - 186, 700 of 4096 x 11008 - / 670 - 835 / 449 - 556, fp32 104 of 4096 x 12992 - / 1218 - 1409 / 828 - 851.
// What bounds it now: the three or four projections (63 us each at the first of these sizes), then launches, 2.4 us each also where nothing is
// left to do.  The bracket answers for thresholds outside it as a monotone mean would; inside, every probe is measured.
constexpr int SAMPLES = 4096;      // sorted sample of the pool; neighbours are 2.7 magnitudes per token apart at 11008 neurons
constexpr int CLOSE = 16;          // sample places left between the bracket's ends when the dense probes end
constexpr int DENSE_PROBES = 5;    // launched; those past the end return at once
constexpr int CURVE_TOKENS = 32, CURVE_BINS = 256, CURVE_STEP = SAMPLES / CURVE_BINS;
// The search over a table takes the curve of up to 128 tokens, which costs no more, and two dense probes before each of two tables.
constexpr int CURVE_TABLE = 128, TABLE_PROBES = 2;
// Places of the sample that the table goes past the expected answer, and that the first probe stays below it, for a table of at most
// `window` places: the first estimate was within 12 places (22 for layers of a few thousand neurons), one through a measured
// point within 4 (11 where d is 64).
__host__ __device__ __forceinline__ int table_past(int window) { return window < 24 ? 4 : window < 128 ? window / 4 : 32; }
__host__ __device__ __forceinline__ int table_below(int window) { return window < 24 ? 6 : window < 120 ? window / 3 : 40; }
// Tokens up to which every workgroup of a probe forms the previous one's mean itself: that saves a launch a probe, and costs
// T^2 reads.  In place / by a launch of its own, us per search: 533 / 564 and 1142 / 1171 (512 tokens, 1024 x 4096 and
// 4096 x 11008), 631 / 633 and 1805 / 1785 (1024), 949 / 870 and 3119 / 2910 (2048), 3848 / 2271 (8192), 92600 / 8200 (65536).
constexpr int MEAN_IN_PLACE = 1024;

// The sorted bit patterns of SAMPLES pool entries.  The entries lie at the fractions i * phi mod 1 of the pool (phi the golden
// ratio, 2^64 phi^-1 below): evenly spread over the tokens, without a stride that could meet the same neurons of every token.
// Every workgroup reads them all and places 16 of them by counting the smaller ones, 16 threads an entry (34 us as a sorting network
// in one workgroup, 17 with 64 entries a workgroup and four threads each, 10 so).  The workgroups behind those form the denominators of
// the gated families, den[t] = || MLP(x_t) ||_2 from the sums of squares per column tile, ascending.
constexpr int SAMPLE_WGS = SAMPLES / 16;
__global__ void __launch_bounds__(256)
k_cett_sample(CettState *st, const float *__restrict__ pool, unsigned long long n, unsigned int *__restrict__ sample, float bound,
              const float *__restrict__ rowsq, int n_tn, int T, float *__restrict__ den, unsigned long long *__restrict__ curve)
{
    __shared__ __align__(16) unsigned int s[SAMPLES];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= SAMPLE_WGS) {
        const int t = ((int)blockIdx.x - SAMPLE_WGS) * 256 + tid;
        if (t >= T) return;
        float v = 0.0f;
#pragma unroll 8
        for (int i = 0; i < n_tn; ++i) v += rowsq[(size_t)i * T + t];
        den[t] = sqrtf(v);
        return;
    }
#pragma unroll
    for (int k = 0; k < SAMPLES / 256; ++k) {
        const int i = k * 256 + tid;
        const unsigned long long r = (unsigned long long)(i + 1) * 0x9e3779b97f4a7c15ull;
        const unsigned int u = __float_as_uint(pool[__umul64hi(r, n)]) & 0x7fffffffu;
        s[i] = u < 0x7f800000u ? u : 0x7f800000u;
    }
    __syncthreads();
    const int i = blockIdx.x * 16 + (tid >> 4), share = tid & 15;
    const unsigned int mine = s[i];
    int below = 0;
    // groups of four entries, the shares in turn: those in front of this workgroup's, which also win ties, its own, those behind
    const int own = blockIdx.x * 4;
    auto group = [&](int j) { return reinterpret_cast<const u32x4 *>(s)[j]; };
#pragma unroll 4
    for (int j = share; j < own; j += 16) {
        const u32x4 v = group(j);
#pragma unroll
        for (int e = 0; e < 4; ++e) below += v[e] <= mine ? 1 : 0;
    }
    if (share < 4) {
        const int j = own + share;
        const u32x4 v = group(j);
#pragma unroll
        for (int e = 0; e < 4; ++e) below += v[e] < mine || (v[e] == mine && 4 * j + e < i) ? 1 : 0;
    }
#pragma unroll 4
    for (int j = own + 4 + share; j < SAMPLES / 4; j += 16) {
        const u32x4 v = group(j);
#pragma unroll
        for (int e = 0; e < 4; ++e) below += v[e] < mine ? 1 : 0;
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) below += __shfl_xor(below, o);
    if (share == 0) sample[below] = mine;
    if (blockIdx.x == 0) curve[tid] = 0ull;                  // (CURVE_BINS threads)
    if (blockIdx.x == 0 && tid == 0) {
        st->skip = 0; st->done = 0; st->sel = 1;
        st->known_lo = 0u; st->known_hi = 0x7f800000u; st->known_mean = 0.0f;
        st->xlo = -1; st->xhi = SAMPLES; st->side = 0; st->same = 0;
        st->glo = -bound; st->ghi = 1.0f - bound;
        st->kept = 1; st->base = 0u; st->edge = st->cut = 0u; st->at = -1; st->arrive = 0;
        st->lo = 0u; st->hi = 0x7f800000u; st->mean_lo = 0.0f;
    }
}

// The curve at a place of the sample, and the place where it reaches a value (linear between its entries; m[b] at place 16 (b + 1)).
__device__ __forceinline__ float curve_at(const float *m, int x)
{
    const int b = x / CURVE_STEP;
    const float lo = b > 0 ? m[b - 1] : 0.0f, hi = b < CURVE_BINS ? m[b] : 1.0f;
    return lo + (hi - lo) * (float)(x - b * CURVE_STEP) / (float)CURVE_STEP;
}
__device__ __forceinline__ int curve_place(const float *m, float v)
{
    int b = 0;                                               // entries below v
    for (int w = CURVE_BINS / 2; w > 0; w >>= 1) b += m[b + w - 1] < v ? w : 0;
    const float lo = b > 0 ? m[b - 1] : 0.0f, hi = m[b];
    return b * CURVE_STEP + (hi > lo && v > lo ? (int)fminf((v - lo) / (hi - lo) * CURVE_STEP, (float)CURVE_STEP) : 0);
}

// One token of the curve: entry b = sqrt(sum of h^2 where |a| is below the sample's place 16 b, over the sum of all).  The sums are
// integers (a bin's share of 2^40), so that the order of the additions does not matter.
template <int ES>
__global__ void __launch_bounds__(1024)
k_cett_curve(CettState *st, const float *__restrict__ pool, const char *__restrict__ h, const unsigned int *__restrict__ sample, int T, int F,
             int Fp, unsigned long long *__restrict__ total, float *__restrict__ mean, float bound, int below)
{
    constexpr int AHEAD = 12;                                // values of a thread in hand at a time (all of them up to 12288 neurons)
    __shared__ unsigned int s_edge[CURVE_BINS];
    __shared__ unsigned long long s_sum[CURVE_BINS];
    __shared__ float s_part[16];
    __shared__ float s_m[CURVE_BINS];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63;
    const size_t t = (size_t)blockIdx.x * T / gridDim.x;
    float sq[AHEAD];
    auto squares = [&](int j0) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int j = j0 + k * 1024 + tid;
            const size_t at = t * Fp + (j < F ? j : 0);
            const float v = ES == 4 ? reinterpret_cast<const float *>(h)[at]
                                    : __uint_as_float((unsigned int)reinterpret_cast<const unsigned short *>(h)[at] << 16);
            sq[k] = j < F ? v * v : 0.0f;
        }
    };
    if (tid < CURVE_BINS) {
        s_edge[tid] = sample[tid * CURVE_STEP];
        s_sum[tid] = 0ull;
    }
    float sum = 0.0f;
    for (int j0 = 0; j0 < F; j0 += AHEAD * 1024) {
        squares(j0);
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) sum += sq[k];
    }
    sum = wave_sum(sum);
    if (lane == 0) s_part[tid >> 6] = sum;
    __syncthreads();
    float all = 0.0f;
    for (int w = 0; w < 16; ++w) all += s_part[w];
    const float scale = all > 0.0f && all < 1e38f ? 1099511627776.0f / all : 0.0f;
    for (int j0 = 0; j0 < F; j0 += AHEAD * 1024) {
        unsigned int a[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int j = j0 + k * 1024 + tid;
            a[k] = __float_as_uint(pool[t * F + (j < F ? j : 0)]) & 0x7fffffffu;
        }
        if (F > AHEAD * 1024) squares(j0);
        int bin[AHEAD];
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) bin[k] = 0;          // the last edge that a reaches; below the first: bin 0 as well
#pragma unroll
        for (int w = CURVE_BINS / 2; w > 0; w >>= 1)
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) bin[k] += s_edge[bin[k] + w] <= a[k] ? w : 0;
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const float v = sq[k] * scale;
            if (v > 0.0f && v < 2e12f) atomicAdd(&s_sum[bin[k]], (unsigned long long)v);       // (a NaN fails the test)
        }
    }
    __syncthreads();
    if (tid < CURVE_BINS) {                                  // (four whole waves)
        unsigned long long run = 0ull;                       // below edge tid + 1: the bins up to this one
        for (int b = 0; b < CURVE_BINS; b += 64) {
            unsigned long long c = s_sum[b + lane];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long x = __shfl_up(c, o);
                if (lane >= o) c += x;
            }
            if (b == (tid & ~63)) run += c;
            else if (b < tid) run += __shfl(c, 63);
        }
        // (again an integer, a token's share of 2^48: the workgroups add up in any order.  The old value is waited for: the sum is
        // where all of them meet then, with no cache written back: 16.8 us, 42 with an agent-scope fence)
        const unsigned long long old = atomicAdd(&total[tid], (unsigned long long)(sqrtf((float)run * (1.0f / 1099511627776.0f)) * 281474976710656.0f));
        if (old == ~0ull) s_last = 0;                        // (never)
    }
    // the last workgroup to arrive: the mean of the tokens' curves, and the first probe, so many places below their answer
    __syncthreads();
    if (tid == 0) s_last = __hip_atomic_fetch_add(&st->arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    if (tid < CURVE_BINS) {
        const unsigned long long all = __hip_atomic_load(&total[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float m = (float)all * (1.0f / 281474976710656.0f) / (float)gridDim.x;
        mean[tid] = m;
        s_m[tid] = m;
    }
    __syncthreads();
    if (tid != 0) return;
    int x = curve_place(s_m, bound) - below;
    x = x < 1 ? 1 : x > SAMPLES - 2 ? SAMPLES - 2 : x;
    if (below > 0 && sample[x] == 0u) {                      // (nothing lies below 0: the first place above it)
        int at = x;
        for (int w = SAMPLES / 2; w > 0; w >>= 1) at += at + w < SAMPLES && sample[at + w] == 0u ? w : 0;
        x = at < SAMPLES - 2 ? at + 1 : SAMPLES - 2;
    }
    st->x = x;
    st->mid = sample[x];
}

// Mean CETT of the probe (as in k_cett_update; the sum over the column tiles and over the tokens in the same order).
__device__ __forceinline__ float mean_cett(const float *__restrict__ rowsq, int n_tn, int T, const float *__restrict__ den, float *s_sum)
{
    const int tid = threadIdx.x;
    float acc = 0.0f;
    for (int t = tid; t < T; t += 1024) {
        float s = 0.0f;
#pragma unroll 8
        for (int i = 0; i < n_tn; ++i) s += rowsq[(size_t)i * T + t];
        const float dn = den[t];
        acc += dn > 0.0f ? sqrtf(s) / dn : 0.0f;
    }
    s_sum[tid] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) s_sum[tid] += s_sum[tid + w];
        __syncthreads();
    }
    return s_sum[0] / (float)T;
}

// The bisection up to the next threshold that has to be measured.
__device__ __forceinline__ void bisect_on(CettState &s)
{
    while (s.hi - s.lo > 1u) {
        const unsigned int mid = s.lo + ((s.hi - s.lo) >> 1);
        if (mid <= s.known_lo) s.lo = mid;
        else if (mid >= s.known_hi) s.hi = mid;
        else { s.mid = mid; return; }
    }
    s.done = 1;
    s.mean_lo = s.known_mean;                                // (lo has come to rest on known_lo)
}

// The next dense probe at place x of the sample, if its threshold lies inside the bracket.
__device__ __forceinline__ bool probe_at(CettState &s, const unsigned int *sample, int x)
{
    if (x <= s.xlo || x >= s.xhi || sample[x] <= s.known_lo || sample[x] >= s.known_hi) return false;
    s.x = x;
    s.mid = sample[x];
    return true;
}

// After a dense probe: the bracket, and the next probe between its ends.  window: places that a table holds (0: there is none);
// stage: 0 after the first probe, 1 after the second, which the first table follows, 2 after others, 3 after the last one.
__global__ void __launch_bounds__(1024)
k_cett_next(CettState *st, const float *__restrict__ rowsq, int n_tn, int T, const float *__restrict__ den, float bound,
            const unsigned int *__restrict__ sample, const float *__restrict__ curve, int window, int two, int stage)
{
    __shared__ float s_sum[1024], s_m[CURVE_BINS];
    if (st->skip) return;
    if (threadIdx.x < CURVE_BINS) s_m[threadIdx.x] = curve[threadIdx.x];
    const float mean = mean_cett(rowsq, n_tn, T, den, s_sum);
    if (threadIdx.x != 0) return;
    CettState s = *st;
    const bool feasible = mean <= bound;                     // NaN: over the bound
    if (feasible) { if (s.mid > s.known_lo) { s.known_lo = s.base = s.mid; s.known_mean = mean; s.sel ^= 1; } }     // (its sums are kept)
    else if (s.mid < s.known_hi) s.known_hi = s.mid;
    auto take = [&](bool low, float g) {                     // the place x becomes an end of the bracket
        if (low) { s.xlo = s.x; s.glo = g; if (s.side < 0) s.ghi *= 0.5f; s.side = -1; }
        else { s.xhi = s.x; s.ghi = g; if (s.side > 0) s.glo *= 0.5f; s.side = 1; }
    };
    float g = mean - bound;
    if (!feasible && !(g > 0.0f)) g = 1.0f;                  // (NaN)
    take(feasible, g);
    // The window is final: it begins where the cut sums are, at the last feasible probe or at 0.  With one buffer of sums they are formed
    // again where a probe that failed came after that.
    auto finish = [&](unsigned int edge, int place) {
        s.skip = 1;
        s.edge = s.cut = edge;
        s.xt = place;
        if (!two) {
            s.sel = 0;
            if (!s.kept) s.base = s.mid = s.known_lo;
        }
        *st = s;
    };
    if (window > 0) {
        s.kept = two || feasible || s.base == 0u;
        // the answer by the curve through the measured point
        int at = -1;
        if (mean > 0.0f && mean < 1e30f) {
            at = curve_place(s_m, curve_at(s_m, s.x) * (bound / mean));
            at = at > s.xlo ? at < s.xhi ? at : s.xhi : s.xlo;
        } else if (feasible) {
            at = (s.x + s.xhi) / 2;                          // (nothing cut yet)
        }
        s.at = at;
        const int past = table_past(window);
        int up = at + past < s.xhi ? at + past : s.xhi;
        while (up < s.xhi && sample[up] <= s.known_lo) ++up;
        if (up < s.xhi && sample[up] >= s.known_hi) up = s.xhi;
        // the first table's upper end need not be measured, the second one's is
        if (stage < 2 && at >= 0 && up - s.xlo <= window) { finish(up < s.xhi ? sample[up] : s.known_hi, up); return; }
        if (stage == 3 || (s.xhi < SAMPLES && s.xhi - s.xlo <= window)) { finish(s.known_hi, s.xhi); return; }
        if (at >= 0) {
            const int further = past << (2 * s.same);
            int x;
            if (s.xhi >= SAMPLES) x = stage == 0 ? at - past : at + further;        // nothing measured above it
            else if (s.xlo < 0) x = at - further;                                   // nothing below
            else x = at - s.xlo >= s.xhi - at ? at - past : at + past;              // the wider side
            ++s.same;
            if (probe_at(s, sample, x)) { *st = s; return; }
        }
    }
    const bool one_side = s.xlo < 0 || s.xhi >= SAMPLES;     // only one end of the bracket is a measured one
    if (one_side && s.same < 4 && mean > 0.0f && mean < 1e30f) {
        // the curve through the measured point, a little past its answer (further each time the answer stays on one side)
        const int at = curve_place(s_m, curve_at(s_m, s.x) * (bound / mean)), past = (CLOSE / 2) << (2 * s.same);
        int x = feasible ? at + past : at - past;
        if (feasible && x <= s.xlo) x = s.xlo + past;
        if (!feasible && x >= s.xhi) x = s.xhi - past;
        ++s.same;
        if (x > s.xlo && x < s.xhi && sample[x] > s.known_lo && sample[x] < s.known_hi) {
            s.x = x;
            s.mid = sample[x];
            *st = s;
            return;
        }
    }
    for (int guard = 0;; ++guard) {
        if (s.xhi - s.xlo <= CLOSE || guard >= 64) { s.skip = 1; break; }
        const float pos = (float)s.xlo + (float)(s.xhi - s.xlo) * (-s.glo / (s.ghi - s.glo));
        // a little past the estimate, towards the end that did not move last: the bracket closes from both sides
        int x = (int)(s.side > 0 ? pos - 0.4f * CLOSE : pos + 0.4f * CLOSE);
        x = x > s.xlo ? x : s.xlo + 1;
        s.x = x < s.xhi ? x : s.xhi - 1;
        s.mid = sample[s.x];
        if (s.mid <= s.known_lo) take(true, s.glo);          // equal magnitudes: measured already
        else if (s.mid >= s.known_hi) take(false, s.ghi);
        else break;
    }
    if (window > 0 && s.skip) finish(s.known_hi, s.xhi);
    else *st = s;
}

// The threshold of the cut sums (the bracket's lower end), and the start of the bisection.  stage 1: the sums were formed by a pass of
// their own, in the first buffer; stage 2: by the probe that measured the threshold.
__global__ void k_cett_base(CettState *st, int stage)
{
    if (threadIdx.x != 0) return;
    if (stage == 0) { st->mid = st->known_lo; return; }      // for the masking pass
    CettState s = *st;
    s.base = s.known_lo;
    if (stage == 1) s.sel = 0;
    s.listed = 1;
    s.lo = 0u;
    s.hi = 0x7f800000u;
    bisect_on(s);
    st[0] = s;
}

// Ascending list of the entries i of [0, n) that want(i) names, by a workgroup of 256 threads, 16 per thread and round of
// 4096; f(position, i) for each, then done(count) by all threads between barriers.
template <typename Want, typename Put, typename Done>
__device__ __forceinline__ void list_ascending(int n, int *s_cnt, Want want, Put put, Done done)
{
    constexpr int PER = 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int seg = 0; seg < n; seg += 256 * PER) {
        unsigned int in = 0u;
        int before[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            before[k] = 0;
            if (seg + k * 256 < n) {
                const int i = seg + k * 256 + tid;
                const bool w = want(i < n ? i : n - 1) && i < n;
                const unsigned long long m = __ballot(w);
                in |= w ? 1u << k : 0u;
                before[k] = __popcll(m & ((1ull << lane) - 1ull));
                if (lane == 0) s_cnt[k * 4 + wave] = __popcll(m);
            } else if (lane == 0) {
                s_cnt[k * 4 + wave] = 0;
            }
        }
        __syncthreads();
        const int c = s_cnt[lane];                           // 64 counts in ascending order of their entries
        int inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(inc, o);
            if (lane >= o) inc += x;
        }
        const int total = __shfl(inc, 63), excl = inc - c;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int at = __shfl(excl, k * 4 + wave) + before[k];
            if ((in >> k) & 1u) put(at, seg + k * 256 + tid);
        }
        __syncthreads();
        done(total);
    }
}

// The neurons of every token with base <= |a| < known_hi, the only ones that later probes add: cap of them per token
// fit; a token with more leaves `listed` at zero, and the probes look through the whole pool.
__global__ void __launch_bounds__(1024)
k_cett_list(CettState *st, const float *__restrict__ pool, int F, int *__restrict__ list, int cap, int *__restrict__ count)
{
    constexpr int PER = 4;                                   // consecutive neurons of a thread in a round of 4096
    __shared__ int s_part[2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t t = blockIdx.x;
    if (st->done) return;
    const float lo = __uint_as_float(st->base), hi = __uint_as_float(st->known_hi);
    int *mine = list + t * cap;
    float a[PER], next[PER];
    auto ask = [&](float (&v)[PER], int seg) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int j = seg + PER * tid + e;
            v[e] = pool[t * F + (j < F ? j : F - 1)];
        }
    };
    ask(a, 0);
    int at = 0;
    for (int seg = 0, turn = 0; seg < F; seg += PER * 1024, turn ^= 1) {
        if (seg + PER * 1024 < F) ask(next, seg + PER * 1024);
        int c = 0, in = 0;
#pragma unroll
        for (int e = 0; e < PER; ++e)
            if (a[e] >= lo && a[e] < hi && seg + PER * tid + e < F) { in |= 1 << e; ++c; }
        int inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(inc, o);
            if (lane >= o) inc += x;
        }
        if (lane == 63) s_part[turn][wave] = inc;
        __syncthreads();                                     // (two buffers: a wave writes the next one while another reads this)
        int put = at + inc - c;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) put += s_part[turn][w];
            at += s_part[turn][w];
        }
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            if ((in >> e) & 1) {
                if (put < cap) mine[put] = seg + PER * tid + e;
                ++put;
            }
            a[e] = next[e];
        }
    }
    if (tid == 0) {
        count[t] = min(at, cap);
        if (at > cap) st->listed = 0;
    }
}

// A measured threshold's answer, and the bisection up to the next one.
__device__ __forceinline__ void answer(CettState &s, bool feasible, float mean)
{
    if (feasible) {
        s.known_lo = s.mid;
        s.known_mean = mean;
    } else {
        s.known_hi = s.mid;                                  // NaN: over the bound
    }
    bisect_on(s);
}

// The search over a table, up to 1024 tokens.  The rows of the neurons inside the window [known_lo, edge) of a token, added in the
// order of their magnitudes to the cut sums at known_lo, give the token's CETT at every threshold of the window: a step function of as many
// steps.  One pass forms them all, and the rest of the bisection reads them, in one workgroup: two launches where the probes
// below need a launch per three steps of the bisection.  The window's upper end need not be measured, so that one or two
// dense probes are enough.  The entries lie in the registers of one workgroup, 44 a thread (two words each of 128): 256 a
// token up to 128 tokens, 176 up to 256, 88 up to 512, 44 beyond.
// Searches whose first two probes fail or fall short by more than the window take the probes' way on; so does a token with more than
// 512 neurons to add.
constexpr int TABLE_TOKENS = 1024, TABLE_REGS = 44;       // entries a thread
constexpr int LADDER_MAX = 512;                          // neurons of a token that the pass can sort; beyond, the window ends at known_lo

// Threads a token in k_cett_bisect, entries of a token, places of the sample that give two thirds of them.
__host__ __device__ constexpr int table_threads(int T) { return T > 512 ? 1 : T > 256 ? 2 : T > 128 ? 4 : 8; }
__host__ __device__ constexpr int table_cap(int T) { return T > 128 ? table_threads(T) * TABLE_REGS : 256; }
// (a token whose cut sums lie below the window lists the neurons in between too; those that the sort has no room for leave the window empty)
static_assert(2 * table_cap(1) <= LADDER_MAX && table_cap(129) <= table_cap(1), "a full window and as many neurons below it can be sorted");
int table_window(int T, int F) { return (int)((long long)table_cap(T) * 2 / 3 * SAMPLES / F); }

// A workgroup of NT threads per token.  mag [cap][T], cett [cap + 1][T] (at known_lo, and behind each entry), count [T].
template <int ES, int NV, int NT>
__global__ void __launch_bounds__(NT)
k_cett_ladder(CettState *st, const float *__restrict__ pool, const char *__restrict__ h, const char *__restrict__ wd,
              const float *__restrict__ buf0, const float *__restrict__ buf1, const float *__restrict__ den, int T, int F, int Fp, int d, int cap,
              float *__restrict__ mag, float *__restrict__ cett, int *__restrict__ count)
{
    constexpr int VEC = 16 / ES, AHEAD = 8, SCAN = 12, WAVES = NT / 64;
    __shared__ unsigned int s_a[LADDER_MAX];
    __shared__ int s_i[LADDER_MAX], s_j[LADDER_MAX + 2 * AHEAD];
    __shared__ float s_h[LADDER_MAX + 2 * AHEAD], s_sq[WAVES][257];
    __shared__ int s_n, s_pre;
    __shared__ unsigned int s_edge;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t t = blockIdx.x;
    if (st->done || !st->skip) return;
    const unsigned int base = st->base, lo = st->known_lo, edge = st->edge;
    const float *src = (st->sel ? buf1 : buf0) + t * d;
    const int col0 = tid * VEC;                              // group v of this thread: columns col0 + v NT VEC ..
    if (tid == 0) { s_n = 0; s_pre = 0; s_edge = edge; }
    __syncthreads();
    // the window's neurons and those between the sums' threshold and the window, in any order
    unsigned int next[SCAN];
    auto ask = [&](int j0) {
#pragma unroll
        for (int k = 0; k < SCAN; ++k) {
            const int j = j0 + k * NT + tid;
            next[k] = __float_as_uint(pool[t * F + (j < F ? j : F - 1)]);
        }
    };
    ask(0);
    float acc[NV][VEC];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int col = col0 + v * NT * VEC;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[v][e] = col < d && base != 0u ? src[col + e] : 0.0f;    // (nothing lies below 0)
    }
    for (int j0 = 0; j0 < F; j0 += SCAN * NT) {
        unsigned int a[SCAN];
#pragma unroll
        for (int k = 0; k < SCAN; ++k) a[k] = next[k];
        if (j0 + SCAN * NT < F) ask(j0 + SCAN * NT);
#pragma unroll
        for (int k = 0; k < SCAN; ++k) {
            const int j = j0 + k * NT + tid;
            const bool in = a[k] >= base && a[k] < edge && j < F;       // (magnitudes are not negative; a NaN lies above +inf)
            const unsigned long long who = __ballot(in);
            if (who) {
                int at = 0;
                if (lane == 0) at = atomicAdd(&s_n, __popcll(who));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(who & ((1ull << lane) - 1ull));
                if (in && at < LADDER_MAX) { s_a[at] = a[k]; s_i[at] = j; }
            }
        }
    }
    __syncthreads();
    const int found = s_n;
    for (int i = tid; i < min(found, LADDER_MAX); i += NT)
        if (s_a[i] < lo) atomicAdd(&s_pre, 1);
    __syncthreads();
    const int pre = s_pre;
    if (found > LADDER_MAX) {                                // (uniform) too many to sort: nothing is known about the window
        if (tid == 0) { atomicMin(&st->cut, lo); count[t] = 0; }
        return;
    }
    // their places by magnitude, equal ones by neuron; those from `cap` on, and all equal to the first of them, are left out
    int rank[LADDER_MAX / NT];
#pragma unroll
    for (int u = 0; u < LADDER_MAX / NT; ++u) {
        const int i = tid + NT * u;
        rank[u] = LADDER_MAX;
        if (i < found) {
            const unsigned int a = s_a[i];
            const int j = s_i[i];
            int r = 0;
#pragma unroll 8
            for (int k = 0; k < found; ++k) r += s_a[k] < a || (s_a[k] == a && s_i[k] < j) ? 1 : 0;
            rank[u] = r;
            if (r == cap + pre) s_edge = a;
        }
    }
    if (tid == 0) s_n = 0;
    __syncthreads();
    const unsigned int end = s_edge;
#pragma unroll
    for (int u = 0; u < LADDER_MAX / NT; ++u) {
        const int i = tid + NT * u;
        const bool in = i < found && rank[u] < cap + pre && s_a[i] < end;
        const unsigned long long who = __ballot(in);
        if (who && lane == 0) atomicAdd(&s_n, __popcll(who));
        if (in) {
            const int j = s_i[i];
            s_j[rank[u]] = j;
            s_h[rank[u]] = ES == 4 ? reinterpret_cast<const float *>(h)[t * Fp + j]
                                   : __uint_as_float((unsigned int)reinterpret_cast<const unsigned short *>(h)[t * Fp + j] << 16);
            if (rank[u] >= pre) mag[(size_t)(rank[u] - pre) * T + t] = __uint_as_float(s_a[i]);
        }
    }
    __syncthreads();
    const int n = s_n;
    if (tid < 2 * AHEAD) { s_j[n + tid] = n > 0 ? s_j[n - 1] : 0; s_h[n + tid] = 0.0f; }       // (what is requested past the end)
    if (tid == 0) {
        if (end != edge) atomicMin(&st->cut, end);
        count[t] = n - pre;
    }
    auto norm2 = [&]() {
        float q = 0.0f;
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (col0 + v * NT * VEC < d)
#pragma unroll
                for (int e = 0; e < VEC; ++e) q = fmaf(acc[v][e], acc[v][e], q);
        return q;
    };
    const float before = wave_sum(norm2());
    if (lane == 0 && pre == 0) s_sq[wave][0] = before;
    __syncthreads();
    u32x4 w[2][AHEAD][NV];
    auto rows = [&](u32x4 (&to)[AHEAD][NV], int e0) {
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            const char *row = wd + (size_t)s_j[e0 + q] * d * ES;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int col = col0 + v * NT * VEC;
                to[q][v] = *reinterpret_cast<const u32x4 *>(row + (size_t)(col < d ? col : 0) * ES);
            }
        }
    };
    auto add = [&](const u32x4 (&from)[AHEAD][NV], int e0) {
        float sq[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            const float hv = s_h[e0 + q];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                float f[VEC];
                unpack_row16(from[q][v], f);
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[v][e] = fmaf(hv, f[e], acc[v][e]);
            }
            sq[q] = norm2();
        }
        // eight sums over 64 lanes: halves exchanged until a lane holds one of them, then eight lanes each
        const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
        float s4[4], s2[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float give = b5 ? sq[i] : sq[i + 4], keep = b5 ? sq[i + 4] : sq[i];
            s4[i] = keep + __shfl_xor(give, 32);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float give = b4 ? s4[i] : s4[i + 2], keep = b4 ? s4[i + 2] : s4[i];
            s2[i] = keep + __shfl_xor(give, 16);
        }
        float s1 = (b3 ? s2[1] : s2[0]) + __shfl_xor(b3 ? s2[0] : s2[1], 8);
        s1 += __shfl_xor(s1, 4);
        s1 += __shfl_xor(s1, 2);
        s1 += __shfl_xor(s1, 1);
        const int e = e0 + (b5 ? 4 : 0) + (b4 ? 2 : 0) + (b3 ? 1 : 0);
        if ((lane & 7) == 0 && e < n && e + 1 >= pre) s_sq[wave][e + 1 - pre] = s1;
    };
    if (n > 0) {
        rows(w[0], 0);
        for (int e0 = 0; e0 < n; e0 += 2 * AHEAD) {
            if (e0 + AHEAD < n) rows(w[1], e0 + AHEAD);
            add(w[0], e0);
            if (e0 + 2 * AHEAD < n) rows(w[0], e0 + 2 * AHEAD);
            if (e0 + AHEAD < n) add(w[1], e0 + AHEAD);
        }
    }
    __syncthreads();
    const float dn = den[t];
    for (int i = tid; i <= n - pre; i += NT) {
        float q = 0.0f;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) q += s_sq[v][i];
        cett[(size_t)i * T + t] = dn > 0.0f ? sqrtf(q) / dn : 0.0f;
    }
}

// The bisection over the table, one workgroup, TPT threads a token (the entries in turn).  A threshold past the window, where that
// ends below what has been measured, is left to the probes below, which go on from the cut sums at the window's lower end.
template <int TPT>
__global__ void __launch_bounds__(1024)
k_cett_bisect(CettState *st, const float *__restrict__ mag, const float *__restrict__ cett, const int *__restrict__ count, int T, float bound,
              const unsigned int *__restrict__ sample, const float *__restrict__ curve, int window, int second)
{
    constexpr int N = TPT == 8 ? 256 / TPT : TABLE_REGS;
    __shared__ float s_sum[2][16];
    __shared__ int s_most;
    const int tid = threadIdx.x, lane = tid & 63, t = tid / TPT, u = tid % TPT;
    const bool here = t < T;
    const int n = here ? count[t] : 0;
    int word[sizeof(CettState) / 4];                         // (the state in scalar registers)
#pragma unroll
    for (int i = 0; i < (int)(sizeof(CettState) / 4); ++i) word[i] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int *>(st)[i]);
    CettState s;
    __builtin_memcpy(&s, word, sizeof(s));
    if (s.done || !s.skip) return;
    if (tid == 0) s_most = 0;
    __syncthreads();
    const int share = (n + TPT - 1) / TPT, own = min(max(n - u * share, 0), share);        // entries u share ..
    float a[N], c[N];
    // (loads without branches: past the end, the token's first entry is read and not taken)
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const size_t at = (size_t)(k < own ? u * share + k : 0) * T + (here ? t : 0);
        a[k] = mag[at];
        c[k] = cett[at + (k < own ? T : 0)];
    }
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] = k < own ? a[k] : __uint_as_float(0x7f800000u);
    const float first = cett[here ? t : 0];
    if (lane == 0 || own > 0) atomicMax(&s_most, own);
    __syncthreads();
    const int most = s_most;                                 // (at most N)
    int turn = 0;
    auto mean_at = [&](unsigned int bits) {                  // (all threads)
        const float eps = __uint_as_float(bits);
        float v = first;                                     // the last entry below eps
#pragma unroll
        for (int k0 = 0; k0 < N; k0 += 4) {
            if (k0 < most) {
#pragma unroll
                for (int k = k0; k < k0 + 4; ++k) {
                    v = a[k] < eps ? c[k] : v;
                }
            }
        }
        // of a token's shares, the last one that begins below eps
        const bool begins = u == 0 || a[0] < eps;
        const unsigned long long who = __ballot(begins);
        const bool mine = begins && (u == TPT - 1 || !((who >> ((lane + 1) & 63)) & 1ull));
        const float sum = wave_sum(mine && here ? v : 0.0f);
        if (lane == 0) s_sum[turn][tid >> 6] = sum;
        __syncthreads();
        float m = 0.0f;
#pragma unroll
        for (int w = 0; w < 16; ++w) m += s_sum[turn][w];
        turn ^= 1;
        return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(m / (float)T)));
    };
    s.kept = 1;
    s.listed = 1;
    s.lo = 0u;
    s.hi = 0x7f800000u;
    float beyond = -1.0f;                                    // the mean at the window's end, where that satisfies the bound
    const unsigned int edge = s.cut;
    bool table = edge > s.known_lo;
    if (table && edge < s.known_hi) {                        // the window's end first
        const float mean = mean_at(edge);
        if (mean <= bound) {
            s.known_lo = edge;
            s.known_mean = beyond = mean;
            table = false;
        } else {
            s.known_hi = edge;                               // NaN: over the bound
        }
    }
    bisect_on(s);
    while (table && !s.done) {
        const float mean = mean_at(s.mid);
        answer(s, mean <= bound, mean);
    }
    if (tid != 0) return;
    if (!s.done && !second) {
        // past the window, or too many neurons in it: the dense probes go on, above what is known
        const int past = table_past(window);
        if (beyond >= 0.0f) {
            s.xlo = s.xt;
            s.glo = beyond - bound;
            s.side = -1;
            if (beyond > 0.0f) {
                const int at = curve_place(curve, curve_at(curve, s.xt) * (bound / beyond));
                s.at = at > s.xlo ? at < s.xhi ? at : s.xhi : s.xlo;
            }
        }
        s.same = 1;
        s.skip = 0;
        if (!probe_at(s, sample, s.at + past) && !probe_at(s, sample, (s.xlo + s.xhi) / 2)) {
            s.skip = 1;
            s.edge = s.cut = s.known_hi;
        }
    }
    *st = s;
}

// The probes inside the bracket.  A launch measures the thresholds that the next LEVELS steps of the bisection can ask for, a binary
// tree of NODES = 2^LEVELS - 1 of them, and the walk down the tree afterwards is the bisection's own: seven thresholds cost little
// more than one (the rows up to the highest are read once), and the launches follow each other 7 us apart whatever they do
// (one threshold a launch: 224 us of a search of 512 tokens of 4096 x 11008, seven: 170, most of it launches that find nothing left).

// Down the tree with the means of its thresholds in ascending order.
template <int LEVELS>
__device__ __forceinline__ void walk(CettState &s, const float *mean, float bound)
{
    int at = (1 << LEVELS) / 2 - 1;
    for (int l = LEVELS - 2; l >= -1 && !s.done; --l) {
        const bool feasible = mean[at] <= bound;
        answer(s, feasible, mean[at]);
        if (l >= 0) at += feasible ? 1 << l : -(1 << l);
    }
}

// Threshold `node` (ascending) of the tree below s, or the next one up the path where the bisection ends before it gets there.
template <int LEVELS>
__device__ __forceinline__ unsigned int node_threshold(CettState s, int node)
{
    int at = (1 << LEVELS) / 2 - 1;
    unsigned int mid = s.mid;
    for (int l = LEVELS - 2; l >= 0 && at != node; --l) {
        const bool right = node > at;
        answer(s, right, 0.0f);
        if (s.done) break;
        mid = s.mid;
        at += right ? 1 << l : -(1 << l);
    }
    return mid;
}

// The means of the previous launch's thresholds (its row norms: [node][part][T]), by a workgroup of NT threads: to s_mean.
template <int NODES, int NT>
__device__ __forceinline__ void node_means(const float *__restrict__ rowsq, int parts, int T, const float *__restrict__ den, float (*s_sum)[NODES], float *s_mean)
{
    const int tid = threadIdx.x, lane = tid & 63;
    float acc[NODES];
#pragma unroll
    for (int v = 0; v < NODES; ++v) acc[v] = 0.0f;
    for (int t = tid; t < T; t += NT) {
        float sq[NODES];
#pragma unroll
        for (int v = 0; v < NODES; ++v) sq[v] = 0.0f;
        for (int i = 0; i < parts; ++i)
#pragma unroll
            for (int v = 0; v < NODES; ++v) sq[v] += rowsq[((size_t)v * parts + i) * T + t];
        const float dn = den[t];
#pragma unroll
        for (int v = 0; v < NODES; ++v) acc[v] += dn > 0.0f ? sqrtf(sq[v]) / dn : 0.0f;
    }
#pragma unroll
    for (int v = 0; v < NODES; ++v) {
        const float w = wave_sum(acc[v]);
        if (lane == 0) s_sum[tid >> 6][v] = w;
    }
    __syncthreads();
    if (tid < NODES) {
        float m = 0.0f;
        for (int w = 0; w < NT / 64; ++w) m += s_sum[w][tid];
        s_mean[tid] = m / (float)T;
    }
    __syncthreads();
}

// The walk as a launch of its own, in place, for more than MEAN_IN_PLACE tokens.
template <int LEVELS>
__global__ void __launch_bounds__(1024)
k_cett_take(CettState *st, const float *__restrict__ rowsq, int parts, int T, const float *__restrict__ den, float bound)
{
    constexpr int NODES = (1 << LEVELS) - 1;
    __shared__ float s_sum[16][NODES], s_mean[NODES];
    if (st->done) return;
    node_means<NODES, 1024>(rowsq, parts, T, den, s_sum, s_mean);
    if (threadIdx.x == 0) {
        CettState s = *st;
        walk<LEVELS>(s, s_mean, bound);
        *st = s;
    }
}

// Up to MEAN_IN_PLACE tokens every workgroup first takes in the previous launch's answers (the same state and the same norms, so the
// same result; workgroup 0 leaves it for the next launch), beyond k_cett_take has done that (taken).  Then, a workgroup per
// token and part of the columns: the cut sums at `base` plus h_j W_down[j,:] of the neurons up to the largest feasible threshold,
// stored as the new sums, and on to the thresholds of the tree, threshold after threshold, ascending within each; the
// sums of squares at each of them to rowsq.
template <int ES, int NV, int LEVELS>
__global__ void __launch_bounds__(256)
k_cett_between(CettState *__restrict__ sts, int launch, int taken, const float *__restrict__ pool, const char *__restrict__ h,
               const char *__restrict__ wd, const int *__restrict__ list, int cap, const int *__restrict__ count,
               float *__restrict__ buf0, float *__restrict__ buf1, const float *__restrict__ rowsq_in, float *__restrict__ rowsq,
               const float *__restrict__ den, float bound, int T, int F, int Fp, int d)
{
    constexpr int VEC = 16 / ES, SEG = 4096, NODES = (1 << LEVELS) - 1, AHEAD = 8;
    __shared__ int s_cnt[64], s_j[SEG], s_end[NODES + 1];
    __shared__ float s_h[SEG], s_sum[4][NODES], s_mean[NODES], s_edge[NODES + 2];
    __shared__ CettState s_st;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, parts = gridDim.y, part = blockIdx.y;
    const CettState *in = sts + (launch & 1);
    const bool take = !taken && launch > 0 && !in->done;
    if (take) node_means<NODES, 256>(rowsq_in, parts, T, den, s_sum, s_mean);
    if (tid == 0) {
        CettState s = *in;
        if (take) walk<LEVELS>(s, s_mean, bound);
        s_st = s;
        if (blockIdx.x == 0 && part == 0) {
            if (!s.done && s.base != s.known_lo) { s.base = s.known_lo; s.sel ^= 1; }       // what this launch leaves
            sts[(launch + 1) & 1] = s;
        }
    }
    __syncthreads();
    if (s_st.done) return;
    if (tid == 0) { s_edge[0] = __uint_as_float(s_st.base); s_edge[1] = __uint_as_float(s_st.known_lo); }
    if (tid < NODES) s_edge[2 + tid] = __uint_as_float(node_threshold<LEVELS>(s_st, tid));
    __syncthreads();
    // segment i: edge[i] <= |a| < edge[i + 1]; a threshold that is not needed repeats another one and leaves the order: made ascending here
    float edge[NODES + 2];
    edge[0] = s_edge[0]; edge[1] = s_edge[1];
#pragma unroll
    for (int v = 0; v < NODES; ++v) edge[2 + v] = fmaxf(edge[1 + v], s_edge[2 + v]);
    const size_t t = blockIdx.x;
    const bool listed = s_st.listed != 0, moved = s_st.base != s_st.known_lo;
    const float *src = (s_st.sel ? buf1 : buf0) + t * d;
    float *dst = (s_st.sel ? buf0 : buf1) + t * d;
    const int col0 = (part * NV * 256 + tid) * VEC;          // group v of this thread: columns col0 + v 256 VEC ..
    float acc[NV][VEC], sq[NODES];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int col = col0 + v * 256 * VEC;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[v][e] = col < d && s_st.base != 0u ? src[col + e] : 0.0f;      // (nothing lies below 0)
    }
    const int *mine = list + t * cap;
    auto magnitude = [&](int i) { return pool[t * F + (listed ? mine[i] : i)]; };
    auto put = [&](int at, int i) {
        const int j = listed ? mine[i] : i;
        s_j[at] = j;
        s_h[at] = ES == 4 ? reinterpret_cast<const float *>(h)[t * Fp + j]
                          : __uint_as_float((unsigned int)reinterpret_cast<const unsigned short *>(h)[t * Fp + j] << 16);
    };
    // the end of segment i: the new sums, or the norm at a threshold
    auto ended = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        float q = 0.0f;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int col = col0 + v * 256 * VEC;
            if (col < d) {
                if constexpr (i == 0) {
                    if (moved)
#pragma unroll
                        for (int e = 0; e < VEC; e += 4)
                            *reinterpret_cast<float4 *>(dst + col + e) = make_float4(acc[v][e], acc[v][e + 1], acc[v][e + 2], acc[v][e + 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) q = fmaf(acc[v][e], acc[v][e], q);
                }
            }
        }
        if constexpr (i > 0) sq[i - 1] = q;
    };
    // entries [0, total) of s_j / s_h added in order, AHEAD rows requested together; before entry e is added, done(e)
    auto add_rows = [&](int total, auto done) {
        for (int e0 = 0; e0 < total; e0 += AHEAD) {
            u32x4 w[AHEAD][NV];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                const char *row = wd + (size_t)s_j[min(e0 + q, total - 1)] * d * ES;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int col = col0 + v * 256 * VEC;
                    w[q][v] = *reinterpret_cast<const u32x4 *>(row + (size_t)(col < d ? col : 0) * ES);
                }
            }
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                if (e0 + q < total) {
                    done(e0 + q);
                    const float hv = s_h[e0 + q];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        float f[VEC];
                        unpack_row16(w[q][v], f);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) acc[v][e] = fmaf(hv, f[e], acc[v][e]);
                    }
                }
            }
        }
    };
    const int n = listed ? count[t] : F;
    if (listed && n <= 256) {                                // an entry per thread: all segments in one go, in their order
        const float a = tid < n ? magnitude(tid) : -1.0f;
        int seg = -1;                                        // NaN and everything outside: none
#pragma unroll
        for (int i = 0; i <= NODES; ++i) seg = a >= edge[i] && a < edge[i + 1] ? i : seg;
        int before = 0;
#pragma unroll
        for (int i = 0; i <= NODES; ++i) {
            const unsigned long long who = __ballot(seg == i);
            if (lane == 0) s_cnt[i * 4 + wave] = __popcll(who);
            if (seg == i) before = __popcll(who & ((1ull << lane) - 1ull));
        }
        __syncthreads();
        int at = 0, run = 0;
#pragma unroll
        for (int i = 0; i <= NODES; ++i) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if (seg == i && w == wave) at = run;
                run += s_cnt[i * 4 + w];
            }
            if (tid == 0) s_end[i] = run;
        }
        if (seg >= 0) put(at + before, tid);
        __syncthreads();
        int open = 0;                                        // segments that have ended (uniform)
        auto close = [&](int e, bool all) {
            while (open <= NODES && (all || s_end[open] <= e)) {
                switch (open) {
                case 0: ended(std::integral_constant<int, 0>{}); break;
                case 1: ended(std::integral_constant<int, 1>{}); break;
                case 2: if constexpr (NODES >= 2) ended(std::integral_constant<int, 2 < NODES ? 2 : NODES>{}); break;
                case 3: if constexpr (NODES >= 3) ended(std::integral_constant<int, 3 < NODES ? 3 : NODES>{}); break;
                case 4: if constexpr (NODES >= 4) ended(std::integral_constant<int, 4 < NODES ? 4 : NODES>{}); break;
                case 5: if constexpr (NODES >= 5) ended(std::integral_constant<int, 5 < NODES ? 5 : NODES>{}); break;
                case 6: if constexpr (NODES >= 6) ended(std::integral_constant<int, 6 < NODES ? 6 : NODES>{}); break;
                case 7: if constexpr (NODES >= 7) ended(std::integral_constant<int, 7 < NODES ? 7 : NODES>{}); break;
                }
                ++open;
            }
        };
        add_rows(run, [&](int e) { close(e, false); });
        close(0, true);
    } else {
        auto one = [&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if (edge[i] < edge[i + 1])
                list_ascending(n, s_cnt, [&](int k) { const float a = magnitude(k); return a >= edge[i] && a < edge[i + 1]; }, put,
                               [&](int total) { add_rows(total, [](int) {}); __syncthreads(); });
            ended(ic);
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        if constexpr (NODES >= 3) { one(std::integral_constant<int, 2>{}); one(std::integral_constant<int, 3>{}); }
        if constexpr (NODES >= 7) {
            one(std::integral_constant<int, 4>{}); one(std::integral_constant<int, 5>{});
            one(std::integral_constant<int, 6>{}); one(std::integral_constant<int, 7>{});
        }
    }
#pragma unroll
    for (int v = 0; v < NODES; ++v) {
        const float q = wave_sum(sq[v]);
        if (lane == 0) s_sum[wave][v] = q;
    }
    __syncthreads();
    if (tid < NODES) rowsq[((size_t)tid * parts + part) * T + t] = (s_sum[0][tid] + s_sum[1][tid]) + (s_sum[2][tid] + s_sum[3][tid]);
}

struct CettWs {
    float *part, *pool, *rowsq_den, *rowsq_num, *den, *splitk;
    size_t splitk_bytes;
    char *h, *hcut, *ytmp;
    CettState *state;
    // room for the parts of a down projection; `one` ([T][d] fp32) is free while it runs, or receives its fp32 rows
    DownRoom room(void *one) const { return {splitk, splitk_bytes, reinterpret_cast<float *>(one)}; }
};

CettWs carve(char *ws, size_t bytes, int d, int F, int T)
{
    const size_t n_tm = (size_t)clada_prefix_token_tiles(T), n_tn = (size_t)clada_prefix_col_tiles(d);
    const size_t Fp = align_up((size_t)F, 64);
    CettWs w;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = ws + off; off += align_up(bytes, 256); return p; };
    w.part = reinterpret_cast<float *>(take(sizeof(float) * 4 * n_tm * F));
    w.pool = reinterpret_cast<float *>(take(sizeof(float) * (size_t)T * F));
    w.h = take((size_t)T * Fp * 4);
    w.hcut = take((size_t)T * Fp * 4);
    w.rowsq_den = reinterpret_cast<float *>(take(sizeof(float) * n_tn * T));
    w.rowsq_num = reinterpret_cast<float *>(take(sizeof(float) * n_tn * T));
    w.den = reinterpret_cast<float *>(take(sizeof(float) * (size_t)T));
    w.state = reinterpret_cast<CettState *>(take(sizeof(CettState)));
    w.ytmp = take((size_t)T * d * 4);
    w.splitk = reinterpret_cast<float *>(ws + off);          // whatever room is left
    w.splitk_bytes = bytes - off;
    return w;
}

clada_status check_common(clada_ctx *ctx, const clada_layer *layer, const void *x, int32_t T)
{
    if (!ctx) return CLADA_ERR_NULL;
    clada_status st = clada_check_layer(ctx, layer);
    if (st != CLADA_OK) return st;
    if (!x) return clada_fail(ctx, CLADA_ERR_NULL, "x_val is NULL");
    if (T < 1 || T > (1 << 20)) return clada_fail(ctx, CLADA_ERR_SHAPE, "T=%d outside [1,2^20]", T);
    if (!aligned16(x)) return clada_fail(ctx, CLADA_ERR_ALIGN, "x_val must be 16-byte aligned");
    const size_t need = CLADA_WS_HEADER + clada_ws_cett(layer->d, layer->d_ff, T);
    if (ctx->ws_bytes < need)
        return clada_fail(ctx, CLADA_ERR_WORKSPACE, "workspace %zu < %zu bytes needed", ctx->ws_bytes, need);
    return CLADA_OK;
}

// Gate/up GEMM, dense down projection for the denominators, bracket / probe set-up.
clada_status begin(clada_ctx *ctx, const clada_layer *layer, const void *x, int T, const CettWs &w, int search,
                   float eps, bool large, hipStream_t stream)
{
    const int n_tn = clada_prefix_col_tiles(layer->d);
    CLADA_CHECK_HIP(ctx, clada_prefix_gateup(layer, x, T, w.part, w.pool, w.h, ctx->opt_prefix_tile, stream, ctx->num_cu));
    const float *rowsq_den = w.rowsq_den;
    if (layer->kind == CLADA_FFN_RELU) {
        // || sum_j a_j W_out[j,:] + b_out ||: through the stored output, which carries the bias
        // (the masked h is not there yet, and holds [T][d] where a bf16 layer is split without room for it: d_ff >= 2 d)
        CLADA_CHECK_HIP(ctx, clada_prefix_down(layer, w.h, T, w.ytmp, nullptr, w.room(layer->dtype == CLADA_BF16 ? w.hcut : w.ytmp), ctx->opt_prefix_tile,
                                               stream, ctx->num_cu));
        if (layer->dtype == CLADA_BF16)
            hipLaunchKernelGGL(k_cett_row_norm<2>, dim3((T + 3) / 4), dim3(256), 0, stream, w.ytmp, T, layer->d, w.den);
        else
            hipLaunchKernelGGL(k_cett_row_norm<4>, dim3((T + 3) / 4), dim3(256), 0, stream, w.ytmp, T, layer->d, w.den);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
        rowsq_den = nullptr;
    } else {
        CLADA_CHECK_HIP(ctx, clada_prefix_down(layer, w.h, T, nullptr, w.rowsq_den, w.room(w.ytmp), ctx->opt_prefix_tile, stream, ctx->num_cu));
    }
    if (large) return CLADA_OK;                             // (k_cett_sample does what is left)
    hipLaunchKernelGGL(k_cett_begin, dim3((T + 255) / 256), dim3(256), 0, stream, w.state, rowsq_den, n_tn, T,
                       w.den, search, eps);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}

// One probe: mask h at the state's eps, project, reduce, (bisect).
clada_status probe(clada_ctx *ctx, const clada_layer *layer, int T, const CettWs &w, float bound, int search,
                   float *cett_out, float *mean_out, hipStream_t stream)
{
    const int d = layer->d, F = layer->d_ff, n_tn = clada_prefix_col_tiles(d);
    const int Fp = (int)align_up((size_t)F, 64);
    const size_t groups = (size_t)T * (Fp / 8);
    const int grid = (int)((groups + 255) / 256 < 4096 ? (groups + 255) / 256 : 4096);
    if (layer->dtype == CLADA_BF16)
        hipLaunchKernelGGL(k_cett_mask<2>, dim3(grid), dim3(256), 0, stream, w.state, w.pool, w.h, w.hcut, T, F, Fp, 0);
    else
        hipLaunchKernelGGL(k_cett_mask<4>, dim3(grid), dim3(256), 0, stream, w.state, w.pool, w.h, w.hcut, T, F, Fp, 0);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    CLADA_CHECK_HIP(ctx, clada_prefix_down(layer, w.hcut, T, nullptr, w.rowsq_num, w.room(w.ytmp), ctx->opt_prefix_tile, stream, ctx->num_cu));
    hipLaunchKernelGGL(k_cett_update, dim3(1), dim3(1024), 0, stream, w.state, w.rowsq_num, n_tn, T, w.den, bound,
                       search, cett_out, mean_out);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}

// Columns per thread and workgroups per token of the probes inside the bracket: two workgroups where a row has at least two
// groups of 256 x 16 bytes (a row in one: 28 us a probe of 512 tokens x 4096 that looks through the pool).
struct BetweenShape { int nv, parts; };
BetweenShape between_shape(int d, int es)
{
    const int vecs = (d * es / 16 + 255) / 256;              // 1 .. 4
    return vecs == 1 ? BetweenShape{1, 1} : vecs == 2 ? BetweenShape{1, 2} : BetweenShape{2, 2};
}

// steps of the bisection a launch: as many thresholds as the row norms' buffers take
int between_levels(int d, int parts)
{
    const int room = clada_prefix_col_tiles(d) / parts;
    return room >= 7 ? 3 : room >= 3 ? 2 : 1;
}

template <int ES>
void launch_between(const CettWs &w, const clada_layer *layer, int T, int Fp, int launch, const int *list, int cap, const int *count,
                    float *const (&sums)[2], float bound, hipStream_t st)
{
    const int d = layer->d;
    const BetweenShape sh = between_shape(d, ES);
    const int levels = between_levels(d, sh.parts);
    auto kern = sh.nv == 1 ? (levels == 3 ? k_cett_between<ES, 1, 3> : levels == 2 ? k_cett_between<ES, 1, 2> : k_cett_between<ES, 1, 1>)
                           : (levels == 3 ? k_cett_between<ES, 2, 3> : levels == 2 ? k_cett_between<ES, 2, 2> : k_cett_between<ES, 2, 1>);
    auto take = levels == 3 ? k_cett_take<3> : levels == 2 ? k_cett_take<2> : k_cett_take<1>;
    float *sq[2] = {w.rowsq_num, w.rowsq_den};
    const bool taken = T > MEAN_IN_PLACE;
    if (taken && launch > 0)
        hipLaunchKernelGGL(take, dim3(1), dim3(1024), 0, st, w.state + (launch & 1), sq[launch & 1], sh.parts, T, w.den, bound);
    hipLaunchKernelGGL(kern, dim3(T, sh.parts), dim3(256), 0, st, w.state, launch, taken ? 1 : 0, w.pool, w.h, (const char *)layer->w_down,
                       list, cap, count, sums[0], sums[1],
                       sq[launch & 1], sq[(launch + 1) & 1], w.den, bound, T, layer->d_ff, Fp, d);
}

// Words that the large search keeps in the place of the partial aggregates (the curves' sum lies elsewhere: 100 tokens of 1024 x 3000
// fit now, 690 us as a plain bisection, 172 so), and whether they fit there.
bool large_fits(int T, int F)
{
    return (size_t)4 * clada_prefix_token_tiles(T) * F >= SAMPLES + CURVE_BINS + (size_t)T;
}

// The large search after begin().
clada_status search_large(clada_ctx *ctx, const clada_layer *layer, int T, const CettWs &w, float bound, hipStream_t stream)
{
    const int d = layer->d, F = layer->d_ff, n_tn = clada_prefix_col_tiles(d);
    const int Fp = (int)align_up((size_t)F, 64);
    const size_t groups = (size_t)T * (Fp / 8);
    const int grid = (int)((groups + 255) / 256 < 4096 ? (groups + 255) / 256 : 4096);
    // (the partial aggregates are not used here: large_fits)
    unsigned int *sample = reinterpret_cast<unsigned int *>(w.part);
    float *curve = reinterpret_cast<float *>(sample + SAMPLES);
    int *count = reinterpret_cast<int *>(curve + CURVE_BINS);
    // The table where it takes in what a probe's estimate leaves open; else the bracket is closed by dense probes and the rest of the
    // bisection measured a few thresholds a launch.
    const int window = T <= TABLE_TOKENS ? table_window(T, F) : 0;
    const bool table = window >= table_past(window) + table_below(window) && 2 * table_cap(T) < Fp;      // (and fits the masked h's part)
    const int curve_tokens = table ? (T < CURVE_TABLE ? T : CURVE_TABLE) : CURVE_TOKENS;
    unsigned long long *curves = reinterpret_cast<unsigned long long *>(w.hcut);      // (not masked yet)
    auto mask = [&](int may_skip) {
        if (layer->dtype == CLADA_BF16)
            hipLaunchKernelGGL(k_cett_mask<2>, dim3(grid), dim3(256), 0, stream, w.state, w.pool, w.h, w.hcut, T, F, Fp, may_skip);
        else
            hipLaunchKernelGGL(k_cett_mask<4>, dim3(grid), dim3(256), 0, stream, w.state, w.pool, w.h, w.hcut, T, F, Fp, may_skip);
        return hipGetLastError();
    };
    const bool den = layer->kind != CLADA_FFN_RELU;          // (the non-gated family's are there)
    hipLaunchKernelGGL(k_cett_sample, dim3(SAMPLE_WGS + (den ? (T + 255) / 256 : 0)), dim3(256), 0, stream, w.state, w.pool, (unsigned long long)T * F,
                       sample, bound, w.rowsq_den, n_tn, T, w.den, curves);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL((layer->dtype == CLADA_BF16 ? k_cett_curve<2> : k_cett_curve<4>), dim3(curve_tokens), dim3(1024), 0, stream, w.state, w.pool, w.h,
                       sample, T, F, Fp, curves, curve, bound, table ? table_below(window) : 0);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    // The cut sums at the bracket's lower end are the output of the last feasible probe.  With room for two buffers of them beside
    // the masked h (bf16: the upper half of h's part, which is sized for fp32) the probes alternate between them; else one more
    // projection forms them (68 us for 512 tokens of 4096 x 11008, against 2 a probe).
    const bool two = layer->dtype == CLADA_BF16 && Fp >= 2 * d;
    float *sums[2] = {reinterpret_cast<float *>(w.ytmp), reinterpret_cast<float *>(two ? w.h + (size_t)T * Fp * 2 : w.hcut)};
    // (with both buffers of sums taken, the half of the masked h's part that a bf16 one leaves is free)
    const DownRoom room = w.room(two ? w.hcut + (size_t)T * Fp * 2 : w.ytmp);
    const auto dense = [&](int stage) -> clada_status {
        CLADA_CHECK_HIP(ctx, mask(1));
        CLADA_CHECK_HIP(ctx, clada_prefix_down(layer, w.hcut, T, nullptr, w.rowsq_num, room, ctx->opt_prefix_tile, stream, ctx->num_cu,
                                               two || table ? sums[0] : nullptr, &w.state->skip, two ? sums[1] : nullptr, two ? &w.state->sel : nullptr));
        hipLaunchKernelGGL(k_cett_next, dim3(1), dim3(1024), 0, stream, w.state, w.rowsq_num, n_tn, T, w.den, bound, sample, curve,
                           table ? window : 0, two ? 1 : 0, stage);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
        return CLADA_OK;
    };
    // the masked h is not needed any more once the probes are done: its part takes the lists, behind the second buffer of cut sums if
    // that is there
    int *list = reinterpret_cast<int *>(w.hcut) + (two ? 0 : (size_t)T * d);
    const int list_cap = two ? Fp : Fp - d;
    const auto tail = [&](int launches) -> clada_status {
        hipLaunchKernelGGL(k_cett_list, dim3(T), dim3(1024), 0, stream, w.state, w.pool, F, list, list_cap, count);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
        for (int it = 0; it < launches; ++it) {
            if (layer->dtype == CLADA_BF16) launch_between<2>(w, layer, T, Fp, it, list, list_cap, count, sums, bound, stream);
            else launch_between<4>(w, layer, T, Fp, it, list, list_cap, count, sums, bound, stream);
            CLADA_CHECK_HIP(ctx, hipGetLastError());
        }
        return CLADA_OK;
    };
    clada_status st;
    if (table) {
        const int cap = table_cap(T), vecs = (d * (int)dtype_size(layer->dtype) / 16 + 255) / 256;      // 1 .. 4 groups of 256 x 16 bytes a row
        float *mag = reinterpret_cast<float *>(w.hcut), *cett = mag + (size_t)cap * T;        // (2 cap + 1 <= Fp words a token)
        const auto ladder = layer->dtype == CLADA_BF16 ? (vecs == 1 ? k_cett_ladder<2, 1, 256> : vecs == 2 ? k_cett_ladder<2, 1, 512> : k_cett_ladder<2, 2, 512>)
                                                       : (vecs == 1 ? k_cett_ladder<4, 1, 256> : vecs == 2 ? k_cett_ladder<4, 1, 512> : k_cett_ladder<4, 2, 512>);
        const int tpt = table_threads(T);
        const auto bisect = tpt == 1 ? k_cett_bisect<1> : tpt == 2 ? k_cett_bisect<2> : tpt == 4 ? k_cett_bisect<4> : k_cett_bisect<8>;
        for (int round = 0; round < 2; ++round) {
            for (int it = 0; it < TABLE_PROBES; ++it)
                if ((st = dense(round == 0 ? it : it < TABLE_PROBES - 1 ? 2 : 3)) != CLADA_OK) return st;
            if (!two) {                                      // the sums again, where a probe that failed came after the window's lower end
                CLADA_CHECK_HIP(ctx, mask(2));
                CLADA_CHECK_HIP(ctx, clada_prefix_down(layer, w.hcut, T, nullptr, nullptr, room, ctx->opt_prefix_tile, stream, ctx->num_cu, sums[0], &w.state->kept));
            }
            hipLaunchKernelGGL(ladder, dim3(T), dim3(vecs == 1 ? 256 : 512), 0, stream, w.state, w.pool, w.h, (const char *)layer->w_down, sums[0], sums[1],
                               w.den, T, F, Fp, d, cap, mag, cett, count);
            CLADA_CHECK_HIP(ctx, hipGetLastError());
            hipLaunchKernelGGL(bisect, dim3(1), dim3(1024), 0, stream, w.state, mag, cett, count, T, bound, sample, curve, window, round);
            CLADA_CHECK_HIP(ctx, hipGetLastError());
        }
        // What the tables left open (a great many equal magnitudes): an even number of launches, the last of which takes in the 31st
        // step.  (Most find nothing left: 32 of them / 12 at 700 tokens of 4096 x 11008 529 / 471 us, at 1024 of 1024 x 4096 292 / 218.)
        const int levels = between_levels(d, between_shape(d, (int)dtype_size(layer->dtype)).parts);
        return tail(levels == 3 ? 12 : levels == 2 ? 18 : 32);
    }
    for (int it = 0; it < DENSE_PROBES; ++it)
        if ((st = dense(it)) != CLADA_OK) return st;
    if (two) {
        hipLaunchKernelGGL(k_cett_base, dim3(1), dim3(64), 0, stream, w.state, 2);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
    } else {
        hipLaunchKernelGGL(k_cett_base, dim3(1), dim3(64), 0, stream, w.state, 0);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
        CLADA_CHECK_HIP(ctx, mask(0));
        CLADA_CHECK_HIP(ctx, clada_prefix_down(layer, w.hcut, T, nullptr, nullptr, room, ctx->opt_prefix_tile, stream, ctx->num_cu, sums[0]));
        hipLaunchKernelGGL(k_cett_base, dim3(1), dim3(64), 0, stream, w.state, 1);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
    }
    return tail(32);                                         // (the last one only takes in the 31st probe)
}

}  // namespace

size_t clada_ws_cett(int32_t d, int32_t d_ff, int32_t T)
{
    if (T <= 0) return 0;
    const size_t n_tm = (size_t)clada_prefix_token_tiles(T), n_tn = (size_t)clada_prefix_col_tiles(d);
    const size_t Fp = align_up((size_t)d_ff, 64);
    return align_up(sizeof(float) * 4 * n_tm * d_ff, 256) + align_up(sizeof(float) * (size_t)T * d_ff, 256) +
           2 * align_up((size_t)T * Fp * 4, 256) + 2 * align_up(sizeof(float) * n_tn * T, 256) +
           align_up(sizeof(float) * (size_t)T, 256) + 256 + align_up((size_t)T * d * 4, 256) +
           clada_ws_down_splitk(d, d_ff, T);
}
size_t clada_ws_cett_room(int32_t d, int32_t d_ff, int32_t T)
{
    if (T <= 0) return 0;
    return clada_ws_cett(d, d_ff, T) - clada_ws_down_splitk(d, d_ff, T) + clada_ws_down_room(d, d_ff, T);
}

extern "C" clada_status clada_cett_eval(clada_ctx *ctx, const clada_layer *layer, const void *x_val, int32_t T,
                                        float eps, float *cett_out, float *mean_out, void *hip_stream)
{
    clada_status st = check_common(ctx, layer, x_val, T);
    if (st != CLADA_OK) return st;
    if (!cett_out && !mean_out) return clada_fail(ctx, CLADA_ERR_NULL, "cett_out and mean_out are both NULL");
    if (eps != eps) return clada_fail(ctx, CLADA_ERR_VALUE, "eps is NaN");
    hipStream_t stream = (hipStream_t)hip_stream;
    const CettWs w = carve(ctx->ws + CLADA_WS_HEADER, ctx->ws_bytes - CLADA_WS_HEADER, layer->d, layer->d_ff, T);
    st = begin(ctx, layer, x_val, T, w, 0, eps, false, stream);
    if (st != CLADA_OK) return st;
    return probe(ctx, layer, T, w, 0.0f, 0, cett_out, mean_out, stream);
}

extern "C" clada_status clada_threshold_search_cett(clada_ctx *ctx, const clada_layer *layer, const void *x_val,
                                                    int32_t T, float bound, int32_t n_probes, float *tau_base_out,
                                                    float *mean_cett_out, void *hip_stream)
{
    if (!ctx) return CLADA_ERR_NULL;
    if (!tau_base_out) return clada_fail(ctx, CLADA_ERR_NULL, "tau_base_out is NULL");
    if (!(bound >= 0.0f && bound < 1.0f)) return clada_fail(ctx, CLADA_ERR_VALUE, "bound=%g outside [0,1)", (double)bound);
    if (n_probes < 1 || n_probes > 31) return clada_fail(ctx, CLADA_ERR_VALUE, "n_probes=%d outside [1,31]", n_probes);
    clada_status st = check_common(ctx, layer, x_val, T);
    if (st != CLADA_OK) return st;
    hipStream_t stream = (hipStream_t)hip_stream;
    const CettWs w = carve(ctx->ws + CLADA_WS_HEADER, ctx->ws_bytes - CLADA_WS_HEADER, layer->d, layer->d_ff, T);
    // The large search pays where 31 dense probes, four launches each, cost more than a pass over the tokens and a table: up to 1024
    // tokens from 64 tokens and 1024 neurons on, as far as its words fit (us, plain / large: 613 / 180 for 197 tokens of 512 x 1185,
    // 571 / 557 for 78 of 512 x 1024, where they do not; 1096 / 189 for 72 of 1024 x 1398; fp32 1562 / 305 for 71 of 768 x 1746; 60 such
    // searches ended at the same threshold either way: a bracket of a few hundred magnitudes is several times as wide as the stretch where single
    // neurons turn the mean).  Beyond, a probe inside the bracket is a workgroup per token, and the bracket is only trusted from 2^18 magnitudes
    // on (ms, 1.43 / 0.33 for 64 tokens of 4096 x 11008, 0.86 / 0.27 for 256 of 512 x 1999), 2^20 below 1024 neurons; fewer probes
    // than the full 31 end somewhere on the way, which only the plain bisection passes through.  A bf16 projection of fewer than 2048
    // neurons costs less once the tokens fill the chip (ms, large / plain: 6.6 / 3.9 and 8.2 / 6.4 at 65536 tokens of 64 and 512 x 512,
    // 7.9 / 7.1 of 256 x 1024, 1.9 / 1.7 at 16384 of 256 x 512; 0.79 / 1.04 at 4096 of 256 x 512, 8.2 / 11.1 at 65536 of 64 x 2048); an
    // fp32 one never does (2.1 / 2.7 at 16384 of 64 x 512).
    const int F = layer->d_ff;
    const bool large = n_probes == 31 && bound > 0.0f && T >= 64 && (size_t)T * F >= (F < 1024 ? 1u << 20 : T > TABLE_TOKENS ? 1u << 18 : 0u) && F >= layer->d &&
                       F >= 512 && large_fits(T, F) && (layer->dtype == CLADA_F32 || T <= 4096 || F >= 2048);
    st = begin(ctx, layer, x_val, T, w, 1, 0.0f, large, stream);
    if (st != CLADA_OK) return st;
    if (large) {
        st = search_large(ctx, layer, T, w, bound, stream);
        if (st != CLADA_OK) return st;
    }
    for (int it = 0; it < n_probes && !large; ++it) {
        st = probe(ctx, layer, T, w, bound, 1, nullptr, nullptr, stream);
        if (st != CLADA_OK) return st;
    }
    hipLaunchKernelGGL(k_cett_finish, dim3(1), dim3(64), 0, stream, w.state, tau_base_out, mean_cett_out);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}
