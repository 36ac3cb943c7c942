// Prefill statistics (section 3.2.1, neuron-activation equation; algorithm
// "CLADA Inference", prefill phase): dense SwiGLU FFN over the prefix on the
// matrix cores with the per-neuron aggregates fused into the GEMM epilogue.
//
//   kernel 1 (gate+up): C_g = X W_gate^T and C_u = X W_up^T share the X tile;
//     both operands are K-contiguous (X [T][d], W [F][d]) so fragments come
//     straight from LDS.  Epilogue on the accumulators: a = SiLU(C_g),
//     h = a*C_u, per-neuron partial sums over the tile's tokens (|a|, a^2, h^2,
//     max|a|), the |a| pool, and h stored in the layer dtype for kernel 2.
//   kernel 2 (down): Y = H W_down.  W_down lies neuron-major, k by columns: the bf16 kernels keep it so in LDS and read the
//     fragments transposed, the fp32 kernel transposes it on its way into LDS.  Short prefixes split d_ff.
//   kernel 3: the parts of a split added up, and a fixed-order reduction of the per-token-tile partials,
//     A_j = sqrt(sum_t h_tj^2) * ||W_down[j,:]||_2.
// bf16 layers run on the pipelined tiles of prefix_tiles.h: the gate/up product for rows of whole k-tiles (d % 64 == 0), the down
// projection for d % 256 == 0.  The rest, and fp32 layers, run on plain tiles (gate/up 128 or 64 tokens x 64 neurons, down 128 x 128) of
// four wavefronts, MFMA 32x32x16 (bf16) or 32x32x2 (fp32), fp32 accumulation.  Block ids are remapped so that the eight XCDs each
// walk their own range of tiles (operand slices stay in that XCD's L2).
#include <math.h>

#include "prefix_tiles.h"

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int BM = 128, BN = 128;
// k-tile depth: 64 for bf16 (half as many barriers per flop), 32 for fp32 (LDS budget)
template <int ES> constexpr int BKV = (ES == 2) ? 64 : 32;

template <int ES> struct Tile {
    static constexpr int ROW = BKV<ES> * ES + 16;       // padded LDS row stride, bytes
    static constexpr int CHUNKS = BKV<ES> * ES / 16;    // 16-byte chunks per tile row
    static constexpr int PER_THREAD = BM * CHUNKS / 256; // chunks each thread moves per tile
};

// One k-tile of MFMAs for a wave tile of 32 MB x 32 NK.  sa / sb point at the wave's first
// row of the A / B tile in LDS.
template <int ES, int NB, int MB, int NK>
__device__ __forceinline__ void mma_tile(const char *sa, const char *const (&sb)[NB], f32x16 (&acc)[NB][MB][NK], int lane)
{
    constexpr int ROW = Tile<ES>::ROW;
    const int r = lane & 31, q = lane >> 5;
    if (ES == 2) {
#pragma unroll
        for (int ks = 0; ks < BKV<ES> / 16; ++ks) {
            bf16x8 a[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                a[mb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(sa + (mb * 32 + r) * ROW + (ks * 16 + q * 8) * 2));
#pragma unroll
            for (int w = 0; w < NB; ++w)
#pragma unroll
                for (int nb = 0; nb < NK; ++nb) {
                    const bf16x8 bv = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(sb[w] + (nb * 32 + r) * ROW + (ks * 16 + q * 8) * 2));
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[w][mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mb], bv, acc[w][mb][nb], 0, 0, 0);
                }
        }
    } else {
#pragma unroll
        for (int ks = 0; ks < BKV<ES> / 2; ++ks) {
            float a[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                a[mb] = *reinterpret_cast<const float *>(sa + (mb * 32 + r) * ROW + (ks * 2 + q) * 4);
#pragma unroll
            for (int w = 0; w < NB; ++w)
#pragma unroll
                for (int nb = 0; nb < NK; ++nb) {
                    const float bv = *reinterpret_cast<const float *>(sb[w] + (nb * 32 + r) * ROW + (ks * 2 + q) * 4);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[w][mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mb], bv, acc[w][mb][nb], 0, 0, 0);
                }
        }
    }
}

// SiLU of the prefill epilogues: hardware exp2 and reciprocal (a few ulp), a third of the instructions
// of the division form; +-inf and NaN behave as in g / (1 + exp(-g)).
__device__ __forceinline__ float silu_prefill(float g)
{
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * g));
}

// Tanh-form GELU the same way: g * sigmoid(2 sqrt(2/pi) (g + 0.044715 g^3)).
__device__ __forceinline__ float gelu_prefill(float g)
{
    const float u2 = 1.5957691216057308f * fmaf(0.044715f * g, g * g, g);
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * u2));
}

// Row of accumulator register r of a 32x32 MFMA block held by `lane`.
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// XCD-aware remap: consecutive block ids alternate over the 8 XCDs; give each XCD a
// contiguous run of tiles, token tile fastest.
__device__ __forceinline__ int remap_block(int id, int total)
{
    const int per = (total + 7) / 8;
    return (id & 7) * per + (id >> 3);
}

struct GateUpParams {
    const char *x, *wg, *wu;
    int T, d, F, n_tm, n_tn;
    float *part;        // [n_tm][4][F]  partial aggregates (sum|a|, sum a^2, max|a|, sum h^2)
    float *pool;        // [T][F] or nullptr
    char *hbuf;         // [T][Fp] layer dtype (Fp = F rounded up to BK, zero past F) or nullptr
    int Fp;             // F rounded up to a multiple of 64
    const float *b_in;  // non-gated family: input bias [F] or nullptr
    int relu;           // non-gated family: a = max(0, C_g + b_in), h = a (wu then aliases wg and C_u is ignored)
    int gelu;           // gated family: sigma = tanh-form GELU instead of SiLU
    // Workgroups behind the GEMM's (bf16 kernels): they form || W_down[j,:] ||^2 on the compute units that the tiles
    // leave idle; k_prefix_reduce, which would read W_down for it, then finds it in wnorm2.
    const char *wd;
    float *wnorm2;                 // [norm_rows] or nullptr
    int gemm_blocks, norm_blocks, norm_rows;
};

// Epilogue of the gate/up GEMM on the accumulators (shared by the fp32 and bf16 kernels):
// a = SiLU(C_g), h = a*C_u, per-neuron partial sums over the tile's tokens, |a| pool, h store.
template <int ES, int MB, int NK, int NEU>
__device__ __forceinline__ void gateup_epilogue(const f32x16 (&acc)[2][MB][NK], const GateUpParams &p, int tm, int tn,
                                                int wm, int wn, int lane, int tid, float (&s_stat)[2][4][NEU])
{
    // ------------------------------------------------------------------ epilogue
    const int n = lane & 31;
#pragma unroll
    for (int nb = 0; nb < NK; ++nb) {
        const int jl = wn * 32 * NK + nb * 32 + n;          // neuron inside the tile
        const int j = tn * NEU + jl;
        float s_abs = 0.f, s_sq = 0.f, mx = 0.f, s_h2 = 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = (tm * 2 + wm) * 32 * MB + mb * 32 + acc_row(r, lane);
                float a, h;
                if (p.relu) {
                    const float g = acc[0][mb][nb][r] + ((p.b_in && j < p.F) ? p.b_in[j] : 0.0f);
                    a = g > 0.0f ? g : (g != g ? g : 0.0f);
                    h = a;
                } else {
                    a = p.gelu ? gelu_prefill(acc[0][mb][nb][r]) : silu_prefill(acc[0][mb][nb][r]);
                    h = a * acc[1][mb][nb][r];
                }
                if (t < p.T && j < p.F) {
                    const float aa = fabsf(a);
                    s_abs += aa;
                    s_sq = fmaf(a, a, s_sq);
                    mx = (aa > mx || aa != aa) ? aa : mx;
                    s_h2 = fmaf(h, h, s_h2);
                    if (p.pool) p.pool[(size_t)t * p.F + j] = aa;
                }
                if (p.hbuf && t < p.T && j < p.Fp) {
                    const float hv = j < p.F ? h : 0.0f;
                    if (ES == 4) reinterpret_cast<float *>(p.hbuf)[(size_t)t * p.Fp + j] = hv;
                    else reinterpret_cast<unsigned short *>(p.hbuf)[(size_t)t * p.Fp + j] = (unsigned short)f32_to_bf16_bits(hv);
                }
            }
        // lanes l and l^32 hold the same neuron
        s_abs += __shfl_xor(s_abs, 32);
        s_sq += __shfl_xor(s_sq, 32);
        s_h2 += __shfl_xor(s_h2, 32);
        const float mo = __shfl_xor(mx, 32);
        mx = (mo > mx || mo != mo) ? mo : mx;
        if (lane < 32) {
            s_stat[wm][0][jl] = s_abs;
            s_stat[wm][1][jl] = s_sq;
            s_stat[wm][2][jl] = mx;
            s_stat[wm][3][jl] = s_h2;
        }
    }
    __syncthreads();
    if (tid < NEU) {
        const int j = tn * NEU + tid;
        if (j < p.F) {
            float *dst = p.part + (size_t)tm * 4 * p.F + j;
            dst[0] = s_stat[0][0][tid] + s_stat[1][0][tid];
            dst[(size_t)p.F] = s_stat[0][1][tid] + s_stat[1][1][tid];
            const float m0 = s_stat[0][2][tid], m1 = s_stat[1][2][tid];
            dst[2 * (size_t)p.F] = (m1 > m0 || m1 != m1) ? m1 : m0;
            dst[3 * (size_t)p.F] = s_stat[0][3][tid] + s_stat[1][3][tid];
        }
    }
}

// TT tokens x 64 neurons a workgroup, four waves of (TT / 2) x 32: two workgroups fit a compute unit (148 registers), so that one's
// products cover the other's staging, and a short prefix still has tiles for the chip.  Before, 128 x 128 with 280 registers (fp32, us,
// without y): 4096 x 11008 at 512 tokens 1217 / 927, at 128 618 / 359, 2048 x 6000 at 200 299 / 167; 64-token tiles for up to 64 tokens,
// 4096 x 9000 at 32: 594 / 225.
template <int ES, int TT>
__global__ void __launch_bounds__(256)
k_prefix_gateup(const GateUpParams p)
{
    constexpr int NEU = 64, ROW = Tile<ES>::ROW, CH = Tile<ES>::CHUNKS, PT = NEU * CH / 256, PX = TT * CH / 256;
    constexpr int MB = TT / 64, NK = 1;
    static_assert(PX >= PT, "the token tile is the larger one");
    __shared__ __align__(16) char s_a[TT * ROW];
    __shared__ __align__(16) char s_g[NEU * ROW];
    __shared__ __align__(16) char s_u[NEU * ROW];
    __shared__ float s_stat[2][4][NEU];

    const int total = p.n_tm * p.n_tn;
    const int tile = remap_block(blockIdx.x, total);
    if (tile >= total) return;
    const int tm = tile % p.n_tm, tn = tile / p.n_tm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const size_t rowbytes = (size_t)p.d * ES;

    f32x16 acc[2][MB][NK];
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NK; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[w][mb][nb][r] = 0.0f;

    u32x4 ra[PX], rg[PT], ru[PT];
    auto load_tile = [&](int kt) {
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            const int c = tid + i * 256, row = c / CH, ch = c % CH;
            const int kbyte = kt * BKV<ES> * ES + ch * 16;
            const bool kin = (size_t)kbyte < rowbytes;
            const int t = tm * TT + row, j = tn * NEU + row;
            u32x4 z = {0u, 0u, 0u, 0u};
            ra[i] = (kin && t < p.T) ? *reinterpret_cast<const u32x4 *>(p.x + (size_t)t * rowbytes + kbyte) : z;
            if (i < PT) rg[i < PT ? i : 0] = (kin && j < p.F) ? *reinterpret_cast<const u32x4 *>(p.wg + (size_t)j * rowbytes + kbyte) : z;
            if (i < PT) ru[i < PT ? i : 0] = (kin && j < p.F) ? *reinterpret_cast<const u32x4 *>(p.wu + (size_t)j * rowbytes + kbyte) : z;
        }
    };
    const int nk = (p.d + BKV<ES> - 1) / BKV<ES>;
    load_tile(0);
    for (int kt = 0; kt < nk; ++kt) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            const int c = tid + i * 256, row = c / CH, ch = c % CH;
            *reinterpret_cast<u32x4 *>(s_a + row * ROW + ch * 16) = ra[i];
            if (i < PT) *reinterpret_cast<u32x4 *>(s_g + row * ROW + ch * 16) = rg[i < PT ? i : 0];
            if (i < PT) *reinterpret_cast<u32x4 *>(s_u + row * ROW + ch * 16) = ru[i < PT ? i : 0];
        }
        __syncthreads();
        if (kt + 1 < nk) load_tile(kt + 1);
        const char *const sb[2] = {s_g + wn * 32 * NK * ROW, s_u + wn * 32 * NK * ROW};
        mma_tile<ES, 2, MB, NK>(s_a + wm * 32 * MB * ROW, sb, acc, lane);
    }

    gateup_epilogue<ES, MB, NK, NEU>(acc, p, tm, tn, wm, wn, lane, tid, s_stat);
}

// Sum of squares of a row of W_down, by one wave: 16-byte chunks, lane l takes chunks l, l + 64, .. (eight loads in flight).
template <int ES>
__device__ __forceinline__ float row_norm2(const char *row, int d, int lane)
{
    constexpr int VEC = 16 / ES;
    const int nchunk = d * ES / 16;
    float wn2 = 0.0f;
    for (int c0 = lane; c0 < nchunk; c0 += 8 * 64) {
        u32x4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = c0 + 64 * i < nchunk ? *reinterpret_cast<const u32x4 *>(row + (size_t)(c0 + 64 * i) * 16)
                                        : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float w[VEC];
            unpack_row16(v[i], w);
#pragma unroll
            for (int e = 0; e < VEC; ++e) wn2 = fmaf(w[e], w[e], wn2);
        }
    }
    return wave_sum(wn2);
}

// What a workgroup behind the GEMM's does: the norms of every norm_blocks-th group of eight rows.
__device__ __forceinline__ void spare_norms(const GateUpParams &p)
{
    const int lane = threadIdx.x & 63;
    for (int j = 8 * ((int)blockIdx.x - p.gemm_blocks) + (threadIdx.x >> 6); j < p.norm_rows; j += 8 * p.norm_blocks) {
        const float v = row_norm2<2>(p.wd + (size_t)j * p.d * 2, p.d, lane);
        if (lane == 0) p.wnorm2[j] = v;
    }
}

// ACT: 0 SiLU, 1 tanh-form GELU, 2 ReLU (non-gated family: h = a)
template <int ACT>
__device__ __forceinline__ void prefill_act(float g, float u, float &a, float &h)
{
    if (ACT == 2) {
        a = g > 0.0f ? g : (g != g ? g : 0.0f);
        h = a;
    } else {
        a = ACT == 1 ? gelu_prefill(g) : silu_prefill(g);
        h = a * u;
    }
}

__device__ __forceinline__ unsigned short bf16_of(float v) { return __builtin_bit_cast(unsigned short, (__bf16)v); }

// Epilogue of a tile of the pipelined kernel: activation, per-neuron sums over the tile's tokens, |a| pool, h.  A lane holds tokens
// 16 i + 4 q + r of its wave's 64 and neuron 16 b + n of its 16 NBN; gate and up of a neuron are the column blocks 2 b and 2 b + 1
// (the W tile alternates 16 rows of each).  FULL: the tile lies inside [T] x [F].  The waves of a column of the tile add their sums
// through LDS in fixed order: one partial per tile.
template <class S, bool SINGLE, bool FULL, int ACT>
__device__ __forceinline__ void gateup_tile_epilogue(const f32x4 (&acc)[4][2 * S::NB], const GateUpParams &p, int tm, int tn, int wm, int wn,
                                                     unsigned int scratch)
{
    constexpr int NBN = SINGLE ? 2 * S::NB : S::NB, NEUR = 16 * NBN * S::WN;
    const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
    const size_t F1 = (size_t)p.F, Fp1 = (size_t)p.Fp;
    const int t0 = tm * S::TM + wm * 64;                    // first token and neuron of the wave (uniform)
    const int j0 = tn * NEUR + wn * 16 * NBN;
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
        const int j = j0 + 16 * b + n;
        const bool jok = FULL || j < p.F;
        const float bj = (ACT == 2 && p.b_in && jok) ? p.b_in[j] : 0.0f;
        const unsigned int vp = (unsigned int)(4 * q * p.F + 16 * b + n) * 4u, vh = (unsigned int)(4 * q * p.Fp + 16 * b + n) * 2u;
        float s_abs = 0.0f, s_sq = 0.0f, mx = 0.0f, s_h2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float aa[4], hh[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float a;
                prefill_act<ACT>(acc[i][SINGLE ? b : 2 * b][r] + bj, acc[i][SINGLE ? b : 2 * b + 1][r], a, hh[r]);
                aa[r] = fabsf(a);
                if (FULL || (t0 + 16 * i + 4 * q + r < p.T && jok)) {
                    s_abs += aa[r];
                    s_sq = fmaf(a, a, s_sq);
                    mx = __builtin_elementwise_maximum(mx, aa[r]);       // a NaN sticks
                    s_h2 = fmaf(hh[r], hh[r], s_h2);
                }
            }
            if (p.pool) {
                char *dst = reinterpret_cast<char *>(p.pool + (size_t)(t0 + 16 * i) * F1 + j0);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (FULL || (t0 + 16 * i + 4 * q + r < p.T && jok)) *reinterpret_cast<float *>(dst + r * F1 * 4 + vp) = aa[r];
            }
            if (p.hbuf) {
                char *dst = p.hbuf + ((size_t)(t0 + 16 * i) * Fp1 + j0) * 2;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (FULL || (t0 + 16 * i + 4 * q + r < p.T && j < p.Fp))
                        *reinterpret_cast<unsigned short *>(dst + r * Fp1 * 2 + vh) = bf16_of(jok ? hh[r] : 0.0f);
            }
        }
        s_abs += __shfl_xor(s_abs, 16); s_abs += __shfl_xor(s_abs, 32);
        s_sq += __shfl_xor(s_sq, 16);   s_sq += __shfl_xor(s_sq, 32);
        s_h2 += __shfl_xor(s_h2, 16);   s_h2 += __shfl_xor(s_h2, 32);
        mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 16));
        mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32));
        const unsigned int at = scratch + (unsigned int)(wm * NEUR + wn * 16 * NBN + 16 * b + n) * 4u;
        const float v = q == 0 ? s_abs : q == 1 ? s_sq : q == 2 ? mx : s_h2;     // lane group q keeps sum q
        scratch_put(at + (unsigned int)(q * S::WM * NEUR) * 4u, v);
    }
    // The down projection reads h in whole k-tiles, up to column Fp, and counts on zeros there.  Tiles of a multiple of 64 neurons reach
    // that far; others may end up to 32 columns short of it (d_ff mod 192 from 65 to 96 with 96 neurons).
    if constexpr (NEUR % 64 != 0) {
        static_assert(NEUR % 8 == 0, "whole 16-byte chunks behind the tile");
        const int c0 = (tn + 1) * NEUR;
        if (p.hbuf && c0 >= p.F && c0 < p.Fp) {
            const int chunks = (p.Fp - c0) / 8, rows = min(p.T - tm * S::TM, S::TM);
            for (int v = threadIdx.x; v < rows * chunks; v += 512) {
                const int r = v / chunks, c = v - r * chunks;
                *reinterpret_cast<u32x4 *>(p.hbuf + ((size_t)(tm * S::TM + r) * Fp1 + c0 + 8 * c) * 2) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    }
    lds_barrier();
    for (int v = threadIdx.x; v < 4 * NEUR; v += 512) {
        const int s = v / NEUR, jl = v % NEUR, j = tn * NEUR + jl;
        const unsigned int at = scratch + (unsigned int)(s * S::WM * NEUR + jl) * 4u;
        float sum = scratch_get(at);
#pragma unroll
        for (int w = 1; w < S::WM; ++w) {
            const float o = scratch_get(at + (unsigned int)(w * NEUR) * 4u);
            sum = s == 2 ? __builtin_elementwise_maximum(sum, o) : sum + o;
        }
        if (j < p.F) p.part[((size_t)tm * 4 + s) * F1 + j] = sum;
    }
}

// Gate / up product of the bf16 layers with whole 128-byte rows (d % 64 == 0).  SINGLE: the non-gated family's one matrix.
// Tile: S::TM tokens x S::TN rows of W -- half of them gate, half up rows of the same neurons, 16 and 16 in turn.
template <class S, bool SINGLE>
__global__ void __launch_bounds__(512, 2)
k_prefix_gateup_tiles(const GateUpParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ __align__(16) char s_w[S::LDS];
    constexpr int NEUR = SINGLE ? S::TN : S::TN / 2;
    if ((int)blockIdx.x >= p.gemm_blocks) {
        spare_norms(p);
        return;
    }
    struct Tile {
        struct Id { int tm, tn; };
        int blocks, n_tm, n_tn;
        __device__ __forceinline__ bool operator()(int it, Id &id) const
        {
            const int o = tile_order(it, blocks, n_tm * n_tn);
            if (o < 0) return false;
            tile_coords(o, n_tm, n_tn, id.tm, id.tn);
            return true;
        }
    };
    const Tile tile{p.gemm_blocks, (p.T + S::TM - 1) / S::TM, (p.F + NEUR - 1) / NEUR};
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t rowbytes = (size_t)p.d * 2;
    // transfer i of a wave: rows 8 wave + 64 i .. of the W tile, 16-row block (wave >> 1) + 4 i: odd blocks are up rows
    const char *w = !SINGLE && ((wave >> 1) & 1) ? p.wu : p.wg;
    int vw[S::PW];
#pragma unroll
    for (int i = 0; i < S::PW; ++i) {
        const int row = SINGLE ? 8 * wave + 64 * i + (lane >> 3) : 16 * ((wave >> 2) + 2 * i) + 8 * (wave & 1) + (lane >> 3);
        vw[i] = row * (int)rowbytes + ((lane & 7) ^ (lane >> 3)) * 16;
    }
    auto src = [&](const typename Tile::Id &id) {
        TileSrc s;
        s.x = p.x + (size_t)id.tm * S::TM * rowbytes;
        s.x_bytes = (unsigned int)(min(p.T - id.tm * S::TM, S::TM) * (int)rowbytes);
        s.w = w + (size_t)id.tn * NEUR * rowbytes;
        s.w_bytes = (unsigned int)(min(p.F - id.tn * NEUR, NEUR) * (int)rowbytes);
        s.w_rows = s.w_pitch = s.w_col = 0;
        s.nk = p.d / 64;
        return s;
    };
    auto epi = [&](const f32x4 (&acc)[4][2 * S::NB], const typename Tile::Id &id, unsigned int scratch, int wm, int wn) {
        const bool full = (id.tm + 1) * S::TM <= p.T && (id.tn + 1) * NEUR <= p.F;
        if constexpr (SINGLE) {
            if (full) gateup_tile_epilogue<S, true, true, 2>(acc, p, id.tm, id.tn, wm, wn, scratch);
            else      gateup_tile_epilogue<S, true, false, 2>(acc, p, id.tm, id.tn, wm, wn, scratch);
        } else if (p.gelu) {
            if (full) gateup_tile_epilogue<S, false, true, 1>(acc, p, id.tm, id.tn, wm, wn, scratch);
            else      gateup_tile_epilogue<S, false, false, 1>(acc, p, id.tm, id.tn, wm, wn, scratch);
        } else {
            if (full) gateup_tile_epilogue<S, false, true, 0>(acc, p, id.tm, id.tn, wm, wn, scratch);
            else      gateup_tile_epilogue<S, false, false, 0>(acc, p, id.tm, id.tn, wm, wn, scratch);
        }
    };
    tile_products<S>(s_w, (int)rowbytes, vw, tile, src, epi);
#endif
}

struct DownParams {
    const char *h, *wd;
    char *y;                       // [T][d] layer dtype, or nullptr
    const float *bias;             // output bias [d] of the non-gated family, or nullptr
    float *rowsq;                  // [n_tn][T] per column-tile sums of squares of the fp32 rows, or nullptr
    int T, d, F, Fp, n_tm, n_tn;   // Fp = F rounded up to a multiple of BK (row stride of h)
    float *part_out;               // split: fp32 partial outputs [parts][T][d] instead of y / rowsq
    int S;                         // number of k ranges the neurons are split into (1 = no split)
    // SOME kernels: ranges ks0 .. ks0 + parts of them, the first one added to what lies in part_out (add); or all of them one after the
    // other by the same workgroups, added up in registers (chain = S, parts = 1; otherwise chain = 1)
    int ks0, parts, add, chain;
    float *y32;                    // [T][d] the fp32 rows without a bias, or nullptr
    float *y32_alt;                // they go there instead when *alt is 0 (alt: device flag or nullptr)
    const int *alt;
    const int *skip;               // device flag: nothing to do when set (a probe that is not needed), or nullptr
};

// Row sums of squares of a 128 x 128 output tile held in the accumulators of four waves (2 x 2
// blocks of 32 x 32 each): 32-lane butterfly per row, then the two column halves in fixed order.
__device__ __forceinline__ void down_rowsq(const f32x16 (&acc)[2][2], const DownParams &p, int tm, int tn, int wm,
                                           int wn, int lane, int tid, float (&s_rs)[2][BM])
{
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float v = fmaf(acc[mb][0][r], acc[mb][0][r], acc[mb][1][r] * acc[mb][1][r]);
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 8);
            v += __shfl_xor(v, 4);
            v += __shfl_xor(v, 2);
            v += __shfl_xor(v, 1);
            if ((lane & 31) == 0) s_rs[wn][wm * 64 + mb * 32 + acc_row(r, lane)] = v;
        }
    __syncthreads();
    if (tid < BM) {
        const int t = tm * BM + tid;
        if (t < p.T) p.rowsq[(size_t)tn * p.T + t] = s_rs[0][tid] + s_rs[1][tid];
    }
}

// Where the fp32 rows go.
__device__ __forceinline__ float *rows32_of(const DownParams &p) { return p.alt && *p.alt == 0 ? p.y32_alt : p.y32; }

// f(word, mb, nb, r) of the fp32 rows of a 128 x 128 tile.
template <class Fn>
__device__ __forceinline__ void down_rows32(const DownParams &p, float *rows, int tm, int tn, int wm, int wn, int lane, Fn f)
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int col = tn * BN + wn * 64 + nb * 32 + (lane & 31);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = tm * BM + wm * 64 + mb * 32 + acc_row(r, lane);
                if (t < p.T && col < p.d) f(rows[(size_t)t * p.d + col], mb, nb, r);
            }
    }
}
// Those rows, without a bias.
__device__ __forceinline__ void down_store32(const f32x16 (&acc)[2][2], const DownParams &p, float *rows, int tm, int tn, int wm, int wn, int lane)
{
    down_rows32(p, rows, tm, tn, wm, wn, lane, [&](float &at, int mb, int nb, int r) { at = acc[mb][nb][r]; });
}

// PROBE (the three down kernels): the error-bounded search's form, with y32 and skip.  The others are built without: the
// extra store loop alone raised k_prefix_down_bf16's registers (330 -> 401 us at 2368 x 4096 x 9728).
// SOME: some parts of a split at a time, for a workspace that does not hold all of them; also with skip.
// fp32.
template <bool PROBE, bool SOME = false>
__global__ void __launch_bounds__(256)
k_prefix_down(const DownParams p)
{
    if (PROBE && p.skip && *p.skip) return;
    constexpr int ES = 4, ROW = Tile<ES>::ROW, CH = Tile<ES>::CHUNKS, PT = Tile<ES>::PER_THREAD;
    __shared__ __align__(16) char s_a[BM * ROW];
    __shared__ __align__(16) char s_b[BN * ROW];      // [n][k]: W_down tile transposed
    __shared__ float s_rs[2][BM];

    const int total = p.n_tm * p.n_tn * (SOME ? p.parts : p.S);
    const int o = remap_block(blockIdx.x, total);
    if (o >= total) return;
    const int slot = o / (p.n_tm * p.n_tn), tile = o - slot * p.n_tm * p.n_tn;
    const int tm = tile % p.n_tm, tn = tile / p.n_tm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const size_t hrow = (size_t)p.Fp * ES, wrow = (size_t)p.d * ES;

    f32x16 acc[1][2][2];
    auto clear = [](f32x16 (&a)[2][2]) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) a[mb][nb][r] = 0.0f;
    };

    // B tile in global memory: BK rows (neurons) x BN columns -> BK * BN*ES/16 chunks
    constexpr int BCH = BN * ES / 16;                  // chunks per neuron row of the tile
    constexpr int BPT = BKV<ES> * BCH / 256;
    u32x4 ra[PT], rb[BPT];
    auto load_tile = [&](int kt) {
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int c = tid + i * 256, row = c / CH, ch = c % CH;
            const size_t kbyte = (size_t)kt * BKV<ES> * ES + ch * 16;
            const int t = tm * BM + row;
            u32x4 z = {0u, 0u, 0u, 0u};
            // rows of h are padded to a multiple of BK elements, zero-filled past F
            ra[i] = (t < p.T && kbyte < hrow) ? *reinterpret_cast<const u32x4 *>(p.h + (size_t)t * hrow + kbyte) : z;
        }
#pragma unroll
        for (int i = 0; i < BPT; ++i) {
            const int c = tid + i * 256, k = c / BCH, ch = c % BCH;
            const int j = kt * BKV<ES> + k;
            const size_t nbyte = (size_t)tn * BN * ES + ch * 16;
            u32x4 z = {0u, 0u, 0u, 0u};
            rb[i] = (j < p.F && nbyte < wrow) ? *reinterpret_cast<const u32x4 *>(p.wd + (size_t)j * wrow + nbyte) : z;
        }
    };
    // a part's k-tiles (parts of a split hold at least 256 neurons each)
    const int nk_all = (p.F + BKV<ES> - 1) / BKV<ES>;
    auto product = [&](int ks) {
        const int kt0 = (int)((long long)ks * nk_all / p.S), nk = (int)((long long)(ks + 1) * nk_all / p.S);
        clear(acc[0]);
        load_tile(kt0);
        for (int kt = kt0; kt < nk; ++kt) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < PT; ++i) {
                const int c = tid + i * 256, row = c / CH, ch = c % CH;
                *reinterpret_cast<u32x4 *>(s_a + row * ROW + ch * 16) = ra[i];
            }
#pragma unroll
            for (int i = 0; i < BPT; ++i) {
                const int c = tid + i * 256, k = c / BCH, ch = c % BCH;
#pragma unroll
                for (int e = 0; e < 4; ++e) *reinterpret_cast<unsigned int *>(s_b + (ch * 4 + e) * ROW + k * 4) = rb[i][e];
            }
            __syncthreads();
            if (kt + 1 < nk) load_tile(kt + 1);
            const char *const sb[1] = {s_b + wn * 64 * ROW};
            mma_tile<ES, 1, 2, 2>(s_a + wm * 64 * ROW, sb, acc, lane);
        }
    };
    product(slot + (SOME ? p.ks0 : 0));
    if constexpr (SOME) {
        f32x16 sum[2][2];
        clear(sum);
        for (int c = 1;; ++c) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) sum[mb][nb] += acc[0][mb][nb];
            if (c >= p.chain) break;
            product(c);
        }
        float *rows = p.part_out + (size_t)slot * p.T * p.d;
        if (p.add && slot == 0)                             // (all loads before the first store)
            down_rows32(p, rows, tm, tn, wm, wn, lane, [&](float &at, int mb, int nb, int r) { sum[mb][nb][r] += at; });
        down_store32(sum, p, rows, tm, tn, wm, wn, lane);
        return;
    }
    if (p.part_out) {                                       // split: fp32 partial sums, added up by k_prefix_down_combine
        down_store32(acc[0], p, p.part_out + (size_t)slot * p.T * p.d, tm, tn, wm, wn, lane);
        return;
    }
    if (p.rowsq) down_rowsq(acc[0], p, tm, tn, wm, wn, lane, tid, s_rs);
    if (PROBE && p.y32) down_store32(acc[0], p, rows32_of(p), tm, tn, wm, wn, lane);
    if (!p.y) return;
    const int n = lane & 31;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int col = tn * BN + wn * 64 + nb * 32 + n;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = tm * BM + wm * 64 + mb * 32 + acc_row(r, lane);
                if (t < p.T && col < p.d)
                    reinterpret_cast<float *>(p.y)[(size_t)t * p.d + col] = acc[0][mb][nb][r] + (p.bias ? p.bias[col] : 0.0f);
            }
    }
}

// bf16 down projection Y = H W_down with a 64-deep k-tile: the W_down tile stays row-major
// ([k][n], as it lies in memory) in LDS and the K-major MFMA B-fragments come from
// ds_read_b64_tr_b16 transpose reads (in each 16-lane group lane t = 4r + c4 supplies row
// k0 + r, columns 4*c4..4*c4+3 and receives column t of rows k0..k0+3).
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
constexpr int DBK = 64;
constexpr int DA_PITCH = DBK * 2 + 16;          // h tile row pitch (bytes)
constexpr int DB_PITCH = BN * 2 + 32;           // W_down tile row pitch: 4 rows of a transpose read hit distinct banks

template <bool PROBE>
__global__ void __launch_bounds__(256, 3)
k_prefix_down_bf16(const DownParams p)
{
    if (PROBE && p.skip && *p.skip) return;
    __shared__ __align__(16) char s_a[BM * DA_PITCH];
    __shared__ __align__(16) char s_b[DBK * DB_PITCH];
    __shared__ float s_rs[2][BM];

    const int total = p.n_tm * p.n_tn;
    const int tile = remap_block(blockIdx.x, total);
    if (tile >= total) return;
    const int tm = tile % p.n_tm, tn = tile / p.n_tm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const size_t hrow = (size_t)p.Fp * 2, wrow = (size_t)p.d * 2;

    f32x16 acc[2][2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.0f;

    u32x4 ra[4], rb[4];
    auto load_tile = [&](int kt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = tid + i * 256;
            u32x4 z = {0u, 0u, 0u, 0u};
            {   // h tile: 128 rows x 8 chunks
                const int row = c >> 3, ch = c & 7;
                const size_t kbyte = (size_t)kt * DBK * 2 + ch * 16;
                const int t = tm * BM + row;
                ra[i] = (t < p.T && kbyte < hrow) ? *reinterpret_cast<const u32x4 *>(p.h + (size_t)t * hrow + kbyte) : z;
            }
            {   // W_down tile: 64 rows x 16 chunks
                const int k = c >> 4, ch = c & 15;
                const int j = kt * DBK + k;
                const size_t nbyte = (size_t)tn * BN * 2 + ch * 16;
                rb[i] = (j < p.F && nbyte < wrow) ? *reinterpret_cast<const u32x4 *>(p.wd + (size_t)j * wrow + nbyte) : z;
            }
        }
    };
    const int nk = (p.F + DBK - 1) / DBK;
    const int r32 = lane & 31, q = lane >> 5;
    const int g = lane >> 4, t16 = lane & 15;
    load_tile(0);
    for (int kt = 0; kt < nk; ++kt) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = tid + i * 256;
            *reinterpret_cast<u32x4 *>(s_a + (c >> 3) * DA_PITCH + (c & 7) * 16) = ra[i];
            *reinterpret_cast<u32x4 *>(s_b + (c >> 4) * DB_PITCH + (c & 15) * 16) = rb[i];
        }
        __syncthreads();
        if (kt + 1 < nk) load_tile(kt + 1);
#pragma unroll
        for (int ks = 0; ks < DBK / 16; ++ks) {
            bf16x8 a[2], b[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                a[mb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
                            s_a + (wm * 64 + mb * 32 + r32) * DA_PITCH + (ks * 16 + q * 8) * 2));
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const char *src = s_b + (ks * 16 + 8 * (g >> 1) + (t16 >> 2)) * DB_PITCH +
                                  (wn * 64 + nb * 32 + 16 * (g & 1) + 4 * (t16 & 3)) * 2;
                const s16x4_t b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3))) *)src);
                const s16x4_t b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3))) *)(src + 4 * DB_PITCH));
                const uint2 u0 = __builtin_bit_cast(uint2, b0), u1 = __builtin_bit_cast(uint2, b1);
                b[nb] = __builtin_bit_cast(bf16x8, u32x4{u0.x, u0.y, u1.x, u1.y});
            }
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mb], b[nb], acc[mb][nb], 0, 0, 0);
        }
    }
    if (p.rowsq) down_rowsq(acc, p, tm, tn, wm, wn, lane, tid, s_rs);
    if (PROBE && p.y32) down_store32(acc, p, rows32_of(p), tm, tn, wm, wn, lane);
    if (!p.y) return;
    const int n = lane & 31;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int col = tn * BN + wn * 64 + nb * 32 + n;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int t = tm * BM + wm * 64 + mb * 32 + acc_row(r, lane);
                if (t < p.T && col < p.d)
                    reinterpret_cast<unsigned short *>(p.y)[(size_t)t * p.d + col] =
                        (unsigned short)f32_to_bf16_bits(acc[mb][nb][r] + (p.bias ? p.bias[col] : 0.0f));
            }
    }
}

// bf16 down projection on the pipelined tiles (d % 256 == 0), 256 columns of W_down a tile as they lie in memory: S::TM tokens x 256
// columns x one of the S ranges the neurons are split into.  (128 tokens: split only, for a wave then holds half a tile of the row
// norms.)
template <class S, bool PROBE, bool SOME = false>
__global__ void __launch_bounds__(512, 2)
k_prefix_down_tiles(const DownParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (PROBE && p.skip && *p.skip) return;
    __shared__ __align__(16) char s_w[S::LDS];
    struct Tile {
        struct Id { int tm, tn, ks, pos; };                 // pos: place in a chain
        int blocks, n_tm, n_tn, parts, chain;
        __device__ __forceinline__ bool operator()(int it, Id &id) const
        {
            const int tile = SOME ? it / chain : it;
            const int o = tile_order(tile, blocks, n_tm * n_tn * parts);
            if (o < 0) return false;
            id.pos = it - tile * (SOME ? chain : 1);
            id.ks = o / (n_tm * n_tn);                      // a range's tiles side by side: they share rows of W_down and columns of h
            tile_coords(o - id.ks * n_tm * n_tn, n_tm, n_tn, id.tm, id.tn);
            return true;
        }
    };
    const Tile tile{(int)gridDim.x, (p.T + S::TM - 1) / S::TM, p.d / 256, SOME ? p.parts : p.S, SOME ? p.chain : 1};
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t hrow = (size_t)p.Fp * 2, wrow = (size_t)p.d * 2;
    int vw[S::PW];
#pragma unroll
    for (int i = 0; i < S::PW; ++i) {                       // two rows a transfer; 32-byte piece s of row r at s ^ ((r & 3) | (r >> 3 & 1) << 2)
        const int row = 2 * wave + 16 * i + (lane >> 5), f = (row & 3) | ((row >> 3 & 1) << 2), at = lane & 31;
        vw[i] = row * (int)wrow + ((((at >> 1) ^ f) << 1) | (at & 1)) * 16;
    }
    const int nk_all = p.Fp / 64;                           // h is zero past d_ff, W_down is taken as zero there
    auto src = [&](const typename Tile::Id &id) {
        const int ks = id.ks + (SOME ? p.ks0 + id.pos : 0), kt0 = (int)((long long)ks * nk_all / p.S);
        TileSrc s;
        s.nk = (int)((long long)(ks + 1) * nk_all / p.S) - kt0;
        s.x = p.h + (size_t)id.tm * S::TM * hrow + (size_t)kt0 * 128;
        s.x_bytes = (unsigned int)(min(p.T - id.tm * S::TM, S::TM) * (int)hrow - kt0 * 128);
        s.w = p.wd + (size_t)kt0 * 64 * wrow + (size_t)id.tn * 512;
        s.w_bytes = 0;
        s.w_rows = p.F - kt0 * 64;
        s.w_pitch = (int)wrow;
        s.w_col = id.tn * 512;
        return s;
    };
    f32x4 sum[SOME ? 4 : 1][SOME ? 2 * S::NB : 1];
    auto epi = [&](const f32x4 (&acc)[4][2 * S::NB], const typename Tile::Id &id, unsigned int, int wm, int wn) {
        const int n = lane & 15, q = lane >> 4;
        const int t0 = id.tm * S::TM + wm * 64, c0 = id.tn * 256 + wn * 32 * S::NB;
        const bool full = t0 + 64 <= p.T;
        if (SOME || p.part_out || (PROBE && p.y32)) {       // split: fp32 partial sums, added up by k_prefix_down_combine
            float *rows32 = !PROBE || SOME || p.part_out ? p.part_out + (size_t)id.ks * p.T * p.d : rows32_of(p);
            const unsigned int v = (unsigned int)(4 * q * p.d + n) * 4u;
            auto each = [&](auto f) {                       // the fp32 words of this lane
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        char *dst = reinterpret_cast<char *>(rows32 + (size_t)(t0 + 16 * i + r) * p.d + c0);
                        if (full || t0 + 16 * i + 4 * q + r < p.T)
#pragma unroll
                            for (int j = 0; j < 2 * S::NB; ++j) f(i, j, r, *reinterpret_cast<float *>(dst + v + 64 * j));
                    }
            };
            if constexpr (SOME) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 2 * S::NB; ++j) sum[i][j] = id.pos == 0 ? acc[i][j] : sum[i][j] + acc[i][j];
                if (id.pos + 1 < p.chain) return;
                // (all loads before the first store)
                if (p.add && id.ks == 0) each([&](int i, int j, int r, float &at) { sum[i][j][r] += at; });
                each([&](int i, int j, int r, float &at) { at = sum[i][j][r]; });
            } else {
                each([&](int i, int j, int r, float &at) { at = acc[i][j][r]; });
            }
            if (!PROBE || SOME || p.part_out) return;
        }
        if constexpr (S::NB == 4) {                         // a wave holds one 128-column tile of the row norms
            if (p.rowsq) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float v = 0.0f;
#pragma unroll
                        for (int j = 0; j < 8; ++j) v = fmaf(acc[i][j][r], acc[i][j][r], v);
                        v += __shfl_xor(v, 8);
                        v += __shfl_xor(v, 4);
                        v += __shfl_xor(v, 2);
                        v += __shfl_xor(v, 1);
                        const int t = t0 + 16 * i + 4 * q + r;
                        if (n == 0 && t < p.T) p.rowsq[(size_t)(c0 >> 7) * p.T + t] = v;
                    }
            }
        }
        if (!p.y) return;
        const unsigned int v = (unsigned int)(4 * q * p.d + n) * 2u;
#pragma unroll
        for (int j = 0; j < 2 * S::NB; ++j) {
            const float bv = p.bias ? p.bias[c0 + 16 * j + n] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    char *dst = p.y + ((size_t)(t0 + 16 * i + r) * p.d + c0) * 2;
                    if (full || t0 + 16 * i + 4 * q + r < p.T) *reinterpret_cast<unsigned short *>(dst + v + 32 * j) = bf16_of(acc[i][j][r] + bv);
                }
        }
    };
    tile_products<S>(s_w, (int)hrow, vw, tile, src, epi);
#endif
}

// One wave per neuron: ||W_down[j,:]||^2, then fold the token-tile partials (fixed order)
// and write the requested aggregates.
struct ReduceParams {
    const char *wd;
    const float *part;          // [n_tm][4][F]
    int d, F, n_tm, norm_rows;  // ||W_down[j,:]||^2 of the first norm_rows neurons lies in out.A already
    clada_prefix_out out;
};
template <int ES>
__device__ __forceinline__ void reduce_neurons(const ReduceParams &p, int block)
{
    const char *wd = p.wd;
    const float *part = p.part;
    const int d = p.d, F = p.F, n_tm = p.n_tm, norm_rows = p.norm_rows;
    const clada_prefix_out &out = p.out;
    const int lane = threadIdx.x & 63;
    const int j = block * 4 + (threadIdx.x >> 6);
    if (j >= F) return;
    float wn2 = 0.0f;
    if (out.A) {
        wn2 = j < norm_rows ? out.A[j] : row_norm2<ES>(wd + (size_t)j * d * ES, d, lane);
    }
    // token-tile partials: lane l takes tiles l, l + 64, ... (all loads of a wave in flight together),
    // then the lanes are folded in the fixed order of the wave reductions
    float s_abs = 0.f, s_sq = 0.f, mx = 0.f, s_h2 = 0.f;
    for (int tmi = lane; tmi < n_tm; tmi += 64) {
        const float *src = part + (size_t)tmi * 4 * F + j;
        s_abs += src[0];
        s_sq += src[(size_t)F];
        const float m = src[2 * (size_t)F];
        mx = (m > mx || m != m) ? m : mx;
        s_h2 += src[3 * (size_t)F];
    }
    s_abs = wave_sum(s_abs);
    s_sq = wave_sum(s_sq);
    s_h2 = wave_sum(s_h2);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float m = __shfl_xor(mx, o);
        mx = (m > mx || m != m) ? m : mx;                 // a NaN sticks
    }
    if (lane == 0) {
        if (out.sum_abs_act) out.sum_abs_act[j] = s_abs;
        if (out.sum_sq_act) out.sum_sq_act[j] = s_sq;
        if (out.max_abs_act) out.max_abs_act[j] = mx;
        if (out.sum_sq_h) out.sum_sq_h[j] = s_h2;
        if (out.A) out.A[j] = sqrtf(s_h2) * sqrtf(wn2);
    }
}

template <int ES>
__global__ void __launch_bounds__(256) k_prefix_reduce(const ReduceParams p) { reduce_neurons<ES>(p, blockIdx.x); }

// Sum of the S split-K partial outputs [S][T][d] in ascending order, then what the direct epilogue does:
// y in bf16 (+ bias) and / or the per-row sums of squares of every 128-column tile.  A workgroup takes
// 8 rows x 128 columns: thread = (row tid >> 5, four columns 4 (tid & 31) ..).  The workgroups behind the first `blocks` do the
// per-neuron reductions of the same call, which need nothing of this (bf16; 512 tokens of 4096 x 11008: 22.6 us in two launches and
// eight parts, 16.8 so and with four).  y (fp32) or y32 may be the first part itself: a thread writes what only it has read.
template <int ES>
__global__ void __launch_bounds__(256)
k_prefix_down_combine(int blocks, const ReduceParams red, const float *part, int S, int T, int d, char *y,
                      const float *__restrict__ bias, float *__restrict__ rowsq, float *y32, const int *__restrict__ skip,
                      float *y32_alt, const int *__restrict__ alt)
{
    if ((int)blockIdx.x >= blocks) {
        reduce_neurons<ES>(red, blockIdx.x - blocks);
        return;
    }
    if (skip && *skip) return;
    if (alt && *alt == 0) y32 = y32_alt;
    const int tiles = (T + 7) / 8, tile = blockIdx.x / tiles;
    const int t = (blockIdx.x - tile * tiles) * 8 + (threadIdx.x >> 5);
    const int col = tile * 128 + 4 * (threadIdx.x & 31);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    const bool here = t < T && col < d;                     // (d is a multiple of 4)
    if (here) {
        for (int k = 0; k < S; ++k) {
            const float4 v = *reinterpret_cast<const float4 *>(part + ((size_t)k * T + t) * d + col);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
    }
    if (rowsq) {
        float v = fmaf(s.x, s.x, fmaf(s.y, s.y, fmaf(s.z, s.z, s.w * s.w)));
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 8);
        v += __shfl_xor(v, 4);
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 1);
        if ((threadIdx.x & 31) == 0 && t < T) rowsq[(size_t)tile * T + t] = v;
    }
    if (y32 && here) *reinterpret_cast<float4 *>(y32 + (size_t)t * d + col) = s;
    if (y && here) {
        if (bias) {
            const float4 b = *reinterpret_cast<const float4 *>(bias + col);
            s.x += b.x; s.y += b.y; s.z += b.z; s.w += b.w;
        }
        if (ES == 4) {
            *reinterpret_cast<float4 *>(y + ((size_t)t * d + col) * 4) = s;
            return;
        }
        uint2 o;
        o.x = f32_to_bf16_bits(s.x) | (f32_to_bf16_bits(s.y) << 16);
        o.y = f32_to_bf16_bits(s.z) | (f32_to_bf16_bits(s.w) << 16);
        *reinterpret_cast<uint2 *>(y + ((size_t)t * d + col) * 2) = o;
    }
}

}  // namespace

// Bytes a call needs for certain, and with room for all parts of the down projection's split.
size_t clada_ws_prefix(int32_t d, int32_t d_ff, int32_t T, bool want_y)
{
    if (T <= 0) return 0;
    const size_t n_tm = (size_t)(T + BM - 1) / BM;
    size_t need = align_up(sizeof(float) * 4 * n_tm * d_ff, 256);
    if (want_y) need += align_up((size_t)T * align_up((size_t)d_ff, 64) * 4, 256) + clada_ws_down_splitk(d, d_ff, T);
    return need;
}
size_t clada_ws_prefix_room(int32_t d, int32_t d_ff, int32_t T)
{
    if (T <= 0) return 0;
    return clada_ws_prefix(d, d_ff, T, true) - clada_ws_down_splitk(d, d_ff, T) + clada_ws_down_room(d, d_ff, T);
}

int clada_prefix_token_tiles(int T) { return (T + BM - 1) / BM; }

// Parts that 256 x 256 tiles of the bf16 down projection split d_ff into where they leave compute units idle (fewer than 192): about one
// workgroup per unit, every part at least 256 neurons, at most 8.  1 = no split.
static int down_splits(int d, int F, int T)
{
    if (T <= 0 || d % 256 != 0) return 1;
    const int tiles = ((T + 255) / 256) * (d / 256);
    if (tiles >= 192) return 1;
    int S = 256 / tiles;
    if (S > 8) S = 8;
    if (S > F / 256) S = F / 256;
    return S < 2 ? 1 : S;
}
// The same for tiles of 128 tokens, up to 12 parts, if they are taken: where a part is short, the partial outputs weigh more than the
// operands that a smaller tile reads again (whole calls, us, 256 / 128 tokens: 333 x 2560 x 10240 77.5 / 72.8, 512 x 4096 x 11008
// 136 / 130, 16 x 4096 x 11008 81.9 / 71.3, 200 x 2048 x 8191 56 / 52; parts of more than 4096 neurons: 512 x 5120 x 13824 213 / 220,
// 333 x 8192 x 20011 423 / 438, 777 x 4096 x 11008 218 / 211).  0: not taken.
static int down_splits_half(int d, int F, int T)
{
    if (T <= 0 || d % 256 != 0) return 0;
    int S = 256 / (((T + 127) / 128) * (d / 256));
    if (S > 12) S = 12;
    if (S > F / 256) S = F / 256;
    return S < 2 || F / S > 4096 ? 0 : S;
}
// The split of a call, by its shape alone: the order of the additions, and with it the last bits of y, must not depend on how much
// workspace there is.  Where not all parts fit, they are formed some at a time (prefix_down).
struct DownSplit { int S; bool half; };                     // parts; bf16: tiles of 128 tokens
// Room that a bf16 call asks for at least (an old rule: d_ff in multiples of 32 only).
size_t clada_ws_down_splitk(int d, int F, int T)
{
    const int S = F % 32 == 0 ? down_splits(d, F, T) : 1;
    return S > 1 ? align_up(sizeof(float) * (size_t)S * T * d, 256) : 0;
}
static DownSplit down_split(bool f32, int d, int F, int T, int tile_mode)
{
    if (f32) {
        // 128 x 128 tiles, d_ff split where they leave units idle (us: 4096 x 11008 at 512 tokens 1037 / 500, 4096 x 9000 at 32 869 / 116,
        // 2048 x 6000 at 200 585 / 81)
        const int tiles = ((T + BM - 1) / BM) * ((d + BN - 1) / BN);
        int S = 256 / tiles < 12 ? 256 / tiles : 12;
        if (S > F / 256) S = F / 256;
        return {S < 2 ? 1 : S, false};
    }
    // (tile_mode 1: the plain kernel.)  At least one [T][d] must be there in any workspace that the call accepts: what it asks for, or
    // the half of h's part that a bf16 h leaves.
    if (d % 256 != 0 || tile_mode == 1 || !(clada_ws_down_splitk(d, F, T) > 0 || align_up((size_t)F, 64) >= 2 * (size_t)d)) return {1, false};
    const int S = down_splits_half(d, F, T);
    if (tile_mode != 2 && S >= 2) return {S, true};
    return {down_splits(d, F, T), false};
}
size_t clada_ws_down_room(int d, int F, int T)
{
    size_t room = clada_ws_down_splitk(d, F, T);
    for (int k = 0; T > 0 && k < 4; ++k) {                  // either type; prefix.tile 0 and 2
        const int S = down_split(k & 1, d, F, T, k & 2).S;
        const size_t n = S > 1 ? align_up(sizeof(float) * (size_t)S * T * d, 256) : 0;
        if (n > room) room = n;
    }
    return room;
}
int clada_prefix_col_tiles(int d) { return (d + BN - 1) / BN; }

// Gate/up GEMM with the fused activation epilogue: part [*n_part][4][F] per-neuron partial aggregates of the token tiles (always
// written, at most clada_prefix_token_tiles(T) of them), pool [T][F] |a| or nullptr, hbuf [T][Fp] h in the layer dtype or nullptr
// (Fp = F rounded up to 64, zero past F).
hipError_t clada_prefix_gateup(const clada_layer *layer, const void *x, int T, float *part, float *pool,
                               char *hbuf, int tile_mode, hipStream_t stream, int num_cu, int *n_part, float *wnorm2, int *norm_rows)
{
    const int d = layer->d, F = layer->d_ff, es = (int)dtype_size(layer->dtype);
    GateUpParams g;
    g.wd = (const char *)layer->w_down; g.wnorm2 = wnorm2;
    const bool relu = layer->kind == CLADA_FFN_RELU;
    g.x = (const char *)x; g.wg = (const char *)layer->w_gate;
    g.wu = (const char *)(relu ? layer->w_gate : layer->w_up);
    g.relu = relu ? 1 : 0; g.b_in = relu ? layer->b_in : nullptr;
    g.gelu = layer->kind == CLADA_FFN_GEGLU ? 1 : 0;
    g.T = T; g.d = d; g.F = F; g.n_tm = (T + BM - 1) / BM; g.n_tn = (F + BN - 1) / BN;
    g.part = part; g.pool = pool; g.hbuf = hbuf;
    g.Fp = (int)align_up((size_t)F, 64);
    if (norm_rows) *norm_rows = 0;
    if (num_cu <= 0) num_cu = 256;
    const int total = g.n_tm * g.n_tn;
    if (es == 4 || d % 64 != 0) {
        if (n_part) *n_part = g.n_tm;
        g.n_tn = (F + 63) / 64;
        const auto kern = T <= 64 ? (es == 4 ? k_prefix_gateup<4, 64> : k_prefix_gateup<2, 64>) : (es == 4 ? k_prefix_gateup<4, 128> : k_prefix_gateup<2, 128>);
        hipLaunchKernelGGL(kern, dim3((g.n_tm * g.n_tn + 7) / 8 * 8), dim3(256), 0, stream, g);
        return hipGetLastError();
    }
    // tile_mode: 0 = choose, 1 = 128-token tiles, 2 = 256-token tiles
    // 128-token tiles as long as they all run at once, one per compute unit; beyond, the single round of the 256-token ones is shorter
    // than two (us with statistics, 128- / 256-token tiles: 4096 x 14336 at 200 tokens, 224 / 112 tiles: 84.5 / 91.7, at 333: 130 / 105;
    // 4096 x 11008 at 256: 62.3 / 82.3, at 333, 258 / 172 tiles: 108 / 79.6; at 4096 x 14336 and 2048 tokens 405 / 380).
    const bool wide = tile_mode == 2 || (tile_mode == 0 && T > 128 && total > num_cu);
    const int n_tmw = (T + 255) / 256;
    // One workgroup fills a compute unit, and the units left over take the norms of W_down along, instead of a second pass over it
    // (7B layer, 512 tokens: k_prefix_reduce 16.5 -> 4.5 us), as far as they are done by the time the tiles are: `most` rows per
    // quarter of a unit, all of them or (`some`) the first ones.
    auto launch = [&](auto kern, int tiles, int token_tiles, int most, int cap, bool some = false) {
        const int units = num_cu / 8 * 8 > 8 ? num_cu / 8 * 8 : 8, padded = (tiles + 7) / 8 * 8;
        g.gemm_blocks = padded < units ? padded : units;
        const int spare = num_cu - g.gemm_blocks;
        if (most > cap) most = cap;
        g.norm_rows = F <= 4 * spare * most ? F : some ? 4 * spare * most : 0;
        g.norm_blocks = wnorm2 && norm_rows && g.norm_rows > 0 ? spare : 0;
        if (g.norm_blocks) *norm_rows = g.norm_rows;
        if (n_part) *n_part = token_tiles;
        hipLaunchKernelGGL(kern, dim3(g.gemm_blocks + g.norm_blocks), dim3(512), 0, stream, g);
        return hipGetLastError();
    };
    const int most_wide = 24 + d / 32, most_two = 16 + d / 64, most_one = 20 + d / 128;
    if (relu) {
        if (wide) return launch(k_prefix_gateup_tiles<TileShape<4, 4, 2, false>, true>, n_tmw * ((F + 255) / 256), n_tmw, most_wide, 57);
        return launch(k_prefix_gateup_tiles<TileShape<2, 1, 4, false, true>, true>, total, g.n_tm, most_one, 50);
    }
    if (wide) {
        // Tiles of 96 neurons where rounds of three quarters the length do not grow by more than an eighth in number: the last round
        // fills the chip better (us, 128 / 96 neurons: 4096 x 11008 at 700 tokens 175 / 145, at 1500 268 / 225, at 2048 284 / 296;
        // 4096 x 14336 at 512 tokens 115 / 154).  Not for rows of 512 values (24 / 22 at 512 x 12288, 512 tokens), whose norms
        // go along on the units that the wider tiles leave.
        const int t256 = n_tmw * ((F + 127) / 128), t192 = n_tmw * ((F + 95) / 96);
        if (d > 512 && 8 * ((t192 + num_cu - 1) / num_cu) < 9 * ((t256 + num_cu - 1) / num_cu))
            return launch(k_prefix_gateup_tiles<TileShape<4, 3, 2, false>, false>, t192, n_tmw, most_wide, 57, true);
        return launch(k_prefix_gateup_tiles<TileShape<4, 4, 2, false>, false>, t256, n_tmw, most_wide, 57);
    }
    // one token tile and units left over: 64 neurons a tile (us, 128 / 64 neurons: 4096 x 11008 at 64 tokens 64.5 / 49.5, 2560 x 10240
    // 38.5 / 32.6, 4096 x 14336 79.5 / 73.7; more than one round: 8192 x 20011 183 / 212)
    if (T <= 128 && 2 * total <= num_cu)
        return launch(k_prefix_gateup_tiles<TileShape<2, 1, 4, false, true>, false>, g.n_tm * ((F + 63) / 64), g.n_tm, most_two, 50);
    return launch(k_prefix_gateup_tiles<TileShape<2, 2, 2, false>, false>, total, g.n_tm, most_two, 50);
}

// Down projection of h [T][Fp]: y [T][d] in the layer dtype and/or rowsq [col tiles][T], the
// per-column-tile sums of squares of the fp32 output rows, and/or y32 [T][d], those rows without a bias (any may be
// nullptr; with alt, a device flag, y32 is y32_alt when it is 0).  room: where the partial outputs of a split go.  skip: device
// flag, nothing is computed when it is set (nullptr: always computed).
// red: the call's per-neuron reductions, done along where a pass combines the parts of a split (*red_done).
static hipError_t prefix_down(const clada_layer *layer, const char *h, int T, char *y, float *rowsq, const DownRoom &room,
                              int tile_mode, hipStream_t stream, int num_cu, float *y32, const int *skip, float *y32_alt, const int *alt,
                              const ReduceParams *red, bool *red_done)
{
    const int d = layer->d, F = layer->d_ff, es = (int)dtype_size(layer->dtype);
    DownParams q;
    q.y32 = y32; q.skip = skip; q.y32_alt = y32_alt; q.alt = alt;
    q.h = h; q.wd = (const char *)layer->w_down; q.y = y; q.rowsq = rowsq;
    q.bias = (layer->kind == CLADA_FFN_RELU && y) ? layer->b_out : nullptr;
    q.T = T; q.d = d; q.F = F; q.Fp = (int)align_up((size_t)F, 64);
    q.n_tm = (T + BM - 1) / BM; q.n_tn = (d + BN - 1) / BN;
    q.part_out = nullptr; q.ks0 = q.add = 0; q.chain = 1;
    const bool probe = y32 || skip;
    const DownSplit split = down_split(es == 4, d, F, T, tile_mode);
    q.S = split.S;
    const size_t one = sizeof(float) * (size_t)T * d;
    float *parts = room.bytes >= one ? room.parts : room.one;
    const int fit = room.bytes >= one ? (room.bytes / one < (size_t)q.S ? (int)(room.bytes / one) : q.S) : 1;
    if (q.S > 1 && !parts) return hipErrorInvalidValue;     // (every caller has room for one)
    if (q.S > 1) q.part_out = parts;
    auto product = [&](int n) {                             // n parts, from ks0 on
        q.parts = n;
        const bool some = n < q.S || q.chain > 1;
        if (es == 4) {
            const auto kern = some ? k_prefix_down<true, true> : probe ? k_prefix_down<true> : k_prefix_down<false>;
            hipLaunchKernelGGL(kern, dim3((q.n_tm * q.n_tn * n + 7) / 8 * 8), dim3(256), 0, stream, q);
        } else if (d % 256 != 0 || tile_mode == 1) {        // tile_mode 1 = 128 x 128 tiles of the plain kernel always
            hipLaunchKernelGGL((probe ? k_prefix_down_bf16<true> : k_prefix_down_bf16<false>), dim3((q.n_tm * q.n_tn + 7) / 8 * 8), dim3(256), 0,
                               stream, q);
        } else {                                            // (some: 128-token tiles always, an element's sum is the same)
            using Half = TileShape<2, 2, 2, true>;
            using Whole = TileShape<4, 4, 2, true>;
            const auto kern = some ? k_prefix_down_tiles<Half, true, true>
                            : split.half ? (probe ? k_prefix_down_tiles<Half, true> : k_prefix_down_tiles<Half, false>)
                                         : (probe ? k_prefix_down_tiles<Whole, true> : k_prefix_down_tiles<Whole, false>);
            const int tiles = (some || split.half ? (T + 127) / 128 : (T + 255) / 256) * (d / 256);
            const int units = num_cu / 8 * 8 > 8 ? num_cu / 8 * 8 : 256, padded = (tiles * n + 7) / 8 * 8;
            hipLaunchKernelGGL(kern, dim3(padded < units ? padded : units), dim3(512), 0, stream, q);
        }
        return hipGetLastError();
    };
    auto combine = [&](int n, bool last) {                  // of n parts; not the last ones: in place of the first
        const int blocks = (T + 7) / 8 * q.n_tn;
        ReduceParams r = {};
        const bool reduce = last && red;
        if (reduce) { r = *red; *red_done = true; }
        hipLaunchKernelGGL((es == 4 ? k_prefix_down_combine<4> : k_prefix_down_combine<2>), dim3(blocks + (reduce ? (F + 3) / 4 : 0)), dim3(256), 0,
                           stream, blocks, r, parts, n, T, d, last ? y : nullptr, last ? q.bias : nullptr, last ? rowsq : nullptr,
                           last ? y32 : parts, skip, last ? y32_alt : nullptr, last ? alt : nullptr);
        return hipGetLastError();
    };
    if (q.S == 1) return product(1);
    if (fit == 1) {
        // all parts one after the other by the same workgroups (whole calls, us, a launch per part / so: 768 x 2111 at 300 tokens 96 / 60,
        // 4096 x 9001 at 64 208 / 156)
        q.chain = q.S;
        const hipError_t e = product(1);
        return e != hipSuccess ? e : combine(1, true);
    }
    for (;;) {
        const int n = q.S - q.ks0 < fit ? q.S - q.ks0 : fit;
        hipError_t e = product(n);
        if (e != hipSuccess) return e;
        q.ks0 += n;
        if (q.ks0 == q.S) return combine(n, true);
        if (n > 1 && (e = combine(n, false)) != hipSuccess) return e;
        q.add = 1;
    }
}

hipError_t clada_prefix_down(const clada_layer *layer, const char *h, int T, char *y, float *rowsq, const DownRoom &room, int tile_mode,
                             hipStream_t stream, int num_cu, float *y32, const int *skip, float *y32_alt, const int *alt)
{
    return prefix_down(layer, h, T, y, rowsq, room, tile_mode, stream, num_cu, y32, skip, y32_alt, alt, nullptr, nullptr);
}

extern "C" clada_status clada_prefix_stats(clada_ctx *ctx, const clada_layer *layer, const void *x,
                                           int32_t T, void *y, const clada_prefix_out *out,
                                           void *hip_stream)
{
    if (!ctx) return CLADA_ERR_NULL;
    clada_status st = clada_check_layer(ctx, layer);
    if (st != CLADA_OK) return st;
    if (!x || !out) return clada_fail(ctx, CLADA_ERR_NULL, "x or out is NULL");
    if (T < 1 || T > (1 << 20)) return clada_fail(ctx, CLADA_ERR_SHAPE, "T=%d outside [1,2^20]", T);
    if (!aligned16(x) || (y && !aligned16(y))) return clada_fail(ctx, CLADA_ERR_ALIGN, "x and y must be 16-byte aligned");
    const int d = layer->d, F = layer->d_ff;
    const size_t need = CLADA_WS_HEADER + clada_ws_prefix(d, F, T, y != nullptr);
    if (ctx->ws_bytes < need)
        return clada_fail(ctx, CLADA_ERR_WORKSPACE, "workspace %zu < %zu bytes needed", ctx->ws_bytes, need);
    const int es = (int)dtype_size(layer->dtype);
    char *ws = ctx->ws + CLADA_WS_HEADER;
    hipStream_t stream = (hipStream_t)hip_stream;

    float *part = reinterpret_cast<float *>(ws);
    const size_t h_at = align_up(sizeof(float) * 4 * (size_t)clada_prefix_token_tiles(T) * F, 256);
    char *hbuf = y ? ws + h_at : nullptr;
    int norm_rows = 0, n_part = 0;                          // || W_down[j,:] ||^2 of the first norm_rows neurons already lies in out->A
    CLADA_CHECK_HIP(ctx, clada_prefix_gateup(layer, x, T, part, out->abs_act_pool, hbuf, ctx->opt_prefix_tile, stream, ctx->num_cu, &n_part,
                                             out->A, &norm_rows));
    const bool wanted = out->sum_abs_act || out->sum_sq_act || out->max_abs_act || out->sum_sq_h || out->A;
    const ReduceParams red = {(const char *)layer->w_down, part, d, F, n_part, norm_rows, *out};
    bool reduced = !wanted;
    if (y) {
        // a bf16 h fills half of its part, and the partial outputs begin behind it; an fp32 y is room for one
        const size_t split_at = h_at + align_up((size_t)T * align_up((size_t)F, 64) * es, 256);
        const DownRoom room = {reinterpret_cast<float *>(ws + split_at), ctx->ws_bytes - CLADA_WS_HEADER - split_at,
                               es == 4 ? reinterpret_cast<float *>(y) : nullptr};
        CLADA_CHECK_HIP(ctx, prefix_down(layer, hbuf, T, (char *)y, nullptr, room, ctx->opt_prefix_tile, stream, ctx->num_cu, nullptr, nullptr,
                                         nullptr, nullptr, wanted ? &red : nullptr, &reduced));
    }
    if (!reduced) {
        hipLaunchKernelGGL((es == 4 ? k_prefix_reduce<4> : k_prefix_reduce<2>), dim3((F + 3) / 4), dim3(256), 0, stream, red);
        CLADA_CHECK_HIP(ctx, hipGetLastError());
    }
    return CLADA_OK;
}
