// Decode of up to eight tokens per pass on the vector units, every weight row read once per pass: the fp32 layers, and the
// bf16 widths that neither the batch-1 kernel nor the matrix-core path has an instance for (any row of whole 16 bytes).
//
// Work split.  Workgroup p of P owns the neurons (or list entries) p, p + P, .., in rounds of 64:
//   gate   whole rows per wave, a request of UQ KiB ahead of the one being reduced; the tokens' x sits in LDS and feeds
//          TB dot products per weight chunk; lane t forms sigma and the compare of token t
//   list   the neurons at least one token keeps (the union), by ballot
//   up     kept rows dealt to the waves, again TB dots per chunk; h = a u goes to LDS with the neuron's token mask
//   down   a wave owns column chunks wave, wave + 8 of every row and adds h W_down for the tokens that keep the neuron
//          (the others are skipped, not multiplied by zero: their sums stay free of an infinite weight)
// One partial output [tokens][d] per workgroup; k_ffn_finalize adds them in fixed order.
//
// What bounds it: HBM, and the 256 partial outputs (17 MB written and read at four tokens of 4096).  A 4096 x 11008 fp32
// layer at sparsity 0.45, union of independent tokens: 97.4 us at four tokens (526 MB: 5.4 TB/s; 106 with 92 MB of rows requested
// twice), 135 at eight (136); the generic
// kernel, one token per grid row, reads the weights once per token and takes 394 us.
//
// Arithmetic.  fp32: one chain of fmaf per lane and a fixed tree over the wave for the dots; the kept neurons of a workgroup are
// one chain per column, where the generic kernel folds eight waves' shorter chains (error of that layer at four tokens against
// 64 bits: 2.58e-7 here, 2.48e-7 there).  bf16 dots: v_dot2_f32_bf16, which keeps subnormal inputs, products and sums, and adds
// both products with one rounding (rms error over random operands 2.7e-8, two fmaf 2.9e-8).
#include "clada_internal.h"

namespace {

constexpr int NW = 8;

struct MultiParams {
    const char *wg, *wu, *wd, *x;           // x [B][d]
    const float *tau;                       // [B] (unused when dense)
    float *partial;                         // [P][B][d]
    unsigned char *keep;                    // [B][F] or nullptr
    const int *idx, *n_list;                // list run: neuron indices and their count (device), every one kept; or nullptr
    const float *b_in;                      // non-gated family: input bias [F] or nullptr
    int d, F, B, dense, gelu;
};

// Sum over the wave of TB values per lane; lane t of the result holds the total of value t.
template <int TB>
__device__ __forceinline__ float wave_sums(float (&s)[TB], int lane)
{
    float r = 0.0f;
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        const float v = wave_sum(s[t]);
        r = lane == t ? v : r;
    }
    return r;
}

template <int ES, int TB, int SL, bool RELU>
__global__ void __launch_bounds__(NW * 64)
k_ffn_multi(const MultiParams p)
{
    constexpr int VEC = 16 / ES;
    constexpr int UQ = SL == 2 ? 8 : 4;                      // chunks of a request
    constexpr int DCH = SL == 2 ? 8 : 16;                    // kept neurons per down chunk
    extern __shared__ __align__(16) unsigned char s_x[];     // [TB][parts * UQ] KiB, zero beyond the row and the batch
    __shared__ float s_a[64][TB], s_h[2][DCH][TB];
    __shared__ int s_nl[64], s_km[64], s_list[64], s_lkm[64];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x, P = gridDim.x, d = p.d, F = p.F, B = p.B;
    const size_t rowb = (size_t)d * ES;
    const int nch = (int)((rowb + 1023) / 1024), parts = (nch + UQ - 1) / UQ;
    const int xb = parts * UQ * 1024;                        // bytes of a token's x in LDS
    for (int o = tid * 16; o < TB * xb; o += NW * 64 * 16) {
        const int t = o / xb, c = o - t * xb;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (t < B && c < (int)rowb) v = *reinterpret_cast<const u32x4 *>(p.x + t * rowb + c);
        *reinterpret_cast<u32x4 *>(s_x + o) = v;
    }
    const float tau = p.dense || lane >= B ? 0.0f : p.tau[lane];         // token `lane`
    int n_src = F;
    if (p.idx) n_src = min(max(p.n_list[0], 0), F);
    const int ni_all = blk < n_src ? (n_src - blk + P - 1) / P : 0;

    float acc[TB][SL][VEC];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int s = 0; s < SL; ++s)
#pragma unroll
            for (int k = 0; k < VEC; ++k) acc[t][s][k] = 0.0f;

    // UQ chunks of a row; a lane beyond the row reads the request's start instead, and its value counts as zero.  A wave's last request of
    // a phase has no row (real: uniform): it goes to the start of x, which the caches hold, so that there is no branch around the loads
    // and no row of weights is read twice (618 MB for 526 at 4096 x 11008 fp32, four tokens).  How the address is formed decides over
    // registers and the schedule; us with the row read again / offsets from the part / offsets from the row's start:
    //   offsets from the part: fp32 4096 x 11008 at 1, 2, 4 tokens 75.0 / 67.6 / 68.3, 92.7 / 82.1 / 82.8, 106 / 97.4 / 98.3; 2048 x
    //     5504 at 8 tokens 48.9 / 47.1 / 48.8; bf16 3080 x 8192 at 4 46.6 / 45.0 / 46.6
    //   from the row's start (ROW0), 64 accumulators, which leave no registers, and few of them with short fp32 rows: bf16 4104 x 9000 at
    //     4 tokens 73.1 / 76.3 / 71.0, 6152 x 13000 113 / 115 / 108, fp32 3072 x 8192 at 8 97.0 / 97.1 / 95.9, 1536 x 4099 at 4 27.3 /
    //     28.7 / 27.1, 1024 x 2752 16.8 / 17.6 / 16.7
    //   the row again (AGAIN): bf16 2056 x 5504 at 8 tokens 49.2 / 49.8 / 49.5, bounded by the products
    constexpr bool ROW0 = TB * SL * VEC == 64 || (ES == 4 && SL == 1 && TB <= 4), AGAIN = ES == 2 && SL == 1 && TB == 8;
    auto request = [&](u32x4 (&b)[UQ], const char *w, int j, int part, bool real) {
        const int from = ROW0 ? 0 : part * UQ * 1024;
        const char *row = real || AGAIN ? w + (size_t)j * rowb + from : p.x;
        const int end = real || ROW0 ? (int)rowb - from : 0;
#pragma unroll
        for (int c = 0; c < UQ; ++c) {
            const int o = ((ROW0 ? part * UQ : 0) + c) * 1024 + lane * 16;
            b[c] = ld_stream16(row + (o < end ? o : 0));
        }
    };
    auto reduce = [&](const u32x4 (&b)[UQ], int part, float (&s)[TB]) {
#pragma unroll
        for (int c = 0; c < UQ; ++c) {
            const int o = (part * UQ + c) * 1024 + lane * 16;
            u32x4 w = b[c];
            if (o >= (int)rowb) w = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int t = 0; t < TB; ++t) s[t] = dot16<ES>(w, *reinterpret_cast<const u32x4 *>(s_x + t * xb + o), s[t]);
        }
    };
    // the dots of the rows first, first + NW, .. < n (row_of: their weight row) with all tokens; done(i, sums) takes them
    auto rows = [&](const char *w, int first, int n, auto row_of, auto done) {
        if (first >= n) return;
        u32x4 b0[UQ], b1[UQ];
        float s[TB];
        int i = first, q = 0;                                // request being reduced
        request(b0, w, row_of(i), 0, true);
        auto step = [&](const u32x4 (&cur)[UQ], u32x4 (&nxt)[UQ]) -> bool {
            int ni = i, nq = q + 1;
            if (nq == parts) { nq = 0; ni += NW; }
            const bool more = ni < n;
            request(nxt, w, row_of(more ? ni : i), nq, more);
            if (q == 0) {
#pragma unroll
                for (int t = 0; t < TB; ++t) s[t] = 0.0f;
            }
            reduce(cur, q, s);
            if (nq == 0) done(i, s);
            i = ni; q = nq;
            return more;
        };
        while (step(b0, b1) && step(b1, b0)) {}
    };

    int par = 0;
    for (int r0 = 0; r0 < ni_all; r0 += 64) {
        const int ni = min(64, ni_all - r0);
        __syncthreads();                                     // x is there; the arrays below are free
        if (tid < 64) {
            const int i = blk + P * (r0 + min(tid, ni - 1));
            s_nl[tid] = p.idx ? min(max(p.idx[i], 0), F - 1) : i;
        }
        __syncthreads();
        const auto nl = [&](int i) -> int { return __builtin_amdgcn_readfirstlane(s_nl[i]); };
        rows(p.wg, wave, ni, nl, [&](int i, float (&s)[TB]) {
            const float g = wave_sums<TB>(s, lane);
            const int j = nl(i);
            const float a = ffn_act<RELU>(g, p.b_in, (size_t)j, p.gelu);
            const bool keep = lane < B && (p.dense || fabsf(a) >= tau);
            const unsigned long long km = __ballot(keep);
            if (lane < TB) s_a[i][lane] = a;
            if (lane == 0) s_km[i] = (int)km;
            if (p.keep && lane < B) p.keep[(size_t)lane * F + j] = keep ? 1 : 0;
        });
        __syncthreads();
        // every wave derives the same ascending list of the union
        const int km = lane < ni ? s_km[lane] : 0;
        const unsigned long long mask = __ballot(km != 0);
        const int kp = __popcll(mask);
        if ((mask >> lane) & 1ull) {
            const int t = __popcll(mask & ((1ull << lane) - 1ull));
            s_list[t] = lane;
            s_lkm[t] = km;
        }
        for (int c0 = 0; c0 < kp; c0 += DCH, par ^= 1) {
            const int nc = min(DCH, kp - c0);
            u32x4 dn[DCH][SL];
#pragma unroll
            for (int e = 0; e < DCH; ++e) {
                const char *row = p.wd + (size_t)nl(s_list[c0 + min(e, nc - 1)]) * rowb;
#pragma unroll
                for (int s = 0; s < SL; ++s) {
                    const int o = (wave + s * NW) * 1024 + lane * 16;
                    dn[e][s] = ld_stream16(row + (o < (int)rowb ? o : 0));
                }
            }
            if constexpr (RELU) {
                for (int q = tid; q < nc * TB; q += NW * 64) {
                    const int e = q / TB, t = q % TB;
                    s_h[par][e][t] = s_a[s_list[c0 + e]][t];
                }
            } else {
                rows(p.wu, wave, nc, [&](int e) -> int { return nl(s_list[c0 + e]); }, [&](int e, float (&s)[TB]) {
                    const float u = wave_sums<TB>(s, lane);
                    if (lane < TB) s_h[par][e][lane] = s_a[s_list[c0 + e]][lane] * u;
                });
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < DCH; ++e) {
                if (e < nc) {
                    const int m = __builtin_amdgcn_readfirstlane(s_lkm[c0 + e]);
                    float w[SL][VEC];
#pragma unroll
                    for (int s = 0; s < SL; ++s) unpack_row16(dn[e][s], w[s]);
#pragma unroll
                    for (int t = 0; t < TB; ++t) {
                        if ((m >> t) & 1) {
                            const float h = s_h[par][e][t];
#pragma unroll
                            for (int s = 0; s < SL; ++s)
#pragma unroll
                                for (int k = 0; k < VEC; ++k) acc[t][s][k] = fmaf(h, w[s][k], acc[t][s][k]);
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        if (t < B) {
            float *dst = p.partial + ((size_t)blk * B + t) * d;
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                const int col = ((wave + s * NW) * 64 + lane) * VEC;
                if (col < d) {
#pragma unroll
                    for (int k = 0; k < VEC; k += 4)
                        *reinterpret_cast<float4 *>(dst + col + k) =
                            make_float4(acc[t][s][k], acc[t][s][k + 1], acc[t][s][k + 2], acc[t][s][k + 3]);
                }
            }
        }
    }
}

template <int ES, int TB, int SL>
hipError_t launch(const MultiParams &p, int P, bool relu, hipStream_t st)
{
    constexpr int UQ = SL == 2 ? 8 : 4;
    const int nch = (int)(((size_t)p.d * ES + 1023) / 1024);
    const size_t lds = (size_t)TB * ((nch + UQ - 1) / UQ) * UQ * 1024;
    auto kern = relu ? k_ffn_multi<ES, TB, SL, true> : k_ffn_multi<ES, TB, SL, false>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(P), dim3(NW * 64), lds, st, p);
    return hipGetLastError();
}

template <int ES, int SL>
hipError_t launch_tokens(const MultiParams &p, int P, bool relu, hipStream_t st)
{
    if (p.B <= 2) return p.B == 1 ? launch<ES, 1, SL>(p, P, relu, st) : launch<ES, 2, SL>(p, P, relu, st);
    if constexpr (ES == 4 || SL == 1) {
        if (p.B > 4) return launch<ES, 8, SL>(p, P, relu, st);
    }
    return launch<ES, 4, SL>(p, P, relu, st);
}

}  // namespace

static void multi_passes(const clada_layer *layer, int B, int *n_pass, int *per)
{
    const int most = (size_t)layer->d * dtype_size(layer->dtype) > 8192 && layer->dtype == CLADA_BF16 ? 4 : 8;
    *n_pass = (B + most - 1) / most;                         // (eight tokens of wide bf16 rows do not fit the registers)
    *per = (B + *n_pass - 1) / *n_pass;
}

// Where it is the faster one (time over the generic kernel's, weights from HBM).  A row is requested in groups of four KiB and
// every pass pays for 1, 2, 4 or 8 tokens, so it is the row's length and how full the passes are that decide, not the layer's
// size (768 x 1536 and 768 x 3072 bf16: 0.81 and 0.84 at 8 tokens, 1.20 and 1.23 at 2; 1536 x 3072 and x 6144: 0.48, 0.50 and
// 0.75, 0.85):
//   - rows of more than 1024 values: 0.17 - 0.94; the non-gated family, whose generic kernel has one phase less, 0.25 - 0.99, but
//     0.97 - 1.1 with two tokens up to 1280 values;
//   - 512 < d <= 1024: fp32 0.74 - 0.97 with 3 to 8 tokens, in several passes where the row nearly fills its group (1024: 0.66 -
//     0.96; 640 and 768: 1.02 and less from seven tokens a pass on, 1.07 - 1.1 below) and 1.07 - 1.2 with two; bf16 0.79 - 1.0
//     with 5 to 8 tokens and full passes of eight, 0.97 - 1.24 else; non-gated fp32 0.68 - 0.95 at 4, 6 - 8 tokens and passes of
//     eight, 0.95 - 1.23 else, bf16 0.88 - 1.5;
//   - up to 512 values: 1.0 - 2.2;
//   - fewer neurons than workgroups: 0.75 - 1.3;
//   - one token: gated fp32 rows above 8 KiB, 0.43 - 0.73 (the generic kernel's accumulators leave it one row in flight); the
//     non-gated family 0.91 - 1.10, bf16 41 / 36 us (3584 x 12032).
bool clada_decode_multi_fits(const clada_layer *layer, int32_t B)
{
    const int d = layer->d;
    const bool f32 = layer->dtype == CLADA_F32, relu = layer->kind == CLADA_FFN_RELU;
    if (B == 1) return f32 && !relu && d > 2048;
    if (layer->d_ff < 256 || d <= 512) return false;
    int n_pass, per;
    multi_passes(layer, B, &n_pass, &per);
    if (d > 1024) return !relu || B >= 3 || d > 1280;
    if (relu) return f32 && (per == 8 || per == 4 || (n_pass == 1 && per >= 6));
    if (f32) return d > 768 ? B >= 3 : per >= 7 || (n_pass == 1 && B >= 3);
    return per == 8 || (n_pass == 1 && per >= 5);
}

hipError_t clada_decode_multi(const clada_layer *layer, const void *x, int32_t B, const float *tau, char *y,
                              unsigned char *keep, float *partial, int P, bool dense, const int32_t *idx,
                              const int32_t *n_list, hipStream_t stream, hipEvent_t *ev)
{
    if (ev && hipEventRecord(ev[0], stream) != hipSuccess) return hipGetLastError();
    const int es = (int)dtype_size(layer->dtype), d = layer->d;
    const bool relu = layer->kind == CLADA_FFN_RELU;
    const bool wide = (size_t)d * es > 8192;
    int n_pass, per;
    multi_passes(layer, B, &n_pass, &per);
    for (int b0 = 0; b0 < B; b0 += per) {
        MultiParams p;
        p.wg = (const char *)layer->w_gate; p.wu = (const char *)layer->w_up; p.wd = (const char *)layer->w_down;
        p.x = (const char *)x + (size_t)b0 * d * es;
        p.tau = tau ? tau + b0 : nullptr;
        p.partial = partial;
        p.keep = keep ? keep + (size_t)b0 * layer->d_ff : nullptr;
        p.idx = idx; p.n_list = n_list;
        p.b_in = relu ? layer->b_in : nullptr;
        p.d = d; p.F = layer->d_ff; p.B = B - b0 < per ? B - b0 : per;
        p.dense = dense ? 1 : 0;
        p.gelu = layer->kind == CLADA_FFN_GEGLU ? 1 : 0;
        const hipError_t e = es == 4 ? (wide ? launch_tokens<4, 2>(p, P, relu, stream) : launch_tokens<4, 1>(p, P, relu, stream))
                                     : (wide ? launch_tokens<2, 2>(p, P, relu, stream) : launch_tokens<2, 1>(p, P, relu, stream));
        if (e != hipSuccess) return e;
        const bool last = b0 + per >= B;
        if (ev && last && (hipEventRecord(ev[1], stream) != hipSuccess || hipEventRecord(ev[2], stream) != hipSuccess)) return hipGetLastError();
        clada_launch_finalize(es, partial, P, p.B, d, y + (size_t)b0 * d * es, stream, relu ? layer->b_out : nullptr);
        const hipError_t f = hipGetLastError();
        if (f != hipSuccess) return f;
        if (ev && last && hipEventRecord(ev[3], stream) != hipSuccess) return hipGetLastError();
    }
    return hipSuccess;
}
