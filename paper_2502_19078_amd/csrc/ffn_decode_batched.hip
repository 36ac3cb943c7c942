// Batched (2 <= B <= 16 a pass, 32 in two tiles) thresholded sparse SwiGLU FFN at decode time on the matrix cores
// (algorithm "CLADA Inference", generation phase; bf16 layers).  With B tokens every weight
// element feeds B multiply-adds, which the vector ALUs cannot sustain at HBM speed, so the
// three projections run as MFMA 16x16x32 (bf16 in, fp32 accumulate) with the tokens as the
// 16-wide M dimension.  Weights are still read once, and only for neurons kept by at least
// one token (the union); every output row uses its own mask.  The GELU-gated family differs in
// sigma only; the non-gated ReLU family has no up projection: kernel A runs gate tiles alone and
// writes h = max(0, g + b_in) with the masks, and b_out is added by kernel C.
//
//   kernel A (gate + up -> h): workgroup p owns a contiguous run of neurons (dealt out evenly, to
//     within one), taken 16 at a time.  Its waves (8; 5 for 5 and 10 KiB rows) split the d (= K)
//     dimension: wave w keeps its slice of x as MFMA A-fragments in registers for the whole kernel
//     and streams its slice of the 16 weight rows as B-fragments (whole-KiB pieces of a row per
//     load instruction, turned into the operand layout through a wave-private LDS tile).  The
//     partial 16x16 tiles of the waves are summed through LDS in fixed order; sigma, the per-token
//     fp32 compare and the per-neuron 16-bit keep masks follow.  The neurons of gate tile i that at
//     least one token keeps (the union) are compacted by ballot and form up tile i: the same MFMA
//     loop over their W_up rows gives u, and h = keep ? a*u : 0, split into two bf16, goes to a [d_ff][16]
//     buffer (the 16 tokens of a neuron = one 64-byte line).  Gate and up tiles alternate (G0 G1 U0 G2 U1
//     ...), so the stream of row loads does not drain between the two projections.  The workgroup
//     also leaves the list of its union-kept neurons, ascending, and their count for kernel B.
//   kernel B (down): 2-D split -- column groups of 256 x row groups (a fixed range of neuron
//     indices each: the lists of the gate/up workgroups that own them, laid end to end), so only
//     R partial y's exist instead of one per workgroup.  Work is dealt to the waves in units of 32
//     neurons x 128 columns (wave w: column half w & 1, neuron blocks w >> 1, + 4, ...).  W_down
//     rows arrive as 256-byte segments, are staged per wave in LDS and read
//     back K-major with ds_read_b64_tr_b16 as MFMA B-fragments; h comes as bf16 hi + lo
//     A-fragments (two MFMAs), so the down projection keeps ~fp32 accuracy of h.
//   kernel C: k_ffn_finalize adds the R partials in fixed order.
#include <atomic>
#include <type_traits>

#include "clada_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;

struct BatParams {
    const char *wg, *wu, *wd, *x;
    const float *tau;           // [B]
    unsigned int *hbuf;         // [F][16 or 32] h, split (neuron-major: a 64-byte line or two per neuron), written for union-kept neurons only
    int *ulist;                 // [F] union-kept neurons: gate/up workgroup q writes its own, ascending, from
                                //     the first neuron it owns (q * F / P) on
    int *ucnt;                  // [P] how many each wrote
    unsigned char *keep;        // [B][F] or nullptr
    float *partial;             // [RG][B][d]
    int d, F, B, P, RG, CG;
    int gelu;                   // sigma = tanh-form GELU instead of SiLU
    const float *b_in;          // non-gated family: input bias [F] or nullptr
    const int *list, *list_n;   // prefix-static run (with DENSE): the neurons are the list_n[0] entries of list
                                // (device), every one kept by every token; nullptr: all F neurons
    int row0, rows;             // this unit's first row of the launch's tokens, and their number (stride of the partials)
    int mt;                     // tiles of 16 tokens a pass
};

// A launch of the whole-stack call runs n units, pass blockIdx.y of the tokens of layer blockIdx.z, as many layers as the workspace
// has room for (BatArgs).  A launch of one unit has kernels of its own, which take BatParams as it stands: through BatArgs, whose
// arrays are a second trip to the kernel arguments, a lone call took 0.3 - 0.8 us longer (16.7 / 17.0 at four tokens of 1024 x 4096,
// 26.4 / 26.9 at two of 3072 x 7674 ReLU, 28.9 / 29.3 at 15 of 2048 x 5792, 100.8 / 101.7 at 25 of 5120 x 10272 ReLU).
constexpr int BAT_LAYERS = 48;                  // BAT_UNITS below fits
struct BatArgs {
    BatParams p;                // of unit 0; B: the tokens of a layer
    int n_pass, per_pass;
    const char *wg[BAT_LAYERS], *wu[BAT_LAYERS], *wd[BAT_LAYERS];
    const float *b_in[BAT_LAYERS];
};
__device__ __forceinline__ BatParams bat_unit(const BatParams &p) { return p; }
__device__ __forceinline__ BatParams bat_unit(const BatArgs &)
{
    // (read through the kernel-argument segment: scalar loads at the unit's index)
    const auto *a = (const __attribute__((address_space(4))) BatArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    BatParams p;
    __builtin_memcpy(&p, &a->p, sizeof(p));
    const int layer = blockIdx.z, unit = layer * gridDim.y + blockIdx.y, t0 = blockIdx.y * a->per_pass;
    p.row0 = layer * p.B + t0;
    p.wg = a->wg[layer]; p.wu = a->wu[layer]; p.wd = a->wd[layer];
    p.b_in = a->b_in[layer];
    p.x += (size_t)p.row0 * p.d * 2;
    if (p.tau) p.tau += p.row0;
    p.hbuf += (size_t)unit * p.F * (16 * p.mt);
    p.ulist += (size_t)unit * p.F;
    p.ucnt += (size_t)unit * COOP_MAX_WGS;
    p.B = min(a->per_pass, p.B - t0);
    return p;
}

// An fp32 h as the sum of two bf16: the rounded value below, the rounded rest above (16 to 17 of its 24 bits).  Split once here and not by every
// column group of the down kernel.  The rest is taken from the rounded product, not from the product inside an fma.  What would round up to infinity
// is cut to the largest bf16 first; an infinite h is that and an infinite rest, so that nothing turns into infinity minus infinity.
__device__ __forceinline__ unsigned int split_bf16(float h)
{
#pragma clang fp contract(off)
    const __bf16 hi = (__bf16)__builtin_amdgcn_fmed3f(h, -0x1.fep127f, 0x1.fep127f), lo = (__bf16)(h - (float)hi);       // (nearest even)
    return (unsigned int)__builtin_bit_cast(unsigned short, hi) | ((unsigned int)__builtin_bit_cast(unsigned short, lo) << 16);
}
// h of a neuron that the token cuts: a zero, and no value of the above (its rest has the sign of h, or is +0).
constexpr unsigned int H_CUT = 0x80000000u;
// What gate/up leaves of h.  Rows of 512, 768, 1536 and 3584 values, whose batches of few tokens and whose other types run on the vector units with
// all of fp32, keep it: the down kernel takes it apart into three bf16, exactly (WHOLE).
constexpr bool whole_h(int d) { return d == 512 || d == 768 || d == 1536 || d == 3584; }
template <bool WHOLE>
__device__ __forceinline__ unsigned int kept_h(float h)
{
    if (!WHOLE) return split_bf16(h);
    return h == 0.0f ? 0u : __float_as_uint(h);                      // (-0 is a cut neuron's)
}

__device__ __forceinline__ f32x4 mfma16(const u32x4 a, const u32x4 b, const f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// a line of zeros in global memory (never written): what a load of a row that does not exist reads
__device__ __align__(16) unsigned int k_zero16[4] = {0u, 0u, 0u, 0u};

// first neuron of gate/up workgroup w of P (w = P: d_ff)
__host__ __device__ __forceinline__ int bat_run_lo(int w, int F, int P) { return (int)((long long)w * F / P); }

constexpr int MAX_TILES = 4;    // 16-neuron tiles per workgroup in kernel A (one 64-lane ballot compacts them)

// NW waves split d; KSTEPS = k-steps of 32 per wave: d = NW * KSTEPS * 32.  (NW = 5 gives the 5 and
// 10 KiB rows whole-KiB slices; with 8 waves they would be 640 bytes, which streams slower.)
// LIST (with DENSE): the neurons are the entries of p.list, looked up through LDS; without it neuron
// indices are plain arithmetic on the run's start (fewer registers: the 10 and 16 KiB rows need that).
// RELU: the non-gated family (gate tiles only).  A template flag: as a run-time one it cost the
// 10 and 16 KiB rows ~25 registers and pushed them into scratch (52 -> 68 us at the 13B shape).
// MT: tiles of 16 tokens; two share every fragment of the weights, so that 17 to 32 tokens read them once.  x takes 8 KSTEPS registers
// then, which rows of up to 8 KiB leave room for (16 k-steps a wave; 5 to 8 thousand values would be 24 or 32); the instances of 3584 values
// spill 14 - 24 registers, 60 - 100 bytes a lane, and take 68 us for the vector kernel's 253 at 32 tokens of 3584 x 8048 all the same.  us, passes of 16 / so: one layer
// 117 / 69 at 24 tokens of 4096 x 11008, 61.5 / 38.5 of 2048 x 8192, 35 / 22 of 1024 x 3000, 173 / 132 at 33 (three passes / two); six layers at 24 of
// these 578 / 354, 240 / 159, 86 / 67.
template <int KSTEPS, int NW, bool DENSE, bool LIST, bool RELU, int MT, class Args>
__global__ void __launch_bounds__(NW * 64)
k_bat_gateup(const Args args)
{
    const BatParams p = bat_unit(args);
    static_assert(!LIST || DENSE, "a list run keeps every listed neuron");
    static_assert(NW >= 4 && NW <= 8, "the tile reductions run on waves 0..3");
    constexpr bool WHOLE = whole_h(NW * 32 * KSTEPS);
    constexpr int NBUF = MT == 1 ? 2 : 1, NT = NW * 64, ELEMS = 256 * MT, TURNS = (ELEMS + NT - 1) / NT, HS = 16 * MT;
    __shared__ float s_part[NBUF][NW][ELEMS];               // (two of them for two token tiles would not fit beside the rows)
    __shared__ float s_a[MAX_TILES][HS][16];
    __shared__ int s_km[MAX_TILES * 16];
    __shared__ int s_ul[MAX_TILES * 16];
    __shared__ int s_ku[MAX_TILES];
    __shared__ int s_nl[MAX_TILES * 16];                    // neuron index of every entry of the round

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, q = lane >> 4;
    const int blk = blockIdx.x, P = gridDim.x;
    const int d = p.d, F = p.F, B = p.B;
    const size_t rowb = (size_t)d * 2;
    // This wave's k-slice of every row is SLICE bytes, taken in NPART parts of PB <= 1024 bytes.  The
    // loads of eight rows' parts (8 PB bytes) are packed into NL = PB / 128 full instructions of
    // 64 x 16 bytes: lane l of instruction i takes byte 1024 i + 16 l of the eight parts laid end
    // to end, i.e. contiguous pieces of PB bytes (or the two ends of neighbouring rows) -- measured
    // 6.6 TB/s for whole-KiB pieces against 5.6 TB/s for 16 rows x 64 bytes per instruction, which
    // is what the MFMA operand layout would ask for.  The wave then turns 16 such rows into
    // B-fragments through its private LDS tile: row r is written contiguously at r * PITCH, and lane
    // (neuron n, k-group q) reads chunk q * SP + ks of row n for k-step ks.  The order of k within the
    // slice is free as long as x uses the same one.  PITCH = PB + 16 keeps both directions free of
    // bank conflicts.
    constexpr int SLICE = KSTEPS * 64;
    constexpr int NPART = SLICE > 1024 ? 2 : 1;
    constexpr int PB = SLICE / NPART, SP = PB / 64, PITCH = PB + 16;
    constexpr int NL = PB / 128;                            // load instructions per eight rows of a part
    static_assert(PB % 128 == 0 && PB <= 1024 && NPART * SP == KSTEPS, "slice split");
    __shared__ __align__(16) char s_stage[NW * 16 * PITCH];
    char *stage = s_stage + wave * 16 * PITCH;
    const int koff = wave * SLICE;
    int ld_row[NL], ld_col[NL];                             // (row within the eight, byte within the part) of this lane's piece
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int o = 1024 * i + 16 * lane;
        ld_row[i] = o / PB;
        ld_col[i] = o % PB;
    }
    // Neurons are dealt out in contiguous runs: workgroup q owns [q F / P, (q+1) F / P), so every
    // workgroup streams the same number of rows to within one (a row that a tile lacks costs no
    // memory traffic; 16-neuron granularity would leave an eighth of the chip idle at the end).
    // A run longer than 64 neurons (d_ff above 16384) is worked off in rounds of 64.
    // With a list the same holds for its entries (indices clamped into [0, d_ff) like the count).
    const int Fn = LIST ? min(max(p.list_n[0], 0), F) : F;
    const int j_lo_all = bat_run_lo(blk, Fn, P);
    const int j_hi_all = bat_run_lo(blk + 1, Fn, P);

    // this wave's slice of x as A-fragments: lane = (token n, k-group q)
    u32x4 xa[MT][KSTEPS];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            u32x4 v = {0u, 0u, 0u, 0u};
            const int m = 16 * mt + n;
            if (m < B) v = *reinterpret_cast<const u32x4 *>(p.x + (size_t)m * rowb + koff + (ks / SP) * PB + (q * SP + ks % SP) * 16);
            xa[mt][ks] = v;
        }
    __syncthreads();

    auto stage_write = [&](const u32x4 (&wr)[NL], int half) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            *reinterpret_cast<u32x4 *>(stage + (8 * half + ld_row[i]) * PITCH + ld_col[i]) = wr[i];
    };
    // lanes of this wave exchange data through the tile: order the LDS traffic within the wave
    auto wave_sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto part_mma = [&](int part, f32x4 (&acc)[MT]) {
#pragma unroll
        for (int ks = 0; ks < SP; ++ks) {
            const u32x4 frag = *reinterpret_cast<const u32x4 *>(stage + n * PITCH + (q * SP + ks) * 16);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = mfma16(xa[mt][part * SP + ks], frag, acc[mt]);
        }
    };
    auto part_store = [&](const f32x4 (&acc)[MT], int buf) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) s_part[buf][wave][256 * mt + r * 64 + lane] = acc[mt][r];
    };
    // element (mt, r, ln) of the 16x16 tiles: token m = 16 mt + 4*(ln/16) + r, neuron ln%16; waves summed in order
    auto tile_sum = [&](int buf, int e) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += s_part[buf][w][e];
        return s;
    };
    int nlist = 0;                                          // entries of this workgroup's union list so far (uniform)
    // the token this thread compares for in the gate reduction, and its threshold (kept out of the tile loop)
    auto token_of = [&](int e) { return 16 * (e >> 8) + 4 * ((e & 63) >> 4) + ((e & 255) >> 6); };
    float red_tau[TURNS];
#pragma unroll
    for (int k = 0; k < TURNS; ++k) {
        const int e = tid + k * NT;
        red_tau[k] = (!DENSE && e < ELEMS && token_of(e) < B) ? p.tau[token_of(e)] : 0.0f;
    }
    for (int j_lo = j_lo_all; j_lo < j_hi_all; j_lo += 16 * MAX_TILES) {
    const int nown = min(16 * MAX_TILES, j_hi_all - j_lo);  // <= 64
    const int ni = (nown + 15) / 16;                        // <= MAX_TILES
    __syncthreads();                                        // the previous round is done with s_km, s_a, s_ul
    if (tid < MAX_TILES * 16) {
        s_km[tid] = 0;
        if (LIST) s_nl[tid] = tid >= nown ? 0 : min(max(p.list[j_lo + tid], 0), F - 1);
    }
    __syncthreads();

    // Every 16-neuron gate tile G_i is followed, one tile later, by the up tile U_i over the neurons of
    // G_i that at least one token keeps: G0 G1 U0 G2 U1 ... G_{ni-1} U_{ni-2} U_{ni-1}.  The rows of
    // the next tile in this order are requested while the current one is worked on, so the stream of
    // loads never drains between the gate and the up projection; U_i's rows are known by then
    // because G_i was reduced before the tile in front of U_i started.  (A single tile, ni = 1, has
    // nothing to put between G0 and U0: U0's rows are requested only after G0 is reduced.)
    // The non-gated family has gate tiles only: h is the activation itself.
    const int nseq = RELU ? ni : 2 * ni;
    auto seq_tile = [&](int sq, int &up, int &i) {
        if (RELU) { up = 0; i = sq; }
        else if (ni == 1) { up = sq; i = 0; }
        else if (sq < 2) { up = 0; i = sq; }
        else if (sq == nseq - 1) { up = 1; i = ni - 1; }
        else if (sq & 1) { up = 0; i = (sq + 1) >> 1; }
        else { up = 1; i = (sq >> 1) - 1; }
    };
    // Eight rows (half a tile) of one part of gate tile ti (up = 0: its neurons in order) or up tile ti
    // (up = 1: its union-kept neurons through the compacted list).  A row that does not exist reads
    // one shared line of zeros instead (a select on the address: no branch around any load).  up and
    // ti are uniform; the list is read whether used or not, so the loads are issued without a branch
    // on the kind of tile.
    auto rows_load = [&](u32x4 (&wr)[NL], int up, int ti, int part, int half) {
        const char *base = (up ? p.wu : p.wg) + (LIST ? (size_t)0 : (size_t)(j_lo + 16 * ti) * rowb) + koff + part * PB;
        const int lim = up ? s_ku[ti] : nown - 16 * ti;
        int lr[NL];                                         // row relative to base
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int rr = 8 * half + ld_row[i];
            const int viaList = s_ul[16 * ti + rr];
            if (LIST) lr[i] = s_nl[16 * ti + (up ? viaList & 15 : rr)];
            else lr[i] = up ? viaList : rr;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const char *src = 8 * half + ld_row[i] < lim ? base + (size_t)lr[i] * rowb + ld_col[i]
                                                         : reinterpret_cast<const char *>(k_zero16);
            wr[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src));
        }
    };
    auto gate_reduce = [&](int i, int buf) {
#pragma unroll
        for (int k = 0; k < TURNS; ++k) {
            const int e = tid + k * NT;
            if (e < ELEMS) {
                const int m = token_of(e), nn = e & 15, j = LIST ? s_nl[16 * i + nn] : j_lo + 16 * i + nn;
                const bool here = 16 * i + nn < nown, valid = m < B && here;
                float a = tile_sum(buf, e);
                if (RELU) {
                    if (p.b_in && valid) a += p.b_in[j];
                    a = a > 0.0f ? a : (a != a ? a : 0.0f);
                } else {
                    a = gate_sigma_f32(a, p.gelu);
                }
                const bool keep = valid && (DENSE ? true : (fabsf(a) >= red_tau[k]));
                s_a[i][m][nn] = a;
                if (keep) atomicOr(&s_km[i * 16 + nn], 1 << m);
                if (p.keep && valid) p.keep[(size_t)m * F + j] = keep ? 1 : 0;
                if (RELU && here) p.hbuf[(size_t)j * HS + m] = keep ? kept_h<WHOLE>(a) : H_CUT;     // read back for union-kept neurons only
            }
        }
    };
    // Union-kept neurons of gate tile i, compacted by ballot.  Every wave does it for itself (same
    // values to the same LDS words), so a wave only ever reads what it wrote; wave 0 appends them
    // to the workgroup's list in global memory for the down kernel.
    auto compact = [&](int i) {
        const bool mine = lane < 16 && s_km[16 * i + lane] != 0;       // never set past nown
        const unsigned long long bal = __ballot(mine);
        const int pos = __popcll(bal & ((1ull << lane) - 1ull));
        if (mine) s_ul[16 * i + pos] = lane;
        if (lane == 0) s_ku[i] = __popcll(bal);
        if (wave == 0 && mine) p.ulist[j_lo_all + nlist + pos] = LIST ? s_nl[16 * i + lane] : j_lo + 16 * i + lane;
        nlist += __popcll(bal);
        wave_sync();
    };
    auto up_reduce = [&](int i, int buf) {
#pragma unroll
        for (int k = 0; k < TURNS; ++k) {
            const int e = tid + k * NT, m = token_of(e), nn = e & 15;
            if (e < ELEMS && nn < s_ku[i]) {
                const int l2 = s_ul[16 * i + nn];
                const int j = LIST ? s_nl[16 * i + l2] : j_lo + 16 * i + l2;
                const float usum = tile_sum(buf, e);
                const bool keep = (s_km[16 * i + l2] >> m) & 1;
                p.hbuf[(size_t)j * HS + m] = keep ? kept_h<WHOLE>(s_a[i][m][l2] * usum) : H_CUT;
            }
        }
    };

    // D = X_slice * W_slice^T partial over this wave's k-slice, one tile of the sequence after the other
    u32x4 wa[NL], wb[NL];
    bool have = false;                                      // wa/wb hold the rows of the unit about to start
    int ncomp = 0;                                          // gate tiles compacted so far
    for (int sq = 0; sq < nseq; ++sq) {
        int up, ti, nup = 0, nti = 0;
        seq_tile(sq, up, ti);
        bool nready = false;                                  // the tile after this one can be requested already
        if (sq + 1 < nseq) {
            seq_tile(sq + 1, nup, nti);
            nready = !nup || nti < ncomp;
        }
        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int part = 0; part < NPART; ++part) {            // unrolled: x fragments stay in registers
            if (!have) {
                rows_load(wa, up, ti, part, 0);
                rows_load(wb, up, ti, part, 1);
            }
            const bool last = part == NPART - 1;
            const bool nxt = last ? nready : true;
            const int lup = last ? nup : up, lti = last ? nti : ti, lpart = last ? 0 : part + 1;
            wave_sync();                                      // the previous part's fragment reads are done
            if (nxt) {
                stage_write(wa, 0);
                rows_load(wa, lup, lti, lpart, 0);
                stage_write(wb, 1);
                rows_load(wb, lup, lti, lpart, 1);
            } else {
                stage_write(wa, 0);
                stage_write(wb, 1);
            }
            have = nxt;
            wave_sync();
            part_mma(part, acc);
        }
        const int buf = NBUF == 2 ? sq & 1 : 0;
        part_store(acc, buf);
        __syncthreads();
        if (!up) {
            gate_reduce(ti, buf);
            __syncthreads();                                  // the tile's keep masks are complete
            compact(ti);
            ++ncomp;
        } else {
            up_reduce(ti, buf);
            if (NBUF == 1) __syncthreads();                  // the sums are read before the next tile's are written
        }
    }
    }   // rounds
    if (tid == 0) p.ucnt[blk] = nlist;
}

constexpr int DN_COLS = 256;                    // columns per workgroup in kernel B
constexpr int DN_SUB = 128;                     // columns staged per pass
constexpr int DN_PITCH = DN_SUB * 2 + 32;       // LDS row pitch (bytes): 4 rows of a transpose read hit distinct banks
constexpr int DN_TILE_BYTES = 32 * DN_PITCH;    // one wave's staging tile: 32 neurons x 128 columns
constexpr int DN_MAX_ROWS = 2048;               // union neurons per row group
constexpr int DN_MAX_WGS = 64;                  // gate/up workgroups per row group

template <int MT, bool WHOLE, class Args>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_bat_down(const Args args)
{
    const BatParams p = bat_unit(args);
    extern __shared__ __align__(16) unsigned char smem_dn[];
    unsigned char *s_tile = smem_dn;                                    // [8][DN_TILE_BYTES], later the fold buffers
    int *s_rows = reinterpret_cast<int *>(smem_dn + 8 * DN_TILE_BYTES); // [DN_MAX_ROWS]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups go to the 8 XCDs round-robin by id, and each XCD has its own L2.  The column groups of
    // one row group all read the same h lines and row list, so they are given ids of one residue
    // class mod 8 where the grid divides evenly: an h line then crosses the fabric once, not 8 times.
    int wg = blockIdx.x;
    if (gridDim.x % 8 == 0) wg = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const int cg = wg % p.CG, rg = wg / p.CG;
    const int d = p.d, F = p.F, B = p.B;
    const size_t rowb = (size_t)d * 2;
    const int col0 = cg * DN_COLS;

    // ---- this row group's neurons = those of the gate/up workgroups [w0, w1): their union lists, laid end
    // to end (ascending).  The list entries are requested before the counts are known; an entry past
    // its workgroup's count is stale memory inside the list array and is dropped.
    const int w0 = (int)((long long)rg * p.P / p.RG), w1 = (int)((long long)(rg + 1) * p.P / p.RG);
    const int nw = w1 - w0;                                             // <= DN_MAX_WGS (host check)
    const int Fn = p.list ? min(max(p.list_n[0], 0), F) : F;
    auto run_lo = [&](int w) { return bat_run_lo(w, Fn, p.P); };
    const int cnt_l = lane < nw ? p.ucnt[w0 + lane] : 0;               // every wave: the counts, one per lane
    constexpr int PRE = 4;                                              // entries per thread held in registers
    int pre_v[PRE];
#pragma unroll
    for (int k = 0; k < PRE; ++k) {
        const int w = wave + 8 * k;
        const int jj = w < nw ? run_lo(w0 + w) + lane : F;
        pre_v[k] = jj < F ? p.ulist[jj] : 0;
    }
    int inc = cnt_l;                                                    // inclusive scan over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    const int exc = inc - cnt_l;
    const int nrows = __shfl(inc, 63);                                  // <= DN_MAX_ROWS (host check)
#pragma unroll
    for (int k = 0; k < PRE; ++k) {
        const int w = wave + 8 * k, ws = w < nw ? w : 0;
        const int c = __shfl(cnt_l, ws), o = __shfl(exc, ws);
        if (w < nw && lane < c) s_rows[o + lane] = pre_v[k];
    }
    // whatever the registers did not cover: more than 8 * PRE workgroups, or lists longer than 64
    for (int w = wave; w < nw; w += 8) {
        const int c = __shfl(cnt_l, w), o = __shfl(exc, w);
        for (int e = (w < 8 * PRE ? 64 : 0) + lane; e < c; e += 64) s_rows[o + e] = p.ulist[run_lo(w0 + w) + e];
    }
    __syncthreads();

    // Wave w works on column half sub = w & 1 of the workgroup's 256 columns and on the 32-neuron
    // blocks rw, rw + 4, ... (rw = w >> 1): units of 32 rows x 128 columns dealt round-robin, so the
    // eight waves differ by at most one unit.
    const int sub = wave & 1, rw = wave >> 1;
    f32x4 acc[MT][DN_SUB / 16];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < DN_SUB / 16; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int n = lane & 15, q = lane >> 4;
    unsigned char *tile = s_tile + wave * DN_TILE_BYTES;
    const int nkb = (nrows + 31) / 32;
    static_assert(DN_COLS == 2 * DN_SUB, "two staging passes per block of neurons");

    // eight consecutive list entries; past the list the last one again, whose row is on its way already
    const int last_row = nrows > 0 ? s_rows[nrows - 1] : 0;
    auto rows8 = [&](int (&row)[8], int e0) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(s_rows + e0), b = *reinterpret_cast<const u32x4 *>(s_rows + e0 + 4);
#pragma unroll
        for (int i = 0; i < 8; ++i) row[i] = e0 + i < nrows ? (int)(i < 4 ? a[i & 3] : b[i & 3]) : last_row;
    };
    // h[token n][list entries 8 q ..] of block kb (a token that does not exist: the last one again, or in two tiles one that keeps nothing; its sums are
    // not stored).  No branch around any load: eight of them, one after the other behind a look into the list, held every unit up (one layer of
    // 5120 x 13824 at 16 tokens 87.1 / 86.3 us, six of 2048 x 8192 136 / 135); one branch around all eight for the tokens past the batch: lone calls of
    // 1024 x 4096 and 2560 x 8000 at 4 to 16 tokens 0.5 - 1 % slower, 24 ReLU layers of 2560 x 10240 at eight 0.5 % faster.
    auto h_load = [&](unsigned int (&hv)[MT][8], int kb) {
        int row[8];
        rows8(row, 32 * kb + 8 * q);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 8; ++i) hv[mt][i] = p.hbuf[(size_t)row[i] * (16 * MT) + (MT == 1 ? min(n, B - 1) : 16 * mt + n)];
    };
    // W_down[32 list entries][128 columns]: quarter-waves read 256-byte row pieces, lane group q the entries 8 q ..; columns past d cannot
    // occur for the supported widths (d is a multiple of 256)
    auto w_load = [&](u32x4 (&wv)[8], int kb) {
        const char *wcol = p.wd + (size_t)(col0 + sub * DN_SUB + 8 * n) * 2;
        int row[8];
#pragma unroll
        for (int ii = 0; ii < 8; ++ii) row[ii] = s_rows[min(32 * kb + 4 * ii + q, nrows - 1)];
#pragma unroll
        for (int ii = 0; ii < 8; ++ii) wv[ii] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(wcol + (size_t)row[ii] * rowb));
    };
    auto stage = [&](const u32x4 (&wv)[8]) {
#pragma unroll
        for (int ii = 0; ii < 8; ++ii) *reinterpret_cast<u32x4 *>(tile + (4 * ii + q) * DN_PITCH + n * 16) = wv[ii];
    };
    constexpr int PARTS = WHOLE ? 3 : 2;                                // of h, the largest first
    auto process = [&](const u32x4 (&a)[MT][PARTS]) {
        // K-major B-fragments by transpose reads: in each 16-lane group lane t = 4r + c4 supplies
        // row 8q + r, columns 4*c4 .. 4*c4+3 and receives column t of rows 8q .. 8q+3
        const int r = n >> 2, c4 = n & 3;
#pragma unroll
        for (int t = 0; t < DN_SUB / 16; ++t) {
            const unsigned char *src = tile + (8 * q + r) * DN_PITCH + (t * 16 + 4 * c4) * 2;
            const s16x4 b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)src);
            const s16x4 b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(src + 4 * DN_PITCH));
            const uint2 u0 = __builtin_bit_cast(uint2, b0), u1 = __builtin_bit_cast(uint2, b1);
            const u32x4 bf = {u0.x, u0.y, u1.x, u1.y};
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int k = 0; k < PARTS; ++k) acc[mt][t] = mfma16(a[mt][k], bf, acc[mt][t]);
        }
    };
    auto split_h = [&](unsigned int (&hv)[8], u32x4 (&a)[PARTS], int kb) {
#pragma unroll
        for (int i = 0; i < 8; ++i) hv[i] = 32 * kb + 8 * q + i < nrows ? hv[i] : 0u;
        if constexpr (WHOLE) {                               // eight bits at a time, cut, not rounded: nothing is left behind the third
#pragma unroll
            for (int k = 0; k < PARTS; ++k)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const unsigned int top = hv[i] & 0xffff0000u;
                    if (i & 1) a[k][i / 2] |= top;
                    else a[k][i / 2] = top >> 16;
                    hv[i] = __float_as_uint(__uint_as_float(hv[i]) - __uint_as_float(top));
                }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[0][i] = (hv[2 * i] & 0xffffu) | (hv[2 * i + 1] << 16);
                a[1][i] = (hv[2 * i] >> 16) | (hv[2 * i + 1] & 0xffff0000u);
            }
        }
    };
    auto h_value = [](unsigned int v) { return WHOLE ? __uint_as_float(v) : __uint_as_float(v << 16) + __uint_as_float(v & 0xffff0000u); };

    // A unit is requested and consumed in turn; the waves of two workgroups share a compute unit (at most 128
    // registers per lane, 80 KiB of LDS each; four waves a SIMD and no more: left to itself the compiler aims at six and waits for each load
    // in turn, 13 % slower per call), and it is their loads that cover this wave's consumption.
    // (Requesting the next unit before consuming the current one needed 182 registers, one workgroup per
    // compute unit, and was 1.5 - 4 % slower per step, most with a sparse union.)
    u32x4 wA[8];
    unsigned int hA[MT][8];
    for (int kb = rw; kb < nkb; kb += 4) {
        u32x4 a[MT][PARTS];
        if (MT == 1) h_load(hA, kb);
        w_load(wA, kb);
        if (MT == 2) {                                       // (the order that takes the fewest of the 128 registers: three are spilled, one of them read back in the loop)
            __builtin_amdgcn_sched_barrier(0);
            h_load(hA, kb);
            __builtin_amdgcn_sched_barrier(0);
        }
        stage(wA);
        if (MT == 2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) split_h(hA[mt], a[mt], kb);
        process(a);
    }

    // ---- A cut neuron counts as h = 0 above, and 0 times an infinite weight is NaN.  Finite sums prove that no such weight was in the way, so that
    // the loop looks at none.  Where a sum is not, this wave looks for one in its units (or for an infinite h that was taken apart), and if there is one
    // forms its sums again, neuron by neuron, for the tokens that keep it.
    float finite = 0.0f;                                                // NaN unless every sum is
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < DN_SUB / 16; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) finite = fmaf(acc[mt][t][r], 0.0f, finite);
    if (__ballot(finite != 0.0f)) {
        bool bad = false;
#pragma unroll 1
        for (int kb = rw; kb < nkb; kb += 4) {
            w_load(wA, kb);
#pragma unroll
            for (int ii = 0; ii < 8; ++ii)
#pragma unroll
                for (int k = 0; k < 4; ++k) bad = bad || (wA[ii][k] & 0x7f80u) == 0x7f80u || (wA[ii][k] & 0x7f800000u) == 0x7f800000u;
            if constexpr (WHOLE) {
                h_load(hA, kb);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 8; ++i) bad = bad || (hA[mt][i] & 0x7fffffffu) == 0x7f800000u;
            }
        }
        if (__ballot(bad)) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < DN_SUB / 16; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int e0 = 32 * rw; e0 < nrows; e0 += 128)
#pragma unroll 1
                for (int e = e0; e < min(e0 + 32, nrows); ++e) {
                    const int row = s_rows[e];
                    const unsigned short *w = reinterpret_cast<const unsigned short *>(p.wd + (size_t)row * rowb) + col0 + sub * DN_SUB + n;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const u32x4 h = *reinterpret_cast<const u32x4 *>(p.hbuf + (size_t)row * (16 * MT) + 16 * mt + 4 * q);
#pragma unroll
                        for (int t = 0; t < DN_SUB / 16; ++t) {
                            const float wv = __uint_as_float((unsigned int)w[16 * t] << 16);
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const float sum = fmaf(h_value(h[r]), wv, acc[mt][t][r]);
                                acc[mt][t][r] = h[r] != H_CUT ? sum : acc[mt][t][r];
                            }
                        }
                    }
                }
        }
    }

    // ---- fixed-order fold of the four row-waves of each column half through LDS, then the partial
    // y of this row group
    __syncthreads();
    float *s_red = reinterpret_cast<float *>(s_tile);                   // [2 halves][2][8 tiles][4][64]
    constexpr int ACC_FLOATS = MT * (DN_SUB / 16) * 4 * 64;
    static_assert(4 * ACC_FLOATS * sizeof(float) <= 8 * DN_TILE_BYTES, "the folds take the place of the tiles");
#pragma unroll
    for (int s2 = 2; s2 >= 1; s2 >>= 1) {
        if (rw >= s2 && rw < 2 * s2) {
            float *dst = s_red + (size_t)(sub * 2 + (rw - s2)) * ACC_FLOATS;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < DN_SUB / 16; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) dst[((mt * (DN_SUB / 16) + t) * 4 + r) * 64 + lane] = acc[mt][t][r];
        }
        __syncthreads();
        if (rw < s2) {
            const float *src = s_red + (size_t)(sub * 2 + rw) * ACC_FLOATS;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < DN_SUB / 16; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[mt][t][r] += src[((mt * (DN_SUB / 16) + t) * 4 + r) * 64 + lane];
        }
        __syncthreads();
    }
    if (rw == 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < DN_SUB / 16; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + 4 * q + r, col = col0 + sub * DN_SUB + t * 16 + n;
                    if (m < B && col < d) p.partial[((size_t)rg * p.rows + p.row0 + m) * d + col] = acc[mt][t][r];
                }
    }
}

// The final reduction of several layers of the non-gated family, whose output biases differ: y rows [n][B][d] from partials
// [RG][n B][d], in k_ffn_finalize's order (slice q adds the partials q, q + 32, .., then the 32 slices by the fixed tree).
struct BatBiasArgs {
    const float *partial;
    char *y;
    const float *b_out[BAT_LAYERS];
    int RG, B, d;
};
__global__ void __launch_bounds__(256)
k_bat_finalize_bias(const BatBiasArgs a)
{
    constexpr int CG = 8, SL = 32;
    __shared__ float4 s_sum[SL][CG];
    const int cg = threadIdx.x % CG, sl = threadIdx.x / CG;
    const int col = blockIdx.x * (4 * CG) + cg * 4, row = blockIdx.y;
    const size_t pstride = (size_t)gridDim.y * a.d;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col < a.d) {
        const float *base = a.partial + (size_t)row * a.d + col;
        for (int q = sl; q < a.RG; q += SL) {
            const float4 v = *reinterpret_cast<const float4 *>(base + (size_t)q * pstride);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
    }
    s_sum[sl][cg] = s;
    __syncthreads();
#pragma unroll
    for (int h = SL / 2; h >= 1; h >>= 1) {
        if (sl < h) {
            const float4 v = s_sum[sl + h][cg];
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            s_sum[sl][cg] = s;
        }
        __syncthreads();
    }
    if (sl == 0 && col < a.d) {
        const float *bias = a.b_out[row / a.B];
        if (bias) {
            const float4 bv = *reinterpret_cast<const float4 *>(bias + col);
            s.x += bv.x; s.y += bv.y; s.z += bv.z; s.w += bv.w;
        }
        uint2 o;
        o.x = f32_to_bf16_bits(s.x) | (f32_to_bf16_bits(s.y) << 16);
        o.y = f32_to_bf16_bits(s.z) | (f32_to_bf16_bits(s.w) << 16);
        *reinterpret_cast<uint2 *>(a.y + ((size_t)row * a.d + col) * 2) = o;
    }
}

}  // namespace

size_t clada_ws_decode_batched(int32_t d_ff)
{
    return align_up(sizeof(float) * 16 * (size_t)d_ff, 256) + align_up(sizeof(int) * (size_t)d_ff, 256) +
           align_up(sizeof(int) * COOP_MAX_WGS, 256);
}

// Whether a batch is for the matrix cores: rows that have instances of their own kernels; the narrow ones and two odd widths from the batch on that
// the vector kernel or the generic one takes longer for.  Lone calls, us, vector or generic / matrix cores, gated (ReLU): 512 x 2048 at 9 and 12 tokens
// 16.4 / 16.1, 18.8 / 16.1 (14.8 / 16.3, 16.5 / 15.9), 512 x 1024 at 12 and 16 16.5 / 15.6 (15.4 / 15.8, 19.1 / 16.1); 768 x 1536 at 6, 8 and 16 16.6 / 16.0,
// 18.6 / 15.0, 37.1 / 16.2, at 9 25.5 / 16.0 (14.0 / 15.7, 18.0 / 15.7), 768 x 3072 at 8 and 32 22.6 / 15.8, 85 / 23; 1536 x 3072 at 4 and 6 18.8 / 19.5, 24.5 / 19.7,
// 1536 x 6000 25.9 / 23.2, 35.1 / 23.2, a list of 2500 at 4 18.5 / 19.1, 1536 x 4100 at 32 124 / 30 (1536 x 3072 at 4, 5 and 9 15.9 / 15.9, 19.6 / 16.1, 34.8 / 17.1,
// x 4100 17.3 / 17.8, 21.4 / 17.8, 37.5 / 18.8, x 6000 20.9 / 19.8, 26.0 / 20.3, 45.7 / 21.2); 3584 x 8048 at 2 and 3 36.2 / 37.1, 42.9 / 39.3 (25.5 / 27.9, 29.7 / 28.6),
// 3584 x 14000 at 3 65 / 59 (39.5 / 40.6), 3584 x 8048 at 32 261 / 68.  Stacks gain more (1.3 times at two tokens of 3584, 3 - 5 times at 8 and 16 of 768 and
// 1536) but go the way of the lone call, whose bits they have.
static bool bat_pays(const clada_layer *layer, int B, bool list)
{
    const bool relu = layer->kind == CLADA_FFN_RELU;
    switch (layer->d) {
    case 1024: case 2048: case 2560: case 3072: case 4096: case 5120: case 6144: case 8192: return B >= 2;
    case 512: return B >= (relu ? 14 : 12);
    case 768: return B >= (relu ? 9 : 6);
    case 1536: return B >= (relu ? 5 : list || layer->d_ff < 3840 ? 5 : 4);
    case 3584: return B >= (relu ? 4 : 3);
    default: return false;
    }
}

// Passes over the weights of a batch, of nearly equal size: 16 tokens each, or 32 in two tiles where their x fits the registers and their h the
// room that a call of more than 16 tokens has beside its partial outputs (CLADA_BAT_WIDE floats).  0: not for this path.
int clada_batched_passes(const clada_layer *layer, int32_t B, bool list)
{
    if (layer->dtype != CLADA_BF16 || !bat_pays(layer, B, list)) return 0;
    const int most = B > 16 && layer->d <= 4096 && layer->d_ff <= 16 * (int64_t)layer->d ? 32 : 16;
    return (B + most - 1) / most;
}

// Launch shape of the batched path for a pass of B tokens in tiles of 16 of a layer it takes (clada_batched_passes); false when the shape is
// not eligible (decided by sizes alone, before anything is launched).
static bool bat_plan(const clada_ctx *ctx, const clada_layer *layer, int B, int tiles, int *P_out, int *CG_out, int *RG_out)
{
    const int d = layer->d, F = layer->d_ff;
    if (B < 1 || (B < 2 && tiles < 2) || B > 16 * tiles) return false;
    const int P = ctx->num_cu < COOP_MAX_WGS ? ctx->num_cu : COOP_MAX_WGS;
    const int CG = (d + DN_COLS - 1) / DN_COLS;
    int RG = P / CG;
    if (RG < 1) RG = 1;
    if (RG > 64) RG = 64;
    if (RG > 1 && (CG * RG) % 8 != 0 && (CG * (RG - 1)) % 8 == 0) --RG;     // a grid the XCD-aware map of the down kernel divides
    // row group rg = the neurons of the gate/up workgroups [rg P / RG, (rg+1) P / RG)
    auto group_fits = [&](int rgs) {
        if (rgs > P) return false;
        for (int rg = 0; rg < rgs; ++rg) {
            const int w0 = (int)((long long)rg * P / rgs), w1 = (int)((long long)(rg + 1) * P / rgs);
            if (w1 - w0 > DN_MAX_WGS || bat_run_lo(w1, F, P) - bat_run_lo(w0, F, P) > DN_MAX_ROWS) return false;
        }
        return true;
    };
    while (!group_fits(RG) && RG < 64) RG *= 2;                         // wide layers: more, smaller row groups
    if (!group_fits(RG)) return false;
    *P_out = P; *CG_out = CG; *RG_out = RG;
    return true;
}

// Bytes of partial outputs that a lane of the whole-stack calls has room for in front of a pass's scratch: 64 x 16 rows of fp32
// (CLADA_BAT_WIDE floats a column in two tiles).
size_t clada_ws_decode_batched_partial(int32_t d)
{
    return align_up(sizeof(float) * 64 * 16 * (size_t)d, 256);
}

// Whether a pass can go round the lanes.  A lone pass has room for 512 rows a token; very wide layers whose row groups were doubled past 64
// (72 of 3584 x 66000, 84 of 1536 x 76000, 96 of 5120 x 99000) write more than a lane holds once the pass has tokens enough.
bool clada_decode_batched_fits_lane(const clada_ctx *ctx, const clada_layer *layer, int32_t B, int tiles)
{
    int P, CG, RG;
    return bat_plan(ctx, layer, B, tiles, &P, &CG, &RG) && RG * B <= (tiles == 2 ? CLADA_BAT_WIDE : 64 * 16);
}

// Launches the two kernels for n_layers layers in n_pass passes of tokens: args are BatArgs, or BatParams p for a single unit
// (the only one that may have a list).
template <class Args>
static clada_status bat_launch(clada_ctx *ctx, const Args &args, const BatParams &p, int n_pass, int n_layers, bool relu, bool dense,
                               hipStream_t stream)
{
    constexpr bool LONE = std::is_same_v<Args, BatParams>;
    const int d = p.d;
    const bool list = p.list != nullptr;
    const dim3 grid(p.P, n_pass, n_layers);
#define CLADA_BAT_LAUNCH(KS, NW, RELU, MT)                                                                                                \
    {                                                                                                                                      \
        if (list)       hipLaunchKernelGGL((k_bat_gateup<KS, NW, true, LONE, RELU, MT, Args>), grid, dim3(NW * 64), 0, stream, args);   \
        else if (dense) hipLaunchKernelGGL((k_bat_gateup<KS, NW, true, false, RELU, MT, Args>), grid, dim3(NW * 64), 0, stream, args);  \
        else            hipLaunchKernelGGL((k_bat_gateup<KS, NW, false, false, RELU, MT, Args>), grid, dim3(NW * 64), 0, stream, args); \
    }
#define CLADA_BAT_CASE(D, KS, NW, MT)                                                                        \
    if (d == D && p.mt == MT) {                                                                               \
        static_assert(D == NW * 32 * KS, "waves x k-steps x 32 = d");                                         \
        if (relu) CLADA_BAT_LAUNCH(KS, NW, true, MT) else CLADA_BAT_LAUNCH(KS, NW, false, MT)                 \
    }
    CLADA_BAT_CASE(1024, 4, 8, 1) CLADA_BAT_CASE(2048, 8, 8, 1) CLADA_BAT_CASE(2560, 16, 5, 1) CLADA_BAT_CASE(3072, 12, 8, 1)
    CLADA_BAT_CASE(4096, 16, 8, 1) CLADA_BAT_CASE(5120, 32, 5, 1) CLADA_BAT_CASE(6144, 24, 8, 1) CLADA_BAT_CASE(8192, 32, 8, 1)
    CLADA_BAT_CASE(1024, 4, 8, 2) CLADA_BAT_CASE(2048, 8, 8, 2) CLADA_BAT_CASE(2560, 16, 5, 2) CLADA_BAT_CASE(3072, 12, 8, 2)
    CLADA_BAT_CASE(4096, 16, 8, 2) CLADA_BAT_CASE(512, 4, 4, 2) CLADA_BAT_CASE(768, 6, 4, 2) CLADA_BAT_CASE(1536, 6, 8, 2)
    CLADA_BAT_CASE(3584, 14, 8, 2) CLADA_BAT_CASE(512, 4, 4, 1) CLADA_BAT_CASE(768, 6, 4, 1) CLADA_BAT_CASE(1536, 6, 8, 1)
    CLADA_BAT_CASE(3584, 14, 8, 1)
#undef CLADA_BAT_LAUNCH
#undef CLADA_BAT_CASE
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    const size_t lds = 8 * (size_t)DN_TILE_BYTES + sizeof(int) * DN_MAX_ROWS;
    static std::atomic<bool> attr_set[4];                               // set once per process and kernel (two first callers may both set it)
    const bool whole = whole_h(d);
    const auto down = p.mt == 2 ? (whole ? k_bat_down<2, true, Args> : k_bat_down<2, false, Args>)
                                : (whole ? k_bat_down<1, true, Args> : k_bat_down<1, false, Args>);
    std::atomic<bool> &set = attr_set[2 * (p.mt - 1) + whole];
    if (!set.load(std::memory_order_relaxed)) {
        CLADA_CHECK_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(down), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        set.store(true, std::memory_order_relaxed);
    }
    hipLaunchKernelGGL(down, dim3(p.CG * p.RG, n_pass, n_layers), dim3(512), lds, stream, args);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    return CLADA_OK;
}

// The layers of a whole-stack call in launches of up to 48 units (layer, pass of tokens), or as many layers as `bytes` of scratch
// hold (*ran: the shape fits and did).  Three launches against three lanes of three launches per unit, us per step: 180 / 307 for
// 24 layers of 1024 x 4096 at two tokens, 395 / 466 for 18 of 2048 x 8192 at 16, 243 / 277 for 5 of 4096 x 11008 at 4, 940 / 999
// for 20 of 5120 x 8192 at 16, 2313 / 2415 for 40 of 5120 x 13824 at two.  What they save is ends: long stacks of large layers have
// few of them for their size, and there a second unit's kernels in the gaps of the first one's are worth 1 - 4 % (2822 / 2718 for
// 40 of 4096 x 16384 at 16 tokens, 5350 / 5168 for 40 of 8192 x 16384, 2952 / 2932 for 40 of 5120 x 13824; but 1492 / 1503 for 20
// of the latter, 1829 / 1845 for 40 of 4096 x 11056 at 8 and 0.96 of the lanes' time at two tokens).  More units a launch gain
// nothing (2809 us at 48, 3031 at 80, lanes 2928: 40 layers of 5120 x 5120 at 32 tokens).
constexpr int BAT_UNITS = 48;
clada_status clada_stack_batched(clada_ctx *ctx, const clada_layer *layers, int32_t L, const void *x, int32_t B,
                                 const float *tau, void *y, bool dense, char *scratch, size_t bytes, hipStream_t stream, bool *ran)
{
    *ran = false;
    const int d = layers[0].d, F = layers[0].d_ff;
    const int n_pass = clada_batched_passes(&layers[0], B), per = n_pass ? (B + n_pass - 1) / n_pass : 0, mt = per > 16 ? 2 : 1;
    const int n16 = (B + 15) / 16;                           // (the rule below is by passes of 16)
    const double layer_bytes = (layers[0].kind == CLADA_FFN_RELU ? 2.0 : 3.0) * F * d * 2;
    if (L < 2 || n_pass == 0 || ((B + n16 - 1) / n16 > 4 && layer_bytes > 340e6 && layer_bytes * L * n16 > 12e9)) return CLADA_OK;
    int P, CG, RG;
    if (!bat_plan(ctx, &layers[0], B - (n_pass - 1) * per, mt, &P, &CG, &RG) || !bat_plan(ctx, &layers[0], per, mt, &P, &CG, &RG)) return CLADA_OK;
    const size_t part = sizeof(float) * (size_t)RG * B * d;
    const size_t per_layer = part + n_pass * (sizeof(float) * 16 * mt * (size_t)F + sizeof(int) * ((size_t)F + COOP_MAX_WGS));
    int nl = bytes < 768 ? 0 : (int)((bytes - 768) / per_layer < (size_t)L ? (bytes - 768) / per_layer : (size_t)L);
    if (nl > BAT_UNITS / n_pass) nl = BAT_UNITS / n_pass;
    if (nl < 2) return CLADA_OK;
    const int n_launch = (L + nl - 1) / nl;
    nl = (L + n_launch - 1) / n_launch;
    const bool relu = layers[0].kind == CLADA_FFN_RELU;
    char *hb = scratch + align_up(part * nl, 256);
    char *ul = hb + align_up(sizeof(float) * 16 * mt * (size_t)F * n_pass * nl, 256);
    char *uc = ul + align_up(sizeof(int) * (size_t)F * n_pass * nl, 256);
    for (int l0 = 0; l0 < L; l0 += nl) {
        const int n = L - l0 < nl ? L - l0 : nl;
        const size_t row = (size_t)l0 * B;
        BatArgs a;
        memset(&a, 0, sizeof(a));
        BatParams &p = a.p;
        p.x = (const char *)x + row * d * 2; p.tau = tau ? tau + row : nullptr;
        p.hbuf = reinterpret_cast<unsigned int *>(hb); p.ulist = reinterpret_cast<int *>(ul); p.ucnt = reinterpret_cast<int *>(uc);
        p.partial = reinterpret_cast<float *>(scratch);
        p.d = d; p.F = F; p.B = B; p.P = P; p.RG = RG; p.CG = CG; p.rows = n * B; p.mt = mt;
        p.gelu = layers[0].kind == CLADA_FFN_GEGLU ? 1 : 0;
        a.n_pass = n_pass; a.per_pass = per;
        bool bias = false;
        for (int l = 0; l < n; ++l) {
            const clada_layer &s = layers[l0 + l];
            a.wg[l] = (const char *)s.w_gate; a.wu[l] = (const char *)s.w_up; a.wd[l] = (const char *)s.w_down;
            a.b_in[l] = s.b_in;
            bias = bias || (relu && s.b_out);
        }
        const clada_status st = bat_launch(ctx, a, p, n_pass, n, relu, dense, stream);
        if (st != CLADA_OK) return st;
        char *y0 = (char *)y + row * d * 2;
        if (!bias) {
            clada_launch_finalize(2, p.partial, RG, n * B, d, y0, stream);
        } else {
            BatBiasArgs f;
            memset(&f, 0, sizeof(f));
            f.partial = p.partial; f.y = y0; f.RG = RG; f.B = B; f.d = d;
            for (int l = 0; l < n; ++l) f.b_out[l] = layers[l0 + l].b_out;
            hipLaunchKernelGGL(k_bat_finalize_bias, dim3((d + 31) / 32, n * B), dim3(256), 0, stream, f);
        }
        CLADA_CHECK_HIP(ctx, hipGetLastError());
    }
    *ran = true;
    return CLADA_OK;
}

// Runs the batched MFMA path for a pass of B tokens in tiles of 16 when the shape is eligible (*ran; an ineligible shape launches nothing
// and the caller uses the generic kernels).
clada_status clada_decode_batched(clada_ctx *ctx, const clada_layer *layer, const void *x, int32_t B,
                                  const float *tau, void *y, unsigned char *keep, float *partial,
                                  char *scratch, bool dense, hipStream_t stream, bool *ran, int tiles,
                                  const int32_t *list, const int32_t *list_n)
{
    *ran = false;
    const int d = layer->d, F = layer->d_ff;
    int P, CG, RG;
    if (!bat_plan(ctx, layer, B, tiles, &P, &CG, &RG)) return CLADA_OK;

    BatParams p;
    p.wg = (const char *)layer->w_gate; p.wu = (const char *)layer->w_up; p.wd = (const char *)layer->w_down;
    p.b_in = layer->b_in;
    p.x = (const char *)x; p.tau = tau;
    p.hbuf = reinterpret_cast<unsigned int *>(scratch);
    const size_t h_bytes = align_up(sizeof(float) * 16 * tiles * (size_t)F, 256);
    p.ulist = reinterpret_cast<int *>(scratch + h_bytes);
    p.ucnt = reinterpret_cast<int *>(scratch + h_bytes + align_up(sizeof(int) * (size_t)F, 256));
    p.mt = tiles;
    p.keep = keep; p.partial = partial;
    p.d = d; p.F = F; p.B = B; p.P = P; p.RG = RG; p.CG = CG; p.row0 = 0; p.rows = B;
    p.gelu = layer->kind == CLADA_FFN_GEGLU ? 1 : 0;
    const bool relu = layer->kind == CLADA_FFN_RELU;
    p.list = list; p.list_n = list_n;
    const clada_status st = bat_launch(ctx, p, p, 1, 1, relu, dense, stream);
    if (st != CLADA_OK) return st;
    clada_launch_finalize(2, partial, RG, B, d, (char *)y, stream, relu ? layer->b_out : nullptr);
    CLADA_CHECK_HIP(ctx, hipGetLastError());
    *ran = true;
    return CLADA_OK;
}
