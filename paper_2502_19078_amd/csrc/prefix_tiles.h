// Pipelined bf16 tile products of the prefill GEMMs: C = X W with fp32 accumulation, a persistent workgroup of eight waves per
// compute unit that walks its tiles while one stream of direct-to-LDS transfers runs on across them.
//
// What bounds it: the card's power limit and the L2 -> LDS transfers (one 256 x 256 tile takes 64 KiB of operands per 64-deep
// k-tile).  Measured on the way here (8192^3, random operands, us; the former kernel, four waves of 128 x 128, 32-deep k-tiles: 1120):
//   transfers of 64-byte row pieces (32-deep k-tiles) fetch every 128-byte line twice: 15 TB/s into LDS; whole lines 24.  950 -> 850
//     together with the next point
//   16x16x32 products in place of 32x32x16: the same peak rate, but 2046 against 1776 TFLOP/s under the power limit with operands
//     held in registers; serpentine order over the fragments is worth another 2 % of that
//   two groups of four waves, one per SIMD each, half a k-tile apart: one group's fragment reads run under the other's products
//     (one barrier per step keeps the distance).  Without the distance 985
//   transfers issued between the products instead of next to the reads: 757 -> 745
#pragma once
#include <type_traits>
#include <utility>

#include "clada_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((address_space(3))) char lds_char;

// WM x (8 / WM) waves of 64 x 32 NB outputs; D k-tiles in flight.  X tiles ([TM rows][64 k], 128 bytes a row) ring over D slots, W tiles
// over D + 1.  TR = false: W as it lies for the gate / up product, [TN rows][64 k]; TR = true: [64 k][TN columns], read transposed.
// WHOLE: a group reads and multiplies a whole k-tile between barriers, else half of one: for the smallest tile, whose half is eight
// products (128 clocks) a wave (gate/up of 333 x 2560 x 10240 ReLU 42 -> 38 us with its reduction; 128 x 128 neurons, sixteen
// products a half: 66 -> 72 at 200 x 4096 x 11008).
template <int WM_, int NB_, int D_, bool TR_, bool WHOLE_ = false>
struct TileShape {
    static constexpr int WM = WM_, NB = NB_, D = D_, WN = 8 / WM, TM = 64 * WM, TN = 32 * NB * WN;
    static constexpr bool TR = TR_, WHOLE = WHOLE_;
    static constexpr int XB = TM * 128, WB = TN * 128, LDS = D * XB + (D + 1) * WB;
    static constexpr int PX = TM / 64, PW = TN / 64;        // 1 KiB transfers of a wave per k-tile
    static_assert(LDS <= 160 * 1024 && 2 * NB >= PX && 2 * NB >= PW && (!TR || TN == 256), "tile shape");
};

// Operands of one output tile (uniform).  x / w: first row (TR: first k row at the tile's first column).  Transfers past the rows that
// exist deliver zeros: x_bytes, w_bytes count from x / w to their end; TR: w_rows k rows exist, of w_pitch bytes, the tile
// w_col bytes into them.
struct TileSrc {
    const char *x, *w;
    unsigned int x_bytes, w_bytes;
    int w_rows, w_pitch, w_col;
    int nk;                                                 // k-tiles
};

// f(0) .. f(N - 1) with the index as a constant.
template <class F, int... I>
__device__ __forceinline__ void unrolled_(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void unrolled(F &&f) { unrolled_(f, std::make_integer_sequence<int, N>{}); }

template <int N>
__device__ __forceinline__ void wait_vmcnt() { __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const char *p, unsigned int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00027000);
}

// A barrier that also orders the LDS accesses of the C++ code around it (not the transfers into LDS).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// tile(it, id): the it-th tile of this workgroup (uniform), false when there is none; src(id): its operands; x_pitch: bytes of an X row;
// vw[i]: byte offset of what this lane moves in transfer i of a W tile; epi(acc, id, scratch, wm, wn): what becomes of the
// products -- all eight waves run it together, `scratch` (an LDS byte address) has WB bytes.
// The LDS reads are inline assembly because the compiler would wait for every transfer in flight before them; their results are tied to
// the wait before anything else happens to them.
template <class S, class Tile, class Src, class Epi>
__device__ __forceinline__ void tile_products(char *lds, int x_pitch, const int (&vw)[S::PW], Tile &&tile, Src &&src, Epi &&epi)
{
    using Id = typename std::remove_reference<Tile>::type::Id;
    constexpr int TM = S::TM, NB = S::NB, D = S::D, XB = S::XB, WB = S::WB, PX = S::PX, PW = S::PW, WM = S::WM;
    constexpr int FLY = (D - 1) * (PX + PW);                // transfers of a wave that may be in flight at a wait
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave >> 2, w4 = wave & 3;
    const int wm = grp * (WM / 2) + w4 % (WM / 2), wn = w4 / (WM / 2);      // a group's X rows are its own

    Id id;
    if (!tile(0, id)) return;

    // ---- the stream of transfers: cursor (tile, k-tile), D k-tiles ahead of the products
    int ct = 0, ck = 0;
    TileSrc cs = src(id);
    const int xrow = grp * (TM / 2) + 8 * w4;
    int vx[PX];
#pragma unroll
    for (int i = 0; i < PX; ++i)                            // 8 rows a transfer; chunk c of row r lies at c ^ (r & 7)
        vx[i] = (xrow + 32 * i + (lane >> 3)) * x_pitch + ((lane & 7) ^ (lane >> 3)) * 16;
    auto send_x = [&](auto ic, int slot) {
        constexpr int i = decltype(ic)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(tile_rsrc(cs.x, cs.x_bytes),
            (void __attribute__((address_space(3))) *)((lds_char *)lds + slot + xrow * 128 + i * 4096), 16, vx[i], 0, 0, 0);
    };
    auto send_w = [&](auto ic, int slot) {
        constexpr int i = decltype(ic)::value;
        const unsigned int bytes = S::TR ? (unsigned int)(min(cs.w_rows, 64) * cs.w_pitch - cs.w_col) : cs.w_bytes;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(tile_rsrc(cs.w, bytes),
            (void __attribute__((address_space(3))) *)((lds_char *)lds + slot + wave * 1024 + i * 8192), 16, vw[i], 0, 0, 0);
    };
    auto advance = [&]() {
        if (++ck == cs.nk) {
            Id n;
            if (tile(ct + 1, n)) {
                ++ct;
                cs = src(n);
                ck = 0;
            } else {                                        // nothing left: the last k-tile again, into slots nobody reads any more
                --ck;
            }
        } else {
            cs.x += 128;
            cs.x_bytes -= 128;
            cs.w += S::TR ? (size_t)64 * cs.w_pitch : 128;
            if (S::TR) cs.w_rows -= 64;
            else cs.w_bytes -= 128;
        }
    };

    // ---- fragments
    const int r16 = lane & 15, q = lane >> 4;
    const unsigned int lds0 = (unsigned int)(size_t)(lds_char *)lds;
    const unsigned int xa = lds0 + (unsigned int)((wm * 64 + r16) * 128 + ((q ^ (r16 & 7)) * 16));
    const unsigned int wa = lds0 + (unsigned int)(D * XB + (wn * 32 * NB + r16) * 128 + ((q ^ (r16 & 7)) * 16));
    // TR: group q of 16 lanes takes k rows 8q .. 8q + 7 in two reads; lane t = 4 rr + c4 supplies row rr (then 4 + rr), columns 4 c4 ..,
    // and receives column t.  32-byte piece s of row r lies at s ^ ((r & 3) | (r >> 3 & 1) << 2): the eight rows that half a wave
    // reads come from different banks.
    const int rr = r16 >> 2, sw = rr | ((q & 1) << 2);
    const unsigned int ta = lds0 + (unsigned int)(D * XB + (8 * q + rr) * 512 + (r16 & 3) * 8);
    unsigned int tj[2 * NB];
#pragma unroll
    for (int j = 0; j < 2 * NB; ++j) tj[j] = ta + (unsigned int)(((wn * 2 * NB + j) ^ sw) * 32);
    constexpr int SETS = S::WHOLE ? 2 : 1;
    u32x4 fx[SETS][4], fw[SETS][2 * NB];
    u32x2 ft[SETS][2 * NB][2];
    auto read = [&](u32x4 (&fx)[4], u32x4 (&fw)[2 * NB], u32x2 (&ft)[2 * NB][2], unsigned int xs, unsigned int wslot, auto hc) {
        constexpr int H = decltype(hc)::value;              // half of the k-tile
        const unsigned int px = (xa ^ (unsigned int)(H * 64)) + xs, pw = (wa ^ (unsigned int)(H * 64)) + wslot;
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fx[i]) : "v"(px), "n"(i * 2048));
        if constexpr (!S::TR) {
#pragma unroll
            for (int j = 0; j < 2 * NB; ++j) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fw[j]) : "v"(pw), "n"(j * 2048));
        } else {
#pragma unroll
            for (int j = 0; j < 2 * NB; ++j) {
                const unsigned int pt = tj[j] + wslot;
                asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(ft[j][0]) : "v"(pt), "n"(H * 16384));
                asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(ft[j][1]) : "v"(pt), "n"(H * 16384 + 2048));
            }
        }
    };
    auto landed = [&](u32x4 (&fx)[4], u32x4 (&fw)[2 * NB], u32x2 (&ft)[2 * NB][2]) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fx[0]), "+v"(fx[1]), "+v"(fx[2]), "+v"(fx[3]));
#pragma unroll
        for (int j = 0; j < 2 * NB; ++j) {
            if constexpr (S::TR) asm volatile("" : "+v"(ft[j][0]), "+v"(ft[j][1]));
            else asm volatile("" : "+v"(fw[j]));
        }
    };
    // The products of half a k-tile, columns outer, rows there and back (a fragment is held from one product to the next), with N
    // transfers dealt out between them.
    auto products = [&](f32x4 (&acc)[4][2 * NB], const u32x4 (&fx)[4], const u32x4 (&fw)[2 * NB], const u32x2 (&ft)[2 * NB][2],
                        auto f, auto nc, int slot) {
        constexpr int N = decltype(nc)::value;
        unrolled<2 * NB>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const bf16x8 b = S::TR ? __builtin_bit_cast(bf16x8, u32x4{ft[j][0].x, ft[j][0].y, ft[j][1].x, ft[j][1].y})
                                   : __builtin_bit_cast(bf16x8, fw[j]);
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) {
                const int i = (j & 1) ? 3 - ii : ii;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fx[i]), b, acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (j < N) {
                f(jc, slot);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };

    using NX = std::integral_constant<int, PX>;
    using NW = std::integral_constant<int, PW>;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        unrolled<PW>([&](auto c) { send_w(c, D * XB + i * WB); });
        unrolled<PX>([&](auto c) { send_x(c, i * XB); });
        if (i + 1 < D) advance();
    }
    wait_vmcnt<FLY>();                                      // k-tile 0 has landed
    __builtin_amdgcn_s_barrier();
    int xs = 0, ws = 0, wf = D * WB;                        // slots read, slot to be filled
    for (int it = 0; tile(it, id); ++it) {
        f32x4 acc[4][2 * NB];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2 * NB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        const int nk = src(id).nk;
        if (grp == 1) __builtin_amdgcn_s_barrier();         // half a k-tile behind the other group
        for (int k = 0; k < nk; ++k) {
#define TILE_SB __builtin_amdgcn_sched_barrier(0);
            using H0 = std::integral_constant<int, 0>;
            using H1 = std::integral_constant<int, 1>;
            constexpr int L = SETS - 1;                     // fragment set of the second half
            TILE_SB
            read(fx[0], fw[0], ft[0], xs, ws, H0{});
            if constexpr (S::WHOLE) {
                read(fx[L], fw[L], ft[L], xs, ws, H1{});
                wait_vmcnt<FLY - PW>();                     // this wave's part of the next W tile
            }
            advance();
            landed(fx[0], fw[0], ft[0]);
            if constexpr (S::WHOLE) landed(fx[L], fw[L], ft[L]);
            TILE_SB
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_s_setprio(1);
            TILE_SB
            products(acc, fx[0], fw[0], ft[0], send_w, NW{}, D * XB + wf);      // the slot that both groups left a k-tile ago
            TILE_SB
            if constexpr (!S::WHOLE) {
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_s_barrier();
                TILE_SB
                read(fx[0], fw[0], ft[0], xs, ws, H1{});
                wait_vmcnt<FLY>();                          // this wave's part of the next W tile
                landed(fx[0], fw[0], ft[0]);
                TILE_SB
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_s_setprio(1);
                TILE_SB
            }
            products(acc, fx[L], fw[L], ft[L], send_x, NX{}, xs);       // the rows that this group has just read for the last time
            TILE_SB
            __builtin_amdgcn_s_setprio(0);
            wait_vmcnt<FLY>();                              // and of the next X tile
            __builtin_amdgcn_s_barrier();
            TILE_SB
            xs = xs == (D - 1) * XB ? 0 : xs + XB;
            ws = ws == D * WB ? 0 : ws + WB;
            wf = wf == D * WB ? 0 : wf + WB;
        }
        if (grp == 0) __builtin_amdgcn_s_barrier();         // both groups together again
        epi(acc, id, (unsigned int)(lds0 + D * XB + wf), wm, wn);
    }
#undef TILE_SB
    wait_vmcnt<0>();                                        // nothing may land in LDS after the workgroup has left
}

// One fp32 value to / from the scratch of an epilogue (inline assembly for the reason above).
__device__ __forceinline__ void scratch_put(unsigned int addr, float v) { asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ float scratch_get(unsigned int addr)
{
    float v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr) : "memory");
    return v;
}

// The it-th of `total` tiles for this workgroup of `blocks`: consecutive workgroup ids lie on different XCDs, so each XCD gets a
// run of tiles of its own (in the order of tile_coords, so that the tiles an XCD has in hand share operands in its L2).
__device__ __forceinline__ int tile_order(int it, int blocks, int total)
{
    const int per = (total + 7) >> 3, o = (int)(blockIdx.x >> 3) + it * (blocks >> 3);
    const int t = (int)(blockIdx.x & 7) * per + o;
    return o < per && t < total ? t : -1;
}
// Tiles in bands of eight token tiles, token tile fastest: 32 tiles in a row are 8 x 4, twelve operand slices for 32 products.
__device__ __forceinline__ void tile_coords(int o, int n_tm, int n_tn, int &tm, int &tn)
{
    const int band = o / (8 * n_tn), left = n_tm - 8 * band, h = left < 8 ? left : 8;
    const int w = o - band * 8 * n_tn;
    tm = 8 * band + w % h;
    tn = w / h;
}

}  // namespace
