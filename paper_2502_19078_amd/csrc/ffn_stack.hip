// The batch-1 layers of a whole-stack call as ONE launch over (class of neurons, layer), for gfx950.
//
// The layers of a stack are independent problems, so nothing but the hardware's workgroup dispatcher has to order
// them: workgroups of layer l + 1 take the places that those of layer l leave, the weight stream never drains and a
// step pays for two launches instead of two per layer.
//
// Order of summation.  The per-layer kernel (k_ffn_decode_b1 without balancing) deals the neurons of a layer to 256
// partial outputs -- neuron j belongs to class j mod 256, a class adds its kept neurons in ascending order -- and the
// reduction adds the classes q, q + 32, .., q + 224 one after the other into slice q, then the 32 slices by a fixed
// tree.  Here a workgroup takes either one class, or all eight classes of a slice one after the other (CHAIN): it
// closes a class by adding its accumulators to the slice's sum, so both forms give the per-layer call's bits.
#include "clada_internal.h"

namespace {

constexpr int CLASSES = 256, SLICES = 32, CHAIN = CLASSES / SLICES;

struct StackLaunch {                        // kernel argument; the tables are read by scalar loads at the layer's index
    const char *wg[CLADA_STACK_LAUNCH_LAYERS], *wu[CLADA_STACK_LAUNCH_LAYERS], *wd[CLADA_STACK_LAUNCH_LAYERS];
    const float *b_in[CLADA_STACK_LAUNCH_LAYERS];
    const char *x;                          // [n][d]
    const float *tau;                       // [n] (unused when dense)
    float *partial;                         // [n][256 / chain][d]
    int F, d, chain, dense, gelu;
};
typedef const __attribute__((address_space(4))) StackLaunch *StackLaunchArgs;

// Per row length (NCH chunks of 1 KiB): the workgroup's waves and a wave's ring in LDS, two units of UC loads of 1 KiB.  A
// unit is half a row, a row or two short rows; for the down projection UC * EPL kept rows of the wave's columns (one or half
// a KiB).  The waves of a compute unit keep about 100 KiB of weight rows in flight; 7 TB/s take 55 KiB at 2 us of loaded
// latency.  (Four waves for 2 KiB rows: 62 us per step of 24 layers of 8 MB against 67 us with eight.)  Rows of 1 and 3 KiB have
// two waves for every KiB as well; units of three loads serve the rows of 3 and 6 KiB, rows of 7 KiB go whole.
template <int NCH> struct RowShape {
    static constexpr int NW = NCH < 4 ? 2 * NCH : NCH;
    static constexpr int UC = NCH % 5 == 0 ? 5 : NCH == 3 || NCH == 6 ? 3 : NCH == 7 ? 7 : 4;
    static constexpr int RD = 2;                             // units of a ring
    static constexpr int R = UC > NCH ? UC / NCH : 1;        // rows per gate / up unit
    static constexpr int PARTS = NCH > UC ? NCH / UC : 1;    // units per row
    static constexpr int CWB = NCH * 1024 / NW;              // bytes of a row's columns per wave
    static constexpr int EPL = 1024 / CWB;                   // kept rows per down-projection load
    static_assert((R * NCH == UC || PARTS * UC == NCH) && (EPL == 1 || EPL == 2), "whole rows or whole parts");
};

__device__ __forceinline__ unsigned int lds_offset(const void *p)
{
    return (unsigned int)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
// Loads into LDS and the reads of what they bring are written as assembly: the compiler cannot tell the ring's slots apart
// and would wait for every load in flight before any LDS access.  A load has no register result; its slot is read only
// after the wait for the vector-memory counter below, and is refilled only after that read has returned.  The slot's address
// reaches m0 through its constraint, so the compiler knows what m0 holds.
// The base is the same in every lane, but the compiler is free to compute it in vector registers (it does for some row lengths), and a scalar register
// that a vector instruction has written may be a load's base five wait states later at the earliest, which the assembler does not see to.
// So the load reads a copy that a scalar instruction makes right before it, which the hardware waits for; that is also the wait state behind m0.
__device__ __forceinline__ void ring_load(const char *base, unsigned int voff, unsigned int slot)
{
    const unsigned long long b = (unsigned long long)base;
    const unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)b), hi = __builtin_amdgcn_readfirstlane((unsigned int)(b >> 32));
    unsigned long long copy;
    asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0 nt" : "=&s"(copy) : "v"(voff), "s"(((unsigned long long)hi << 32) | lo), "{m0}"(slot) : "memory");
}
__device__ __forceinline__ void ring_load_lanes(const char *p, unsigned int slot)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(p), "{m0}"(slot) : "memory");
}
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
template <int DW> struct RingWords;
template <> struct RingWords<4> { typedef u32x4 type; };
template <> struct RingWords<2> { typedef u32x2 type; };
// N slots of a unit and the N matching chunks of x; N slots of a unit.
template <int N> __device__ void ring_read_x(unsigned int a, unsigned int b, u32x4 (&w)[N], u32x4 (&x)[N]);
template <int N, int DW> __device__ void ring_read(unsigned int a, typename RingWords<DW>::type (&w)[N]);
template <> __device__ __forceinline__ void ring_read_x<4>(unsigned int a, unsigned int b, u32x4 (&w)[4], u32x4 (&x)[4])
{
    asm volatile("ds_read_b128 %0, %8 offset:0\n\t"
                 "ds_read_b128 %4, %9 offset:0\n\t"
                 "ds_read_b128 %1, %8 offset:1024\n\t"
                 "ds_read_b128 %5, %9 offset:1024\n\t"
                 "ds_read_b128 %2, %8 offset:2048\n\t"
                 "ds_read_b128 %6, %9 offset:2048\n\t"
                 "ds_read_b128 %3, %8 offset:3072\n\t"
                 "ds_read_b128 %7, %9 offset:3072\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])
                 : "v"(a), "v"(b) : "memory");
}
template <> __device__ __forceinline__ void ring_read_x<5>(unsigned int a, unsigned int b, u32x4 (&w)[5], u32x4 (&x)[5])
{
    asm volatile("ds_read_b128 %0, %10 offset:0\n\t"
                 "ds_read_b128 %5, %11 offset:0\n\t"
                 "ds_read_b128 %1, %10 offset:1024\n\t"
                 "ds_read_b128 %6, %11 offset:1024\n\t"
                 "ds_read_b128 %2, %10 offset:2048\n\t"
                 "ds_read_b128 %7, %11 offset:2048\n\t"
                 "ds_read_b128 %3, %10 offset:3072\n\t"
                 "ds_read_b128 %8, %11 offset:3072\n\t"
                 "ds_read_b128 %4, %10 offset:4096\n\t"
                 "ds_read_b128 %9, %11 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4])
                 : "v"(a), "v"(b) : "memory");
}
template <> __device__ __forceinline__ void ring_read<4, 2>(unsigned int a, RingWords<2>::type (&w)[4])
{
    asm volatile("ds_read_b64 %0, %4 offset:0\n\t"
                 "ds_read_b64 %1, %4 offset:1024\n\t"
                 "ds_read_b64 %2, %4 offset:2048\n\t"
                 "ds_read_b64 %3, %4 offset:3072\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(a) : "memory");
}
template <> __device__ __forceinline__ void ring_read<4, 4>(unsigned int a, RingWords<4>::type (&w)[4])
{
    asm volatile("ds_read_b128 %0, %4 offset:0\n\t"
                 "ds_read_b128 %1, %4 offset:1024\n\t"
                 "ds_read_b128 %2, %4 offset:2048\n\t"
                 "ds_read_b128 %3, %4 offset:3072\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(a) : "memory");
}
template <> __device__ __forceinline__ void ring_read<5, 4>(unsigned int a, RingWords<4>::type (&w)[5])
{
    asm volatile("ds_read_b128 %0, %5 offset:0\n\t"
                 "ds_read_b128 %1, %5 offset:1024\n\t"
                 "ds_read_b128 %2, %5 offset:2048\n\t"
                 "ds_read_b128 %3, %5 offset:3072\n\t"
                 "ds_read_b128 %4, %5 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4])
                 : "v"(a) : "memory");
}

template <> __device__ __forceinline__ void ring_read_x<3>(unsigned int a, unsigned int b, u32x4 (&w)[3], u32x4 (&x)[3])
{
    asm volatile("ds_read_b128 %0, %6 offset:0\n\t"
                 "ds_read_b128 %3, %7 offset:0\n\t"
                 "ds_read_b128 %1, %6 offset:1024\n\t"
                 "ds_read_b128 %4, %7 offset:1024\n\t"
                 "ds_read_b128 %2, %6 offset:2048\n\t"
                 "ds_read_b128 %5, %7 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2])
                 : "v"(a), "v"(b) : "memory");
}
template <> __device__ __forceinline__ void ring_read_x<7>(unsigned int a, unsigned int b, u32x4 (&w)[7], u32x4 (&x)[7])
{
    asm volatile("ds_read_b128 %0, %14 offset:0\n\t"
                 "ds_read_b128 %7, %15 offset:0\n\t"
                 "ds_read_b128 %1, %14 offset:1024\n\t"
                 "ds_read_b128 %8, %15 offset:1024\n\t"
                 "ds_read_b128 %2, %14 offset:2048\n\t"
                 "ds_read_b128 %9, %15 offset:2048\n\t"
                 "ds_read_b128 %3, %14 offset:3072\n\t"
                 "ds_read_b128 %10, %15 offset:3072\n\t"
                 "ds_read_b128 %4, %14 offset:4096\n\t"
                 "ds_read_b128 %11, %15 offset:4096\n\t"
                 "ds_read_b128 %5, %14 offset:5120\n\t"
                 "ds_read_b128 %12, %15 offset:5120\n\t"
                 "ds_read_b128 %6, %14 offset:6144\n\t"
                 "ds_read_b128 %13, %15 offset:6144\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6])
                 : "v"(a), "v"(b) : "memory");
}
template <> __device__ __forceinline__ void ring_read<3, 2>(unsigned int a, RingWords<2>::type (&w)[3])
{
    asm volatile("ds_read_b64 %0, %3 offset:0\n\t"
                 "ds_read_b64 %1, %3 offset:1024\n\t"
                 "ds_read_b64 %2, %3 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2])
                 : "v"(a) : "memory");
}
template <> __device__ __forceinline__ void ring_read<3, 4>(unsigned int a, RingWords<4>::type (&w)[3])
{
    asm volatile("ds_read_b128 %0, %3 offset:0\n\t"
                 "ds_read_b128 %1, %3 offset:1024\n\t"
                 "ds_read_b128 %2, %3 offset:2048\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2])
                 : "v"(a) : "memory");
}
template <> __device__ __forceinline__ void ring_read<7, 4>(unsigned int a, RingWords<4>::type (&w)[7])
{
    asm volatile("ds_read_b128 %0, %7 offset:0\n\t"
                 "ds_read_b128 %1, %7 offset:1024\n\t"
                 "ds_read_b128 %2, %7 offset:2048\n\t"
                 "ds_read_b128 %3, %7 offset:3072\n\t"
                 "ds_read_b128 %4, %7 offset:4096\n\t"
                 "ds_read_b128 %5, %7 offset:5120\n\t"
                 "ds_read_b128 %6, %7 offset:6144\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6])
                 : "v"(a) : "memory");
}

// One workgroup streams the rows of its neurons through per-wave rings in LDS.  Round r = 64 neurons: G(r) their gate rows
// (whole rows, dealt to the waves), U(r) the W_up rows of those kept (likewise), D(r) the kept W_down rows, of which every
// wave takes its own columns.  A wave loads and consumes in the order G0 G1 U0 D0 G2 U1 D1 ..: the list of round r is known
// (barrier) while the rows of G(r + 1) are in flight, and the exchange of h (barrier) happens while D(r) is, so the stream
// of loads never waits for either.
template <int ES, int NCH, bool RELU>
__global__ void __launch_bounds__(RowShape<NCH>::NW * 64)
k_ffn_stack(const StackLaunch)
{
    typedef RowShape<NCH> S;
    constexpr int NW = S::NW, RD = S::RD, UC = S::UC, R = S::R, PARTS = S::PARTS, CWB = S::CWB, EPL = S::EPL;
    constexpr int ROWB = NCH * 1024, UNIT = UC * 1024;
    constexpr int DW = CWB / 256, VEC = 4 * DW / ES;          // words / values of a kept row per lane
    constexpr int EPU = UC * EPL;                             // kept rows per down-projection unit
    __shared__ __align__(16) unsigned char s_ring[NW][RD][UNIT];
    __shared__ __align__(16) unsigned char s_x[ROWB];
    __shared__ float s_a[2][64];
    __shared__ int s_keep[2][64];
    __shared__ int s_lrow[2][64], s_lcls[2][64];
    __shared__ float s_la[2][64], s_h[2][64];

    const StackLaunchArgs ka = (StackLaunchArgs)__builtin_amdgcn_kernarg_segment_ptr();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int layer = blockIdx.y, group = blockIdx.x, chain = ka->chain;
    const int F = ka->F, dense = ka->dense, gelu = ka->gelu;
    const char *wg = ka->wg[layer], *wu = ka->wu[layer], *wd = ka->wd[layer];
    const __attribute__((address_space(4))) float *b_in = (const __attribute__((address_space(4))) float *)(RELU ? ka->b_in[layer] : nullptr);
    const char *xg = ka->x + (size_t)layer * ROWB;
    const unsigned int loff = lane * 16;
    const unsigned int ring0 = lds_offset(&s_ring[0][0][0]) + wave * (RD * UNIT), x0 = lds_offset(s_x);

    for (int c = wave; c < NCH; c += NW) ring_load(xg + c * 1024, loff, x0 + c * 1024);

    // local neuron i = (class i / per, position i % per) of this workgroup: neuron group + 32 class + 256 position
    // when it takes a whole slice, group + 256 i when it takes one class
    const int per = (F + CLASSES - 1) / CLASSES, n_local = per * chain, n_round = (n_local + 63) / 64;
    auto neuron_of = [&](int i) -> int {                     // -1: none
        const int cls = i / per, j = group + SLICES * cls + CLASSES * (i - cls * per);
        return i < n_local && j < F ? j : -1;
    };

    // ---------------------------------------------------------------- the loading side: one unit per call
    int jv_load = neuron_of(lane);                           // neurons of the round whose gate rows are being requested
    int ph = 0, lr = 0, li = wave, lp = 0;                   // phase (0 G, 1 U, 2 D, 3 end), its round, row / entry, part
    int lim = min(64, n_local);                              // rows / entries of the phase
    int n_list = 0;                                          // rounds whose list is known
    int kp2[2] = {0, 0};                                     // kept neurons of the last two of them
    int n_fly = 0, head = 0;                                 // units in flight, next to fill
    auto load_unit = [&]() -> bool {
        for (;;) {
            if (lim < 0) {                                   // the list decides
                if (lr >= n_list) return false;              // not known yet: come back later
                lim = kp2[lr & 1];
            }
            if (li < lim) break;
            if (ph == 0) {                                   // after G(lr): U(lr - 1); after G(0) the next round's rows
                if (lr == 0 && n_round > 1) {
                    lr = 1; li = wave; jv_load = neuron_of(64 + lane); lim = min(64, n_local - 64);
                } else {
                    lr = max(lr - 1, 0); ph = RELU ? 2 : 1; li = RELU ? 0 : wave; lim = -1;
                }
            } else if (ph == 1) {
                ph = 2; li = 0;
            } else if (ph == 2) {                            // after D(lr): G(lr + 2), or what is left of the last rounds
                if (lr + 2 < n_round) {
                    lr += 2; ph = 0; li = wave; jv_load = neuron_of(64 * lr + lane); lim = min(64, n_local - 64 * lr);
                } else if (lr + 1 < n_round) {
                    lr += 1; ph = RELU ? 2 : 1; li = RELU ? 0 : wave; lim = -1;
                } else {
                    ph = 3; lim = 0;
                }
            } else {
                return false;
            }
        }
        const unsigned int slot = ring0 + head * UNIT;
        if (ph < 2) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int i = li + NW * q;
                const char *row = xg;                        // past the end, or no such neuron: x instead
                if (ph == 0) {
                    const int j = __builtin_amdgcn_readlane(jv_load, i & 63);
                    if (i < lim && j >= 0) row = wg + (size_t)j * ROWB;
                } else if (i < lim) {
                    row = wu + (size_t)__builtin_amdgcn_readfirstlane(s_lrow[lr & 1][i]) * ROWB;
                }
#pragma unroll
                for (int c = 0; c < UC / R; ++c) ring_load(row + lp * UNIT + c * 1024, loff, slot + (q * (UC / R) + c) * 1024);
            }
            if (++lp == PARTS) { lp = 0; li += NW * R; }
        } else {
            const int kp = lim;
            if constexpr (EPL == 1) {
#pragma unroll
                for (int q = 0; q < UC; ++q) {
                    const int e = min(li + q, kp - 1);
                    ring_load(wd + (size_t)__builtin_amdgcn_readfirstlane(s_lrow[lr & 1][e]) * ROWB + wave * CWB, loff, slot + q * 1024);
                }
            } else {                                         // EPL rows per load, the lanes shared out
                constexpr int LPR = 64 / EPL;
#pragma unroll
                for (int q = 0; q < UC; ++q) {
                    const int e = min(li + q * EPL + lane / LPR, kp - 1);
                    ring_load_lanes(wd + (size_t)s_lrow[lr & 1][e] * ROWB + wave * CWB + (lane % LPR) * 16, slot + q * 1024);
                }
            }
            li += EPU;
        }
        head = head + 1 == RD ? 0 : head + 1;
        ++n_fly;
        return true;
    };
    // ---------------------------------------------------------------- the consuming side, in the same order
    int tail = 0;
    auto wait_oldest = [&]() -> unsigned int {
        if (n_fly == RD) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RD - 1) * UC) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const unsigned int slot = ring0 + tail * UNIT;
        tail = tail + 1 == RD ? 0 : tail + 1;
        return slot;
    };
    auto fill = [&]() { while (n_fly < RD && load_unit()) {} };
    // the next R rows of the stream . x, summed over the wave
    auto row_dots = [&](float (&dot)[R]) {
#pragma unroll
        for (int q = 0; q < R; ++q) dot[q] = 0.0f;
#pragma unroll
        for (int part = 0; part < PARTS; ++part) {
            const unsigned int slot = wait_oldest();
            u32x4 w[UC], xv[UC];
            if constexpr (R == 1) {
                ring_read_x<UC>(slot + loff, x0 + part * UNIT + loff, w, xv);
            } else {
                ring_read<UC, 4>(slot + loff, w);
#pragma unroll
                for (int c = 0; c < UC / R; ++c) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(s_x + c * 1024 + loff);
#pragma unroll
                    for (int q = 0; q < R; ++q) xv[q * (UC / R) + c] = v;
                }
            }
            --n_fly;
            fill();
#pragma unroll
            for (int q = 0; q < R; ++q)
#pragma unroll
                for (int c = 0; c < UC / R; ++c) dot[q] = dot16<ES>(w[q * (UC / R) + c], xv[q * (UC / R) + c], dot[q]);
        }
#pragma unroll
        for (int q = 0; q < R; ++q) dot[q] = wave_sum(dot[q]);
    };

    fill();
    const float tau = dense ? 0.0f : ((const __attribute__((address_space(4))) float *)ka->tau)[layer];
    // x was requested before the ring's first units
    if (n_fly == RD) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RD * UC) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    float acc[VEC], sum[VEC];                                // this wave's columns: the open class, the slice's closed ones
#pragma unroll
    for (int k = 0; k < VEC; ++k) acc[k] = sum[k] = 0.0f;
    auto close_class = [&]() {
#pragma unroll
        for (int k = 0; k < VEC; ++k) { sum[k] += acc[k]; acc[k] = 0.0f; }
    };
    int cur_cls = 0;                                         // class of the last entry listed so far
    unsigned long long opens2[2] = {0ull, 0ull};             // entries of a list that open another class

    for (int r = 0; r <= n_round; ++r) {
        if (r < n_round) {
            const int p = r & 1, jv = neuron_of(64 * r + lane), ni = min(64, n_local - 64 * r);
            for (int i0 = wave; i0 < ni; i0 += NW * R) {
                float g[R];
                row_dots(g);
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int i = i0 + NW * q, j = __builtin_amdgcn_readlane(jv, i & 63);
                    float v = g[q];
                    if (RELU) {
                        if (b_in && j >= 0) v += b_in[j];
                        v = v > 0.0f ? v : (v != v ? v : 0.0f);
                    } else {
                        v = gate_sigma_f32(v, gelu);
                    }
                    if (lane == 0 && i < ni) { s_a[p][i] = v; s_keep[p][i] = dense || fabsf(v) >= tau; }
                }
            }
            __syncthreads();
            // every wave derives the same ascending list
            const int cls = (64 * r + lane) / per;
            const unsigned long long mask = __ballot(jv >= 0 && s_keep[p][lane] != 0);
            const int kp = __popcll(mask);
            if ((mask >> lane) & 1ull) {
                const int t = __popcll(mask & ((1ull << lane) - 1ull));
                s_lrow[p][t] = jv;
                s_lcls[p][t] = cls;
                s_la[p][t] = s_a[p][lane];
            }
            const int lcls = lane < kp ? s_lcls[p][lane] : cur_cls;
            const int up = __shfl_up(lcls, 1), lprev = lane == 0 ? cur_cls : up;
            opens2[p] = __ballot(lane < kp && lcls != lprev);
            if (kp > 0) cur_cls = __builtin_amdgcn_readlane(lcls, kp - 1);
            kp2[p] = kp;
            n_list = r + 1;
            fill();                                          // the ring may have run dry waiting for this list
        }
        if (r > 0) {
            const int p = (r - 1) & 1, kp = kp2[p];
            const unsigned long long opens = opens2[p];
            const float *hs = s_la[p];
            if constexpr (!RELU) {
                for (int e0 = wave; e0 < kp; e0 += NW * R) {
                    float u[R];
                    row_dots(u);
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int e = e0 + NW * q;
                        if (lane == 0 && e < kp) s_h[p][e] = s_la[p][e] * u[q];
                    }
                }
                __syncthreads();
                hs = s_h[p];
            }
            for (int e0 = 0; e0 < kp; e0 += EPU) {
                const unsigned int slot = wait_oldest();
                typename RingWords<DW>::type v[EPL][UC];
#pragma unroll
                for (int q = 0; q < EPL; ++q) ring_read<UC, DW>(slot + q * CWB + lane * (4 * DW), v[q]);
                --n_fly;
                fill();
#pragma unroll
                for (int n = 0; n < EPU; ++n) {
                    const int e = e0 + n;
                    if (e < kp) {
                        if ((opens >> e) & 1ull) close_class();
                        const float h = hs[e];
#pragma unroll
                        for (int k = 0; k < DW; ++k) {
                            const unsigned int w = v[n % EPL][n / EPL][k];
                            if (ES == 2) {
                                acc[2 * k] = fmaf(h, __uint_as_float(w << 16), acc[2 * k]);
                                acc[2 * k + 1] = fmaf(h, __uint_as_float(w & 0xffff0000u), acc[2 * k + 1]);
                            } else {
                                acc[k] = fmaf(h, __uint_as_float(w), acc[k]);
                            }
                        }
                    }
                }
            }
        }
    }
    close_class();
    float *dst = ka->partial + ((size_t)layer * gridDim.x + group) * ka->d + wave * (CWB / ES) + lane * VEC;
#pragma unroll
    for (int k = 0; k < VEC; ++k) dst[k] = sum[k];
}

struct StackReduceArgs {
    const float *b_out[CLADA_STACK_LAUNCH_LAYERS];
    const float *partial;                   // [n][P][d], P = 32 slices or 256 classes
    char *y;                                // [n][d]
    int P, d;
};

// y[l] from the partial outputs, in the order of the per-layer reduction: slice q = the classes q, q + 32, .. one after the
// other (or the slice as it comes), then the slices by the fixed tree q += q + 16, 8, 4, 2, 1.
template <int ES>
__global__ void __launch_bounds__(256)
k_ffn_stack_reduce(const StackReduceArgs a)
{
    __shared__ float4 s_sum[SLICES][8];
    const int cg = threadIdx.x & 7, sl = threadIdx.x >> 3;
    const int col = blockIdx.x * 32 + cg * 4, layer = blockIdx.y;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col < a.d) {
        const float *base = a.partial + (size_t)layer * a.P * a.d + col;
        if (a.P == SLICES) {
            s = *reinterpret_cast<const float4 *>(base + (size_t)sl * a.d);
        } else {
            float4 v[CHAIN];
#pragma unroll
            for (int u = 0; u < CHAIN; ++u) v[u] = *reinterpret_cast<const float4 *>(base + (size_t)(sl + SLICES * u) * a.d);
#pragma unroll
            for (int u = 0; u < CHAIN; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
        }
    }
    s_sum[sl][cg] = s;
    __syncthreads();
#pragma unroll
    for (int h = SLICES / 2; h >= 1; h >>= 1) {
        if (sl < h) {
            const float4 v = s_sum[sl + h][cg];
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            s_sum[sl][cg] = s;
        }
        __syncthreads();
    }
    if (sl == 0 && col < a.d) {
        const float *bias = a.b_out[layer];
        if (bias) {
            const float4 bv = *reinterpret_cast<const float4 *>(bias + col);
            s.x += bv.x; s.y += bv.y; s.z += bv.z; s.w += bv.w;
        }
        char *y = a.y + ((size_t)layer * a.d + col) * ES;
        if (ES == 4) {
            *reinterpret_cast<float4 *>(y) = s;
        } else {
            uint2 o;
            o.x = f32_to_bf16_bits(s.x) | (f32_to_bf16_bits(s.y) << 16);
            o.y = f32_to_bf16_bits(s.z) | (f32_to_bf16_bits(s.w) << 16);
            *reinterpret_cast<uint2 *>(y) = o;
        }
    }
}

template <int ES, int NCH>
hipError_t launch_rows(const StackLaunch &p, dim3 grid, bool relu, hipStream_t st)
{
    constexpr int threads = RowShape<NCH>::NW * 64;
    if constexpr (NCH != 12 && !(ES == 2 && NCH == 3)) {     // (gated rows of 12 KiB: lanes; of 3 KiB: per-layer calls)
        if (!relu) {
            hipLaunchKernelGGL((k_ffn_stack<ES, NCH, false>), grid, dim3(threads), 0, st, p);
            return hipGetLastError();
        }
    }
    if constexpr (ES == 2) {
        if (relu) {
            hipLaunchKernelGGL((k_ffn_stack<ES, NCH, true>), grid, dim3(threads), 0, st, p);
            return hipGetLastError();
        }
    }
    return hipErrorNotSupported;
}

}  // namespace

size_t clada_ws_stack(int32_t d) { return sizeof(float) * (size_t)CLADA_STACK_LAUNCH_LAYERS * SLICES * d; }

// Rows that only run here in a stack and, layer by layer, on the batch-1 kernel without balancing (us per step, per-layer calls of the generic kernel /
// this one: 189 / 36 at 24 layers of 512 x 1376, 282 / 86 at 24 of 1536 x 4096 ReLU, 343 / 112 at 24 of 2048 x 4632 ReLU, 610 / 442 at
// 24 of 3072 x 8192, 686 / 480 at 24 of 3584 x 8496, 368 / 262 at 8 of 6144 x 13000 ReLU, 83 / 36 at 8 of 768 x 2048 fp32; two layers
// 1.03 - 1.3 times as fast).  Gated bf16 rows of 3 KiB and fp32 rows of 4 and 6 KiB stay on the generic kernel, alone and in stacks.
bool clada_stack_b1_only(const clada_layer *layer)
{
    const int row = layer->d * (int)dtype_size(layer->dtype), nch = row / 1024;
    if (row % 1024 != 0) return false;
    if (layer->kind == CLADA_FFN_RELU)
        return layer->dtype == CLADA_BF16 && (nch == 1 || nch == 3 || nch == 4 || nch == 6 || nch == 7 || nch == 12);
    return layer->dtype == CLADA_BF16 ? nch == 1 || nch == 6 || nch == 7 : nch == 3;
}

// Where the launches over all layers are the faster way (us per step of L layers against lanes of per-layer launches, sparsity
// 0.45).  Nearly everywhere: 2 KiB rows 91 / 197 (L = 24, 1024 x 4096), 4 KiB 521 / 557 (24, 2048 x 16384), 5 KiB ReLU 92 / 110
// (6, 2560 x 10240), 8 KiB 967 / 1040 (32, 4096 x 11008), 10 KiB 1425 / 1546 (32, 5120 x 13824); rows of 12 and 16 KiB gain
// nothing (685 / 670, 1180 / 1145 at L = 12).  The lanes stay where they have as little to wait for:
//   - a few layers of 10 KiB rows, dense or of more than 400 MB (4 layers: 1.01 - 1.05 of the lanes' time)
//   - dense gated layers of 4 and 8 KiB rows, for which the lanes have a kernel of which two workgroups fit a unit, once one
//     layer fills the chip for 30 us (4096 x 11008, one launch / lanes: 333 / 353 at L = 8, 522 / 515 at 12, 1331 / 1328 at 32;
//     4096 x 8192: 993 / 1013 at 32; 2048 x 16384: 1.03 at L = 7, 0.98 at 32)
bool clada_stack_b1_fits(const clada_layer *layer, int32_t L, bool dense)
{
    const int es = (int)dtype_size(layer->dtype), nch = layer->d * es / 1024, F = layer->d_ff;
    const bool gated = layer->kind != CLADA_FFN_RELU;
    if (layer->d * es % 1024 != 0 || L < 2) return false;
    if (clada_stack_b1_only(layer)) return true;
    if (es == 4) return gated && (nch == 2 || nch == 8);
    if (nch == 4) return !(dense && gated && F > 12288 && L < 32);
    if (nch == 8) return !(dense && gated && F > 8192 && L > 8);
    if (nch == 10) return L >= 6 || (!dense && (gated ? 3.0 : 2.0) * F * layer->d * es < 400e6);
    return nch == 2 || nch == 5;
}

hipError_t clada_stack_b1(const clada_layer *layers, int32_t L, const void *x, const float *tau, void *y, bool dense,
                          float *partial, size_t partial_bytes, hipStream_t stream)
{
    const int d = layers[0].d, es = (int)dtype_size(layers[0].dtype), nch = d * es / 1024;
    const bool relu = layers[0].kind == CLADA_FFN_RELU;
    const size_t rows = partial_bytes / (sizeof(float) * (size_t)d);         // at least 1024: the workspace of a per-layer call
    const int room = rows < 65536 ? (int)rows : 65536;
    if (room < CLASSES) return hipErrorInvalidValue;
    // Whole slices leave an eighth of the partial outputs and start an eighth of the workgroups, but there have to be enough of
    // them (us, whole slices / single classes: 162 / 176 at 5 layers of 4096 x 11008, 155 / 141 at 4; 5 KiB rows 1.08 / 0.98 of
    // the lanes at 5 of 2560 x 10240, 0.88 / 0.94 at 6; 4 KiB rows 1.04 / 0.95 at 7 of 2048 x 14336, 0.91 / 0.93 at 8; 2 KiB
    // rows 40 / 39 at 8 of 1024 x 4096, 40 / 35 at 6: their workgroups have four waves).
    const int whole = nch <= 4 ? 8 : nch == 5 ? 6 : 5;
    int most = room / SLICES < CLADA_STACK_LAUNCH_LAYERS ? room / SLICES : CLADA_STACK_LAUNCH_LAYERS;
    if (most > 8) most -= most % 8;
    for (int l0 = 0, n; l0 < L; l0 += n) {
        n = L - l0 < most ? L - l0 : most;
        // A whole slice keeps a unit busy for a round of eight layers (32 workgroups a layer, 256 units), and one to three layers
        // more are a round that leaves most units idle: they go as single classes, in a launch of their own (9 layers of
        // 4096 x 11008: 352 us in one launch, 275 in two, 303 in lanes; 17: 584, 510, 537; at four more the two are even, but for
        // 5 KiB rows: 1.10 at 12 dense layers of 2560 x 10240).  Rows of 4 KiB, whose workgroups are half as wide, notice from the
        // third round on, rows of 2 KiB not at all.
        const int more = n % 8, thin = nch <= 3 ? 0 : nch == 5 ? 4 : 3;
        if (n > (nch == 4 ? 16 : 8) && more <= thin) n -= more;
        const int chain = n >= whole ? CHAIN : 1, P = CLASSES / chain;
        if (n > room / P) {                                  // (single classes: launches of like size)
            const int k = (n + room / P - 1) / (room / P);
            n = (n + k - 1) / k;
        }
        StackLaunch p;
        StackReduceArgs r;
        memset(&p, 0, sizeof(p));
        memset(&r, 0, sizeof(r));
        for (int l = 0; l < n; ++l) {
            const clada_layer &s = layers[l0 + l];
            p.wg[l] = (const char *)s.w_gate; p.wu[l] = (const char *)s.w_up; p.wd[l] = (const char *)s.w_down;
            p.b_in[l] = relu ? s.b_in : nullptr;
            r.b_out[l] = relu ? s.b_out : nullptr;
        }
        p.x = (const char *)x + (size_t)l0 * d * es;
        p.tau = tau ? tau + l0 : nullptr;
        p.partial = partial;
        p.F = layers[0].d_ff; p.d = d; p.chain = chain; p.dense = dense ? 1 : 0;
        p.gelu = layers[0].kind == CLADA_FFN_GEGLU ? 1 : 0;
        const dim3 grid(P, n);
        hipError_t e;
        switch (es == 2 ? nch : 100 + nch) {
        case 1: e = launch_rows<2, 1>(p, grid, relu, stream); break;
        case 2: e = launch_rows<2, 2>(p, grid, relu, stream); break;
        case 3: e = launch_rows<2, 3>(p, grid, relu, stream); break;
        case 4: e = launch_rows<2, 4>(p, grid, relu, stream); break;
        case 5: e = launch_rows<2, 5>(p, grid, relu, stream); break;
        case 6: e = launch_rows<2, 6>(p, grid, relu, stream); break;
        case 7: e = launch_rows<2, 7>(p, grid, relu, stream); break;
        case 8: e = launch_rows<2, 8>(p, grid, relu, stream); break;
        case 10: e = launch_rows<2, 10>(p, grid, relu, stream); break;
        case 12: e = launch_rows<2, 12>(p, grid, relu, stream); break;
        case 102: e = launch_rows<4, 2>(p, grid, relu, stream); break;
        case 103: e = launch_rows<4, 3>(p, grid, relu, stream); break;
        case 108: e = launch_rows<4, 8>(p, grid, relu, stream); break;
        default: e = hipErrorNotSupported;
        }
        if (e != hipSuccess) return e;
        r.partial = partial;
        r.y = (char *)y + (size_t)l0 * d * es;
        r.P = P; r.d = d;
        const dim3 rgrid((d + 31) / 32, n);
        if (es == 4) hipLaunchKernelGGL(k_ffn_stack_reduce<4>, rgrid, dim3(256), 0, stream, r);
        else hipLaunchKernelGGL(k_ffn_stack_reduce<2>, rgrid, dim3(256), 0, stream, r);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
