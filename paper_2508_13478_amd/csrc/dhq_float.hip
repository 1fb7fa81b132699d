// Whole-network fused forward with floating-point activations (gfx950): the "W32A32" and
// "W8A32" rows of the paper's comparison (Sec. 1, Fig. 1-2, Table 2).  W32A32 is the plain
// SIREN, y = W a + b, a = sin(omega0 y); W8A32 is the same network run on the weights after
// the offline step and de-quantization, W~ = (s_w Wq) Hn (the caller passes whichever
// weights apply; the kernel does not know the difference).  fp32 throughout, on the fp32
// MFMA (v_mfma_f32_32x32x2_f32: 32 features x 32 coordinates x 2 k per instruction).
//
// Layout: as in the int8 kernels the features are the MFMA M dimension and a wave carries
// 32 coordinates through all layers.  The D layout gives lane (c, h) rows 8g + 4h + e of
// every 32-row tile T, i.e. register R = 16T + 4g + e holds feature 32T + 8g + 4h + e.  The
// B operand of k step kk wants lane half h to hold "k = 2 kk + h" -- and since the order of k
// is free as long as the weights use the same one, k step kk simply takes register R = kk:
// the activations are consumed exactly where the previous layer's epilogue left them, and
// the weights are packed offline in that order.  Nothing is ever shuffled.
//
// Every MFMA needs only 256 B of weights per wave: they are read straight from device memory (they stay
// in L2), one 16-byte load per lane and four MFMAs, eight groups (4096 matrix-unit clocks)
// ahead of use.  The kernel is bound by the matrix unit (64 clocks per instruction); the
// vector ALU only does one multiply-add and one sine per accumulator.
//
// Registers: one wave per SIMD.  The current activations (B operands, 64 per lane at width
// 128) live in accumulation registers a128..a255, addressed by number from inline assembly
// (the MFMA included: the builtin cannot take B from an accumulation register without a
// copy); the build checks on the compiler's assembly output that compiler-generated code never
// touches them.  Wait states the compiler can no longer see (accumulation-register write ->
// MFMA read, MFMA result -> vector ALU read) are covered by explicit s_nop.
//
// Hidden widths of 32, 64 and 128.  Every other shape (and DHQ_LAYERWISE on the shapes above) runs layer by layer through
// float_layer_kernel: one GEMM on bf16 pieces (fp32 accuracy) with the bias + sine epilogue per layer, activations
// in device memory between the layers, a chunk of rows at a time.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <utility>
#include <vector>

#include "dhq_device.h"
#include "dhq_internal.h"

#define FLT_WAVES 4
#define FLT_THREADS (FLT_WAVES * 64)
#define FLT_TILE (FLT_WAVES * 32)
#define FLT_AGPR_X 128   // first accumulation register of the activations
#define FLT_AHEAD 8      // weight groups (of four k steps) in flight
// Bytes of each of the two activation buffers of the layer-by-layer path: both together stay within the 256 MiB
// memory-side cache, which is worth more than fewer launches (width 512, 262 144 rows: 3.47 ms in chunks of 32 768 rows = 96 MiB
// per buffer, 3.68 ms in chunks of 65 536), while narrower networks take as many rows as fit (width 60: 0.24 ms in chunks of
// 65 536 rows, 0.40 ms in chunks of 32 768).
#define FLT_ACT_BYTES ((int64_t)96 << 20)
// A third of that for the narrow networks, whose rows are short (131 072 rows of 64 features; the launches' latency no longer
// shows), and no more than DHQ_CHUNK rows where DHQ_AUTO has the whole-network kernel and only DHQ_LAYERWISE comes here.
#define FLT_ACT_BYTES_NARROW ((int64_t)32 << 20)

typedef float dhq_v16f __attribute__((ext_vector_type(16)));

struct float_layer_desc {
    uint32_t w_off;     // float offset of the layer's packed weights in the blob
    uint32_t b_off;     // float offset of its bias block [tile][h][16]
};

struct float_args {
    const float *coords;
    float *out;
    const float *blob;
    int64_t n;
    int n_layers;
    int k0;          // fan-in of the input layer (<= 4)
    int m_out;       // fan-out of the output layer (<= 32)
    float rev;       // omega0 / (2 pi): the sine takes revolutions
    float c2;        // wavelet activation: 2 pi s0 sqrt(log2 e) / omega0
    float_layer_desc layer[DHQ_MAX_LAYERS];
};

// One layer of the layer-by-layer path: weights as fragments of their three bf16 pieces (see float_layer_kernel), biases
// [feature tile][lane half][16] (times omega0 / 2 pi where an activation follows).
struct float_lw_layer {
    const unsigned char *wfrag_dev = nullptr;  // inside the plan's lw_blob_dev, like the biases
    const float *bias_dev = nullptr;
    int K = 0, M = 0, nkb = 0, Mt = 0;
};

struct dhq_float_plan {
    int nf = 0;              // hidden width of the fused kernel, 0 if the shape has none
    float *blob_dev = nullptr;
    size_t blob_floats = 0;
    float_args args;
    int n_cu = 0;
    int n_layers = 0;
    float rev = 0.f;
    dhq_act actf = {DHQ_ACT_KIND_SINE, 0.f};  // what follows every layer but the last
    float_lw_layer lw[DHQ_MAX_LAYERS];
    unsigned char *lw_blob_dev = nullptr;
    unsigned char *act[2] = {nullptr, nullptr};  // chunk_rows rows of fragments of the widest layer
    int64_t chunk_rows = 0;
    bool narrow = false;  // every layer input up to 64 wide: float_narrow_kernel
    int device = 0;
};

// ----------------------------------------------------------------------------- device code
template <int KK>
__device__ __forceinline__ void flt_x_write(float v)
{
    asm volatile("v_accvgpr_write_b32 a[%1], %0" : : "v"(v), "n"(FLT_AGPR_X + KK));
}
template <int KK>
__device__ __forceinline__ void flt_mfma_first(dhq_v16f &acc, float a)
{
    asm volatile("v_mfma_f32_32x32x2_f32 %0, %1, a[%2], 0" : "=&v"(acc) : "v"(a), "n"(FLT_AGPR_X + KK));
}
template <int KK>
__device__ __forceinline__ void flt_mfma_next(dhq_v16f &acc, float a)
{
    asm volatile("v_mfma_f32_32x32x2_f32 %0, %1, a[%2], %0" : "+v"(acc) : "v"(a), "n"(FLT_AGPR_X + KK));
}
// Idle issue slots that the readers of `acc` cannot be moved ahead of (16-pass MFMA -> vector ALU).
__device__ __forceinline__ void flt_settle(dhq_v16f &acc)
{
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(acc));
}

template <int... Ks>
__device__ __forceinline__ void flt_x_store(const float *y, std::integer_sequence<int, Ks...>)
{
    (flt_x_write<Ks>(y[Ks]), ...);
    asm volatile("s_nop 7" ::: "memory");  // accumulation-register write -> MFMA read
}

// One group of a hidden layer's GEMM: k steps 4q .. 4q+3 for the CHN tiles of pair P.
//   ring   weight groups in flight: ring[(g % FLT_AHEAD) * CHN + j] is the float4 of tile j
//   wl     this lane's pointer into the layer's packed weights: group g, tile j at wl[(g * CHN + j) * 64]
template <int NF, int CHN, int G>
__device__ __forceinline__ void flt_group(const float4 *__restrict__ wl, float4 (&ring)[FLT_AHEAD * CHN],
                                          dhq_v16f (&acc)[CHN])
{
    constexpr int NQ = NF / 8;           // groups per pair (k steps / 4)
    constexpr int NP = NF / 32 / CHN;    // pairs per layer
    constexpr int q = G % NQ;
    constexpr int pf = G + FLT_AHEAD;
    float4 cur[CHN];
#pragma unroll
    for (int j = 0; j < CHN; ++j) cur[j] = ring[(G % FLT_AHEAD) * CHN + j];
    if constexpr (pf < NP * NQ) {
#pragma unroll
        for (int j = 0; j < CHN; ++j) ring[(pf % FLT_AHEAD) * CHN + j] = wl[(pf * CHN + j) * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < CHN; ++j) {
        if constexpr (q == 0)
            flt_mfma_first<4 * q + 0>(acc[j], cur[j].x);
        else
            flt_mfma_next<4 * q + 0>(acc[j], cur[j].x);
    }
#pragma unroll
    for (int j = 0; j < CHN; ++j) flt_mfma_next<4 * q + 1>(acc[j], cur[j].y);
#pragma unroll
    for (int j = 0; j < CHN; ++j) flt_mfma_next<4 * q + 2>(acc[j], cur[j].z);
#pragma unroll
    for (int j = 0; j < CHN; ++j) flt_mfma_next<4 * q + 3>(acc[j], cur[j].w);
    __builtin_amdgcn_sched_barrier(0);
}

// ACTK: the activation (sine, or the wavelet with envelope constant c2).
template <int NF, int CHN, int ACTK, int P, int... Qs>
__device__ __forceinline__ void flt_pair(const float4 *__restrict__ wl, const float4 *__restrict__ bl,
                                         float4 (&ring)[FLT_AHEAD * CHN], float rev, float c2, float (&y)[NF / 2],
                                         std::integer_sequence<int, Qs...>)
{
    constexpr int NQ = NF / 8;
    dhq_v16f acc[CHN];
    // the pair's biases, fetched while the matrix unit works
    float4 bq[CHN][4];
#pragma unroll
    for (int j = 0; j < CHN; ++j)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) bq[j][gg] = bl[(P * CHN + j) * 8 + gg];
    (flt_group<NF, CHN, P * NQ + Qs>(wl, ring, acc), ...);
#pragma unroll
    for (int j = 0; j < CHN; ++j) {
        flt_settle(acc[j]);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float4 bb = bq[j][v >> 2];
            const float bias = (v & 3) == 0 ? bb.x : (v & 3) == 1 ? bb.y : (v & 3) == 2 ? bb.z : bb.w;
            y[16 * (P * CHN + j) + v] = dhq_activate_rev(__builtin_fmaf(acc[j][v], rev, bias), dhq_act{ACTK, c2});
        }
    }
}

template <int NF, int CHN, int ACTK, int... Ps>
__device__ __forceinline__ void flt_hidden_layer(const float4 *__restrict__ wl, const float4 *__restrict__ bl, float rev, float c2,
                                                 float (&y)[NF / 2], std::integer_sequence<int, Ps...>)
{
    constexpr int NQ = NF / 8;
    constexpr int NG = (NF / 32 / CHN) * NQ;
    float4 ring[FLT_AHEAD * CHN];
#pragma unroll
    for (int g = 0; g < FLT_AHEAD; ++g)
        if (g < NG) {
#pragma unroll
            for (int j = 0; j < CHN; ++j) ring[g * CHN + j] = wl[(g * CHN + j) * 64];
        }
    (flt_pair<NF, CHN, ACTK, Ps>(wl, bl, ring, rev, c2, y, std::make_integer_sequence<int, NQ>{}), ...);
}

template <int NF, int... Qs>
__device__ __forceinline__ void flt_out_layer(const float4 *__restrict__ wl, dhq_v16f &acc, std::integer_sequence<int, Qs...>)
{
    // one tile, no look-ahead ring: the compiler's own scheduling of these loads is enough for 1/8 of a layer
    ((Qs == 0 ? flt_mfma_first<4 * Qs>(acc, wl[Qs * 64].x) : flt_mfma_next<4 * Qs>(acc, wl[Qs * 64].x),
      flt_mfma_next<4 * Qs + 1>(acc, wl[Qs * 64].y), flt_mfma_next<4 * Qs + 2>(acc, wl[Qs * 64].z),
      flt_mfma_next<4 * Qs + 3>(acc, wl[Qs * 64].w)),
     ...);
}

template <int NF, int ACTK>
__global__ __launch_bounds__(FLT_THREADS) void dhq_float_kernel(const float_args A)
{
    constexpr int NT = NF / 32;
    constexpr int NR = NF / 2;
    constexpr int CHN = NT >= 2 ? 2 : 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int L = A.n_layers;
    const int64_t n_tiles = (A.n + FLT_TILE - 1) / FLT_TILE;
    // the registers addressed by number count towards the kernel's register allocation
    asm volatile("" ::: "a255");
    static_assert(FLT_AGPR_X + NR <= 256, "register map");

    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t ci = tile * FLT_TILE + wave * 32 + c;
        const bool valid = ci < A.n;
        const int64_t cl = valid ? ci : A.n - 1;
        float y[NR];
        {
            // input layer: k step kk holds coordinate component 2 kk + h of this lane's coordinate
            const float x0 = (h < A.k0) ? A.coords[cl * A.k0 + h] : 0.0f;
            const float x1 = (2 + h < A.k0) ? A.coords[cl * A.k0 + 2 + h] : 0.0f;
            flt_x_write<0>(x0);
            flt_x_write<1>(x1);
            asm volatile("s_nop 7" ::: "memory");
            const float *w0 = A.blob + A.layer[0].w_off + lane;
            const float4 *b0 = reinterpret_cast<const float4 *>(A.blob + A.layer[0].b_off) + h * 4;
#pragma unroll
            for (int T = 0; T < NT; ++T) {
                dhq_v16f acc;
                flt_mfma_first<0>(acc, w0[(T * 2 + 0) * 64]);
                flt_mfma_next<1>(acc, w0[(T * 2 + 1) * 64]);
                float4 bq[4];
#pragma unroll
                for (int gg = 0; gg < 4; ++gg) bq[gg] = b0[T * 8 + gg];
                flt_settle(acc);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float4 bb = bq[v >> 2];
                    const float bias = (v & 3) == 0 ? bb.x : (v & 3) == 1 ? bb.y : (v & 3) == 2 ? bb.z : bb.w;
                    y[16 * T + v] = dhq_activate_rev(__builtin_fmaf(acc[v], A.rev, bias), dhq_act{ACTK, A.c2});
                }
            }
        }
        for (int l = 1; l < L - 1; ++l) {
            flt_x_store(y, std::make_integer_sequence<int, NR>{});
            const float4 *wl = reinterpret_cast<const float4 *>(A.blob + A.layer[l].w_off) + lane;
            const float4 *bl = reinterpret_cast<const float4 *>(A.blob + A.layer[l].b_off) + h * 4;
            flt_hidden_layer<NF, CHN, ACTK>(wl, bl, A.rev, A.c2, y, std::make_integer_sequence<int, NT / CHN>{});
        }
        {
            // output layer: one zero-padded tile, no sine
            flt_x_store(y, std::make_integer_sequence<int, NR>{});
            const float4 *wl = reinterpret_cast<const float4 *>(A.blob + A.layer[L - 1].w_off) + lane;
            const float *bo = A.blob + A.layer[L - 1].b_off + h * 16;
            dhq_v16f acc;
            flt_out_layer<NF>(wl, acc, std::make_integer_sequence<int, NR / 4>{});
            float bias[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) bias[v] = bo[v];
            flt_settle(acc);
            if (valid) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                    if (row < A.m_out) A.out[ci * A.m_out + row] = acc[v] + bias[v];
                }
            }
        }
    }
}

// ---------------------------------------------------------------- layer by layer, any shape
// One GEMM kernel per layer.  The fp32 MFMA delivers 64 multiply-adds per clock and SIMD, the bf16 one 1024, and three
// bf16 pieces hold an fp32 value without loss: hi = bf16(a), mid = bf16(a - hi), lo = a - hi - mid (rounded to nearest,
// 8 significant bits each, both differences exact).  So every product a w is taken as the six bf16 products whose
// weight is at least 2^-17 of it,
//     hi hi + (hi mid + mid hi) + (hi lo + mid mid + lo hi),
// each exact in the MFMA and summed in fp32.  Left out are mid lo, lo mid and lo lo: at most 2^-24 of |a w| together,
// half an ulp of the product, with a random sign.  A layer then costs 6 / 16 of the fp32 MFMA time.
//
// Layout.  Features are the MFMA M dimension (weights = A operand), coordinates its N dimension, so that a lane's
// accumulators are half of one coordinate's features and become, split into pieces, that lane's B operands of the next
// layer without leaving the lane: k block kb = 2 T + b of the next layer takes accumulators 8 b .. 8 b + 7 of tile T, i.e.
// slot j of lane half h is feature 32 T + 8 (2 b + j / 4) + 4 h + j % 4; the weights are packed in that k order.
// Activations cross device memory as fragments, [tile of 32 coordinates][k block][piece][lane] x 16 B, weights as
// [feature tile][k block][piece][lane] x 16 B: every access of a wave is 1 KiB contiguous and goes straight into LDS.
//
// A workgroup of WF x WC waves computes WF TF feature tiles x WC TC coordinate tiles, a wave TF x TC of them.
// Bound by the matrix unit: a 65 536 x 512 x 512 layer takes 173 us = 1.19 PFLOP/s of bf16 products, which is what a large
// bf16 library product reaches on this card with random operands (1.22-1.35; 1.69 with zeros: the clock follows the
// operands).  The fp32 MFMA form of this kernel took 370 us.  Error against fp64 at width 512, six layers: 3.4e-8 rms
// (1.7e-7 largest) against 3.9e-8 (1.9e-7) for the fp32 MFMA, which rounds after every two products instead of every sixteen.
typedef __bf16 flt_v8b __attribute__((ext_vector_type(8)));
typedef __bf16 flt_v2b __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned flt_pack_bf16(float a, float b)
{
    const flt_v2b p = {(__bf16)a, (__bf16)b};  // one packed conversion, rounded to nearest even
    return __builtin_bit_cast(unsigned, p);
}
// The three bf16 pieces of two values, value 0 in the low halves.
__device__ __forceinline__ void flt_split3(float a0, float a1, unsigned &hi, unsigned &mid, unsigned &lo)
{
    hi = flt_pack_bf16(a0, a1);
    const float r0 = a0 - __uint_as_float(hi << 16), r1 = a1 - __uint_as_float(hi & 0xffff0000u);
    mid = flt_pack_bf16(r0, r1);
    lo = flt_pack_bf16(r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xffff0000u));
}
// Eight values to a lane's 16 bytes of each of the three fragments at dst, dst + 1 KiB, dst + 2 KiB.
__device__ __forceinline__ void flt_store_pieces(const float (&y)[8], unsigned char *__restrict__ dst)
{
    uint4 hi, mid, lo;
    flt_split3(y[0], y[1], hi.x, mid.x, lo.x);
    flt_split3(y[2], y[3], hi.y, mid.y, lo.y);
    flt_split3(y[4], y[5], hi.z, mid.z, lo.z);
    flt_split3(y[6], y[7], hi.w, mid.w, lo.w);
    *reinterpret_cast<uint4 *>(dst) = hi;
    *reinterpret_cast<uint4 *>(dst + 1024) = mid;
    *reinterpret_cast<uint4 *>(dst + 2048) = lo;
}

// The six products of one k block, small ones first; w, x: {hi, mid, lo}.
__device__ __forceinline__ dhq_v16f flt_mfma6(const dhq_v4i (&w)[3], const dhq_v4i (&x)[3], dhq_v16f acc)
{
    constexpr int pw[6] = {0, 2, 1, 0, 1, 0}, px[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int i = 0; i < 6; ++i)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(flt_v8b, w[pw[i]]), __builtin_bit_cast(flt_v8b, x[px[i]]), acc, 0, 0, 0);
    return acc;
}

// The network's input: n x K row-major fp32 to fragments in natural k order (slot j of lane half h of block kb is
// k = 16 kb + 8 h + j; zero beyond K and n).  One wave per tile and k block.
__global__ __launch_bounds__(256) void float_pack_kernel(const float *__restrict__ in, int64_t n, int K, int nkb, int64_t n_frag,
                                                         unsigned char *__restrict__ out)
{
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= n_frag) return;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int64_t ct = w / nkb, row = ct * 32 + c;
    const int k0 = 16 * (int)(w - ct * nkb) + 8 * h;
    float y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = (row < n && k0 + j < K) ? in[row * K + k0 + j] : 0.f;
    flt_store_pieces(y, out + (size_t)w * 3072 + lane * 16);
}

struct float_layer_args {
    const unsigned char *in;   // activations, [n_ct][nkb][3] KiB
    const unsigned char *w;    // weights, [n_ft][nkb][3] KiB
    const float *bias;         // [n_ft][lane half][16], times omega0 / 2 pi where a sine follows
    unsigned char *out;        // activations, [n_ct][2 n_ft][3] KiB
    int n_ct, n_ft, nkb;       // nkb: even
    int nF, nC;                // workgroups over the features and over the coordinates
    float rev, c2;
};

// 1 KiB from device memory straight into LDS (as fused_issue_copy does): src and dst wave-uniform, voff = lane * 16.
__device__ __forceinline__ void flt_copy_kib(unsigned voff, const unsigned char *src, unsigned dst)
{
    const unsigned long long a = (unsigned long long)src;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    const unsigned long long sa = ((unsigned long long)hi << 32) | lo;
    const unsigned m0v = __builtin_amdgcn_readfirstlane(dst);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sa), "s"(m0v) : "memory", "m0");
}

// Waits for every load of this wave.  The builtin, not inline assembly: the compiler then knows that the activations it
// loaded one stage ago have arrived and does not wait for the loads that were issued since.
__device__ __forceinline__ void flt_wait_loads()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters unrestricted
    asm volatile("" ::: "memory");
}

// KS: k blocks per stage.  The weights of a stage go through LDS, shared by the WC waves of a row of tiles, in three
// buffers: while stage s computes, stage s + 2 is copied in, and the barrier in front of stage s says that s + 1 is in place,
// so that its first fragments are fetched before stage s ends.  The activations of a tile are used by WF waves only and
// go straight into registers, one stage ahead.  A stage's requests are spread over its MFMAs: all at its start, the
// 64 KiB a CU asks for there keep its memory pipeline busy for 1 kclk, in which no wave gets to its MFMAs.
template <int ACT, int WF, int WC, int TF, int TC, int KS>
struct float_layer_tile {
    static constexpr int NW = WF * WC, FT = WF * TF, CT = WC * TC;
    static constexpr int BLOCKS = 3 * FT * KS;  // KiB of weights per stage: [feature tile][k block][piece]
    static constexpr int PER_WAVE = (BLOCKS + NW - 1) / NW;
    static constexpr int NX = 3 * TC * KS, REQUESTS = NX + PER_WAVE;  // per stage and wave
    static constexpr int NI = KS * TF, GROUPS = 6 * NI;               // steps of a stage, groups of TC MFMAs
    const float_layer_args &A;
    const unsigned char *lds;
    unsigned lds0, voff;
    int lane, wave, wf, wc, f0, c0, n_stages;
    const unsigned char *src[PER_WAVE];
    const unsigned char *xsrc[TC];
    dhq_v4i x[2][TC][KS][3], w[2][3];
    dhq_v16f acc[TF][TC];
    __device__ __forceinline__ float_layer_tile(const float_layer_args &A_) : A(A_) {}

    // 1 KiB of the weights of stage s, this wave's i-th, into buffer buf; nothing past the last k block
    template <int I>
    __device__ __forceinline__ void copy_weights(int s, int buf)
    {
        const int q = wave + I * NW;
        if ((BLOCKS % NW != 0 && q >= BLOCKS) || s * KS + (KS > 1 ? (q / 3) % KS : 0) >= A.nkb) return;
        flt_copy_kib(voff, src[I] + (size_t)s * (3072 * KS), lds0 + (buf * BLOCKS + q) * 1024);
    }
    // the I-th fragment of the activations of stage s (past the last k block: the last one again, not used)
    template <int XB, int I>
    __device__ __forceinline__ void load_x(int s)
    {
        constexpr int k = I / (3 * TC), c = (I / 3) % TC, p = I % 3;
        const int kb = s * KS + k < A.nkb ? s * KS + k : A.nkb - 1;
        x[XB][c][k][p] = *reinterpret_cast<const dhq_v4i *>(xsrc[c] + (size_t)(kb * 3 + p) * 1024 + voff);
    }
    template <int XB, int... I>
    __device__ __forceinline__ void load_x_all(int s, std::integer_sequence<int, I...>) { (load_x<XB, I>(s), ...); }
    template <int... I>
    __device__ __forceinline__ void copy_weights_all(int s, int buf, std::integer_sequence<int, I...>) { (copy_weights<I>(s, buf), ...); }
    template <int WB>
    __device__ __forceinline__ void load_w(int buf, int k, int f)
    {
        const dhq_v4i *b = reinterpret_cast<const dhq_v4i *>(lds + buf * BLOCKS * 1024) + lane;
#pragma unroll
        for (int p = 0; p < 3; ++p) w[WB][p] = b[(((wf * TF + f) * KS + k) * 3 + p) * 64];
    }
    // Request R of stage s, issued in front of MFMA group G: the activations first.
    template <int S, int G, int R>
    __device__ __forceinline__ void request(int s, int b2)
    {
        if constexpr (R < REQUESTS) {
            if constexpr (R * (3 * GROUPS / 4) / REQUESTS == G) {
                if constexpr (R < NX) load_x<S ^ 1, R>(s + 1);
                else copy_weights<R - NX>(s + 2, b2);
                __builtin_amdgcn_sched_barrier(0);
            }
            request<S, G, R + 1>(s, b2);
        }
    }
    // Group G of stage s: product G % 6 (small ones first) of step G / 6 for this wave's TC coordinate tiles.
    template <int S, int G>
    __device__ __forceinline__ void group(int s, int b0, int b1, int b2)
    {
        constexpr int I = G / 6, i = G % 6, k = I / TF, f = I % TF, wb = (S * NI + I) & 1;
        constexpr int pw[6] = {0, 2, 1, 0, 1, 0}, px[6] = {2, 0, 1, 1, 0, 0};
        if constexpr (i == 0) {  // the next step's weight fragments
            if constexpr (I + 1 < NI) load_w<wb ^ 1>(b0, (I + 1) / TF, (I + 1) % TF);
            else load_w<wb ^ 1>(b1, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        request<S, G, 0>(s, b2);
        if (KS == 1 || s * KS + k < A.nkb) {
#pragma unroll
            for (int c = 0; c < TC; ++c)
                acc[f][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(flt_v8b, w[wb][pw[i]]),
                                                                    __builtin_bit_cast(flt_v8b, x[S][c][k][px[i]]), acc[f][c], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (G + 1 < GROUPS) group<S, G + 1>(s, b0, b1, b2);
    }
    // Stage s (its weights in buffer b0, the next one's in b1, the one after that goes to b2); S: parity of s.
    template <int S>
    __device__ __forceinline__ void stage(int s, int b0, int b1, int b2)
    {
        flt_wait_loads();
        __syncthreads();
        group<S, 0>(s, b0, b1, b2);
    }
};

template <int ACT, int WF, int WC, int TF, int TC, int KS>
__global__ __launch_bounds__(64 * WF * WC) void float_layer_kernel(const float_layer_args A)
{
    using tile_t = float_layer_tile<ACT, WF, WC, TF, TC, KS>;
    extern __shared__ __align__(16) unsigned char lds[];
    tile_t R(A);
    const int lane = threadIdx.x & 63, h = lane >> 5;
    R.lane = lane;
    R.voff = lane * 16;
    R.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    R.wf = R.wave % WF;
    R.wc = R.wave / WF;
    // consecutive workgroups go to the eight XCDs in turn: the workgroups that read the same coordinates get the same
    // XCD, so that all but the first find them in its L2
    const int xcd = blockIdx.x & 7, rest = blockIdx.x >> 3;
    const int fb = rest % A.nF, cb = (rest / A.nF) * 8 + xcd;
    if (cb >= A.nC) return;  // the whole workgroup: no barrier has been reached
    R.f0 = fb * tile_t::FT;
    R.c0 = cb * tile_t::CT;
    R.lds = lds;
    R.lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)lds;
    R.n_stages = (A.nkb + KS - 1) / KS;
    // this wave's share of a stage's weights: 1 KiB blocks wave, wave + NW, ...; tiles past the last one are read again
#pragma unroll
    for (int i = 0; i < tile_t::PER_WAVE; ++i) {
        const int q = R.wave + i * tile_t::NW, t = q / (3 * KS), r = q % (3 * KS);
        const int f = R.f0 + t < A.n_ft ? R.f0 + t : A.n_ft - 1;
        R.src[i] = A.w + ((size_t)f * A.nkb * 3 + r) * 1024;
    }
#pragma unroll
    for (int c = 0; c < TC; ++c) {
        const int ct = R.c0 + R.wc * TC + c < A.n_ct ? R.c0 + R.wc * TC + c : A.n_ct - 1;
        R.xsrc[c] = A.in + (size_t)ct * A.nkb * 3072;
    }
#pragma unroll
    for (int f = 0; f < TF; ++f)
#pragma unroll
        for (int c = 0; c < TC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) R.acc[f][c][v] = 0.f;
    R.copy_weights_all(0, 0, std::make_integer_sequence<int, tile_t::PER_WAVE>{});
    R.copy_weights_all(1, 1, std::make_integer_sequence<int, tile_t::PER_WAVE>{});
    R.template load_x_all<0>(0, std::make_integer_sequence<int, tile_t::NX>{});
    flt_wait_loads();
    __syncthreads();
    R.template load_w<0>(0, 0, 0);
    int b0 = 0, b1 = 1, b2 = 2;
    for (int s = 0; s < R.n_stages; s += 2) {
        R.template stage<0>(s, b0, b1, b2);
        R.template stage<1>(s + 1, b1, b2, b0);  // (an odd count: the last one computes nothing)
        const int t = b0;  // two stages on: b0, b1, b2 -> b2, b0, b1
        b0 = b2; b2 = b1; b1 = t;
    }
#pragma unroll
    for (int f = 0; f < TF; ++f) {
        const int T = R.f0 + R.wf * TF + f;
        if (T >= A.n_ft) break;
        float bias[16];
#pragma unroll
        for (int v = 0; v < 16; v += 4) *reinterpret_cast<float4 *>(&bias[v]) = *reinterpret_cast<const float4 *>(A.bias + (T * 2 + h) * 16 + v);
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            const int ct = R.c0 + R.wc * TC + c;
            if (ct >= A.n_ct) break;
            unsigned char *dst = A.out + ((size_t)ct * A.n_ft + T) * 6144 + lane * 16;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                float y[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    y[j] = dhq_activate_rev_any(__builtin_fmaf(R.acc[f][c][8 * b + j], A.rev, bias[8 * b + j]), dhq_act{ACT, A.c2});
                flt_store_pieces(y, dst + b * 3072);
            }
        }
    }
}

// The output layer: one tile of 32 features x 32 coordinates per wave, fragments straight from device memory (each is
// used once), no activation; bound by reading the activations.
__global__ __launch_bounds__(256) void float_out_kernel(const unsigned char *__restrict__ in, const unsigned char *__restrict__ wfrag,
                                                        const float *__restrict__ bias, int64_t n, int n_ct, int nkb, int M,
                                                        float *__restrict__ out)
{
    const int ct = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), T = blockIdx.y;
    if (ct >= n_ct) return;
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const dhq_v4i *xp = reinterpret_cast<const dhq_v4i *>(in + (size_t)ct * nkb * 3072) + lane;
    const dhq_v4i *wp = reinterpret_cast<const dhq_v4i *>(wfrag + (size_t)T * nkb * 3072) + lane;
    dhq_v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int kb0 = 0; kb0 < nkb; kb0 += 4) {
        dhq_v4i x[4][3], w[4][3];  // four k blocks in flight; blocks past the last one are read again and not used
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kb = kb0 + i < nkb ? kb0 + i : nkb - 1;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                x[i][p] = xp[(kb * 3 + p) * 64];
                w[i][p] = wp[(kb * 3 + p) * 64];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (kb0 + i < nkb) acc = flt_mfma6(w[i], x[i], acc);
    }
    const int64_t row = (int64_t)ct * 32 + c;
    if (row >= n) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int f = 32 * T + 8 * (v >> 2) + 4 * h + (v & 3);
        if (f < M) out[row * M + f] = acc[v] + bias[(T * 2 + h) * 16 + v];
    }
}

// ---- narrow networks: hidden widths up to 64 ----------------------------------------------------
// A layer of such a network is a few MFMAs per 32 coordinates, so what it takes is latency and memory, and the tiles above,
// with their stages of LDS copies and fragments of six bytes a value, were slower than one wave per tile that holds the
// layer's whole weights in registers: 4 layers of 20 features on 65 536 rows 45 -> 19 us, 4 of 48 58 -> 37 us.  Between the
// layers the activations travel as floats in the lanes' order, [tile of 32 coordinates][feature tile][float4 q][lane], and
// are split into pieces by the wave that reads them: the same pieces, products and order of sums as above, so the same bits
// (of sines; a wavelet above goes into its pieces before its last product is rounded to fp32).
// NT: feature tiles (of the output layer: one, gridDim.y of them); NKB: k blocks.  A wave takes every gridDim.x * 4-th tile.
struct float_narrow_args {
    const float *in;           // FIRST: n x K coordinates, else the layer below's output
    float *out;                // LAST: n x M, else the layer above's input
    const unsigned char *w;    // [feature tile][k block][piece] KiB
    const float *bias;         // [feature tile][lane half][16]
    int64_t n;
    int n_ct, K, M;
    float rev, c2;
};
template <int ACT, int NT, int NKB, bool FIRST, bool LAST>
__global__ __launch_bounds__(256) void float_narrow_kernel(const float_narrow_args A)
{
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int stride = (int)gridDim.x * 4, T0 = LAST ? (int)blockIdx.y : 0;
    int ct = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (ct >= A.n_ct) return;
    // the eight inputs of k block kb
    auto load = [&](int tile, float (&v)[NKB][8]) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if constexpr (FIRST) {
                const int64_t row = (int64_t)tile * 32 + c;
                const int k0 = 16 * kb + 8 * h;
#pragma unroll
                for (int j = 0; j < 8; ++j) v[kb][j] = (row < A.n && k0 + j < A.K) ? A.in[row * A.K + k0 + j] : 0.f;
            } else {
                const float4 *src = reinterpret_cast<const float4 *>(A.in) + ((size_t)tile * (NKB * 2) + kb * 2) * 64 + lane;
                const float4 a = src[0], b = src[64];
                v[kb][0] = a.x; v[kb][1] = a.y; v[kb][2] = a.z; v[kb][3] = a.w;
                v[kb][4] = b.x; v[kb][5] = b.y; v[kb][6] = b.z; v[kb][7] = b.w;
            }
        }
    };
    float v[NKB][8];
    load(ct, v);
    dhq_v4i w[NT][NKB][3];
    float bias[NT][16];
#pragma unroll
    for (int T = 0; T < NT; ++T) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int p = 0; p < 3; ++p) w[T][kb][p] = reinterpret_cast<const dhq_v4i *>(A.w)[(((T0 + T) * NKB + kb) * 3 + p) * 64 + lane];
#pragma unroll
        for (int i = 0; i < 16; i += 4) *reinterpret_cast<float4 *>(&bias[T][i]) = *reinterpret_cast<const float4 *>(A.bias + ((T0 + T) * 2 + h) * 16 + i);
    }
    for (; ct < A.n_ct; ct += stride) {
        dhq_v4i x[NKB][3];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                unsigned hi, mid, lo;
                flt_split3(v[kb][2 * d], v[kb][2 * d + 1], hi, mid, lo);
                x[kb][0][d] = (int)hi; x[kb][1][d] = (int)mid; x[kb][2][d] = (int)lo;
            }
        if (ct + stride < A.n_ct) load(ct + stride, v);  // arrives during the products
        dhq_v16f acc[NT];
#pragma unroll
        for (int T = 0; T < NT; ++T) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[T][i] = 0.f;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) acc[T] = flt_mfma6(w[T][kb], x[kb], acc[T]);
        }
#pragma unroll
        for (int T = 0; T < NT; ++T) {
            if constexpr (LAST) {
                const int64_t row = (int64_t)ct * 32 + c;
                if (row < A.n) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int f = 32 * (T0 + T) + 8 * (i >> 2) + 4 * h + (i & 3);
                        if (f < A.M) A.out[row * A.M + f] = acc[T][i] + bias[T][i];
                    }
                }
            } else {
                float4 *dst = reinterpret_cast<float4 *>(A.out) + ((size_t)ct * NT + T) * 256 + lane;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        y[e] = dhq_activate_rev_any(__builtin_fmaf(acc[T][4 * q + e], A.rev, bias[T][4 * q + e]), dhq_act{ACT, A.c2});
                    dst[q * 64] = make_float4(y[0], y[1], y[2], y[3]);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------- host code
// Feature held by register kk of lane half h (the D layout of the 32 x 32 MFMA).
static int flt_feature(int kk, int h) { return 32 * (kk >> 4) + 8 * ((kk >> 2) & 3) + 4 * h + (kk & 3); }

bool dhq_float_shape_ok(const int *dims, int L)
{
    if (L < 2) return false;
    if (dims[0] > 4 || dims[L] > 32) return false;
    const int nf = dims[1];
    if (nf != 32 && nf != 64 && nf != 128 && nf != 256) return false;
    for (int l = 1; l < L; ++l)
        if (dims[l] != nf) return false;
    return true;
}

static int float_create_fused(dhq_float_plan *P, const int *dims, int L, double rev, const std::vector<std::vector<float>> &W,
                              const std::vector<std::vector<float>> &b);
static int float_create_layerwise(dhq_float_plan *P, const int *dims, int L, double rev, const std::vector<std::vector<float>> &W,
                                  const std::vector<std::vector<float>> &b);

// W[l]: dims[l+1] x dims[l] fp32 (the weights the network is to run on), b[l]: dims[l+1].
// `act` follows every layer but the last.
int dhq_float_create(const int *dims, int L, float omega0, dhq_act act, const std::vector<std::vector<float>> &W,
                     const std::vector<std::vector<float>> &b, int device, dhq_float_plan **plan_out)
{
    *plan_out = nullptr;
    dhq_float_plan *P = new (std::nothrow) dhq_float_plan();
    if (!P) return DHQ_ENOMEM;
    memset(&P->args, 0, sizeof(P->args));
    const double rev = (double)omega0 / 6.283185307179586476925286766559;
    P->n_layers = L;
    P->rev = (float)rev;
    P->actf = act;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
        delete P;
        return DHQ_EHIP;
    }
    P->n_cu = prop.multiProcessorCount;
    P->device = device;
    int rc = float_create_layerwise(P, dims, L, rev, W, b);
    if (rc == DHQ_OK && dhq_float_shape_ok(dims, L)) rc = float_create_fused(P, dims, L, rev, W, b);
    if (rc != DHQ_OK) {
        dhq_float_destroy(P);
        return rc;
    }
    *plan_out = P;
    return DHQ_OK;
}

// The packed weights and biases of the whole-network kernel.
static int float_create_fused(dhq_float_plan *P, const int *dims, int L, double rev, const std::vector<std::vector<float>> &W,
                              const std::vector<std::vector<float>> &b)
{
    const int nf = dims[1], NT = nf / 32, NR = nf / 2, CHN = NT >= 2 ? 2 : 1;
    P->nf = nf;
    if (nf == 256) return DHQ_OK;  // runs layer by layer (dhq_float_launch)
    std::vector<float> blob;
    auto bias_block = [&](int l, int tiles, bool sine) {
        // [tile][h][16]: register v of lane half h holds feature 32 T + 8 (v / 4) + 4 h + v % 4
        const size_t off = blob.size();
        blob.resize(off + (size_t)tiles * 32, 0.0f);
        for (int T = 0; T < tiles; ++T)
            for (int h = 0; h < 2; ++h)
                for (int v = 0; v < 16; ++v) {
                    const int f = 32 * T + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (f < dims[l + 1])
                        blob[off + (size_t)(T * 2 + h) * 16 + v] = sine ? (float)((double)b[l][f] * rev) : b[l][f];
                }
        return (uint32_t)off;
    };
    for (int l = 0; l < L; ++l) {
        const int K = dims[l], M = dims[l + 1];
        const size_t off = blob.size();
        if (l == 0) {
            // [T][kk0 = 0, 1][lane]: A[m][h] = W[32 T + m][2 kk0 + h]
            blob.resize(off + (size_t)NT * 2 * 64, 0.0f);
            for (int T = 0; T < NT; ++T)
                for (int kk = 0; kk < 2; ++kk)
                    for (int ln = 0; ln < 64; ++ln) {
                        const int row = 32 * T + (ln & 31), k = 2 * kk + (ln >> 5);
                        if (row < M && k < K) blob[off + (size_t)(T * 2 + kk) * 64 + ln] = W[l][(size_t)row * K + k];
                    }
        } else {
            // [group g = pair * NQ + q][tile j of the pair][lane][4 k steps]; the output layer is one tile
            const bool last = (l == L - 1);
            const int chn = last ? 1 : CHN, tiles = last ? 1 : NT, NQ = NR / 4;
            blob.resize(off + (size_t)tiles * NR * 64, 0.0f);
            for (int p = 0; p < tiles / chn; ++p)
                for (int q = 0; q < NQ; ++q)
                    for (int j = 0; j < chn; ++j)
                        for (int ln = 0; ln < 64; ++ln)
                            for (int i = 0; i < 4; ++i) {
                                const int row = 32 * (p * chn + j) + (ln & 31);
                                const int k = flt_feature(4 * q + i, ln >> 5);
                                if (row < M && k < K)
                                    blob[off + ((size_t)((p * NQ + q) * chn + j) * 64 + ln) * 4 + i] = W[l][(size_t)row * K + k];
                            }
        }
        P->args.layer[l].w_off = (uint32_t)off;
        P->args.layer[l].b_off = bias_block(l, l == L - 1 ? 1 : NT, l != L - 1);
    }
    P->blob_floats = blob.size();
    if (hipMalloc((void **)&P->blob_dev, sizeof(float) * blob.size()) != hipSuccess) return DHQ_ENOMEM;
    if (hipMemcpy(P->blob_dev, blob.data(), sizeof(float) * blob.size(), hipMemcpyHostToDevice) != hipSuccess) return DHQ_EHIP;
    P->args.blob = P->blob_dev;
    P->args.n_layers = L;
    P->args.k0 = dims[0];
    P->args.m_out = dims[L];
    P->args.rev = (float)rev;
    P->args.c2 = P->actf.c2;
    return DHQ_OK;
}

// The three bf16 pieces of an fp32 value (nearest even; a value whose first piece would round beyond the largest bf16 is
// truncated instead).
static uint16_t host_bf16(float v)
{
    uint32_t u;
    memcpy(&u, &v, 4);
    uint32_t r = u + 0x7fffu + ((u >> 16) & 1u);
    if (((r >> 23) & 0xffu) == 0xffu) r = u;
    return (uint16_t)(r >> 16);
}
static float host_from_bf16(uint16_t b)
{
    const uint32_t u = (uint32_t)b << 16;
    float v;
    memcpy(&v, &u, 4);
    return v;
}
// A row of n values as three rows of pieces.
static void host_split3(const float *a, int n, uint16_t *hi, uint16_t *mid, uint16_t *lo)
{
    for (int i = 0; i < n; ++i) {
        float r = a[i];
        hi[i] = host_bf16(r);
        r -= host_from_bf16(hi[i]);
        mid[i] = host_bf16(r);
        lo[i] = host_bf16(r - host_from_bf16(mid[i]));
    }
}

// Fragments, biases and the two activation buffers of the layer-by-layer path.
static int float_create_layerwise(dhq_float_plan *P, const int *dims, int L, double rev, const std::vector<std::vector<float>> &W,
                                  const std::vector<std::vector<float>> &b)
{
    int max_nkb = 1;
    P->narrow = true;
    size_t w_off[DHQ_MAX_LAYERS], b_off[DHQ_MAX_LAYERS], bytes = 0;
    for (int l = 0; l < L; ++l) {
        float_lw_layer &Ly = P->lw[l];
        Ly.K = dims[l];
        Ly.M = dims[l + 1];
        Ly.nkb = (l == 0) ? (Ly.K + 31) / 32 * 2 : 2 * P->lw[l - 1].Mt;  // even
        Ly.Mt = (Ly.M + 31) / 32;
        if (Ly.nkb > max_nkb) max_nkb = Ly.nkb;
        if (Ly.nkb > 4) P->narrow = false;
        w_off[l] = bytes;
        b_off[l] = bytes + (size_t)Ly.Mt * Ly.nkb * 3072;
        bytes = (b_off[l] + (size_t)Ly.Mt * 128 + 1023) / 1024 * 1024;
    }
    std::vector<unsigned char> blob(bytes, 0);
    for (int l = 0; l < L; ++l) {
        const float_lw_layer &Ly = P->lw[l];
        uint16_t *frag = reinterpret_cast<uint16_t *>(blob.data() + w_off[l]);
        std::vector<uint16_t> pieces((size_t)3 * Ly.nkb * 16, 0);  // of one row, zero beyond K
        for (int f = 0; f < Ly.M; ++f) {
            uint16_t *row[3] = {pieces.data(), pieces.data() + Ly.nkb * 16, pieces.data() + 2 * Ly.nkb * 16};
            host_split3(W[l].data() + (size_t)f * Ly.K, Ly.K, row[0], row[1], row[2]);
            for (int kb = 0; kb < Ly.nkb; ++kb)
                for (int h = 0; h < 2; ++h) {
                    // slots 0..3 and 4..7 of a lane are four consecutive k each
                    const int k0 = (l == 0) ? 16 * kb + 8 * h : flt_feature(8 * kb, h), k4 = (l == 0) ? k0 + 4 : flt_feature(8 * kb + 4, h);
                    uint16_t *dst = frag + ((size_t)((f >> 5) * Ly.nkb + kb) * 3 * 64 + 32 * h + (f & 31)) * 8;
                    for (int p = 0; p < 3; ++p) {
                        memcpy(dst + (size_t)p * 512, row[p] + k0, 8);
                        memcpy(dst + (size_t)p * 512 + 4, row[p] + k4, 8);
                    }
                }
        }
        float *bias = reinterpret_cast<float *>(blob.data() + b_off[l]);
        for (int T = 0; T < Ly.Mt; ++T)
            for (int h = 0; h < 2; ++h)
                for (int v = 0; v < 16; ++v) {
                    const int f = flt_feature(16 * T + v, h);
                    if (f < Ly.M) bias[(size_t)(T * 2 + h) * 16 + v] = (l != L - 1) ? (float)((double)b[l][f] * rev) : b[l][f];
                }
    }
    if (hipMalloc((void **)&P->lw_blob_dev, bytes) != hipSuccess) return DHQ_ENOMEM;
    if (hipMemcpy(P->lw_blob_dev, blob.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) return DHQ_EHIP;
    for (int l = 0; l < L; ++l) {
        P->lw[l].wfrag_dev = P->lw_blob_dev + w_off[l];
        P->lw[l].bias_dev = reinterpret_cast<const float *>(P->lw_blob_dev + b_off[l]);
    }
    // bytes of 32 rows of the widest hidden layer: fragments, or floats in the narrow networks
    int max_mt = 1;
    for (int l = 0; l < L - 1; ++l) max_mt = P->lw[l].Mt > max_mt ? P->lw[l].Mt : max_mt;
    const int64_t tile_bytes = P->narrow ? (int64_t)max_mt * 4096 : (int64_t)max_nkb * 3072;
    P->chunk_rows = ((P->narrow ? FLT_ACT_BYTES_NARROW : FLT_ACT_BYTES) / tile_bytes * 32) / 256 * 256;
    if (dhq_float_shape_ok(dims, L) && dims[1] != 256 && P->chunk_rows > DHQ_CHUNK) P->chunk_rows = DHQ_CHUNK;
    const size_t act_bytes = (size_t)(P->chunk_rows / 32 * tile_bytes);
    if (hipMalloc((void **)&P->act[0], 2 * act_bytes) != hipSuccess) return DHQ_ENOMEM;
    P->act[1] = P->act[0] + act_bytes;
    return DHQ_OK;
}

void dhq_float_destroy(dhq_float_plan *P)
{
    if (!P) return;
    if (P->blob_dev) (void)hipFree(P->blob_dev);
    if (P->lw_blob_dev) (void)hipFree(P->lw_blob_dev);
    if (P->act[0]) (void)hipFree(P->act[0]);
    delete P;
}

bool dhq_float_has_fused(const dhq_float_plan *P) { return P && P->nf != 0; }

template <int ACT, int WF, int WC, int TF, int TC, int KS>
static hipError_t float_layer_launch_t(float_layer_args a, int device, hipStream_t st)
{
    using tile_t = float_layer_tile<ACT, WF, WC, TF, TC, KS>;
    auto kern = float_layer_kernel<ACT, WF, WC, TF, TC, KS>;
    const size_t lds = (size_t)3 * tile_t::BLOCKS * 1024;
    const hipError_t e = dhq_lds_limit_once(kern, lds, device);
    if (e != hipSuccess) return e;
    a.nF = (a.n_ft + tile_t::FT - 1) / tile_t::FT;
    a.nC = (a.n_ct + tile_t::CT - 1) / tile_t::CT;
    kern<<<(unsigned)((a.nC + 7) / 8 * 8 * a.nF), 64 * WF * WC, lds, st>>>(a);
    return hipGetLastError();
}

// The tile shape (features x coordinates of a workgroup) with the least time for its fullest CU: workgroups per CU, rounded
// up, times what one costs in MFMA tiles.  The cost of a tile is 1 where a workgroup computes 128 x 256 (the fewest LDS and
// L2 bytes per MFMA), 1.2 at 64 x 256 and 128 x 128, 2 at 128 x 32.  Measured, whole forwards in us, for the four in that order:
//   width 512 x 65 536 rows  559  605  603  891        width 300 x 33 000 rows  167  155  184  244
//   width 512 x 9 000 rows   139  139  139  160        width 100 x 100 000 rows 118  135  136  160
//   width 512 x 4 000 rows   137   96   98   84        width 48 x 100 000 rows   76   71   91  110
template <int ACT>
static hipError_t float_layer_launch(const float_layer_args &a, int n_cu, int device, hipStream_t st)
{
    const int64_t f4 = (a.n_ft + 3) / 4, f2 = (a.n_ft + 1) / 2, c8 = (a.n_ct + 7) / 8, c4 = (a.n_ct + 3) / 4;
    auto cost = [&](int64_t workgroups, int64_t each) { return (workgroups + n_cu - 1) / n_cu * each; };
    const int64_t c128x256 = cost(f4 * c8, 32), c64x256 = cost(f2 * c8, 19), c128x128 = cost(f4 * c4, 19), c128x32 = cost(f4 * a.n_ct, 8);
    const int64_t least = std::min(std::min(c128x256, c64x256), std::min(c128x128, c128x32));
    if (c128x32 == least) return float_layer_launch_t<ACT, 4, 1, 1, 1, 2>(a, device, st);
    if (c128x128 == least) return float_layer_launch_t<ACT, 2, 2, 2, 2, 2>(a, device, st);
    if (c64x256 == least) return float_layer_launch_t<ACT, 1, 4, 2, 2, 2>(a, device, st);
    return float_layer_launch_t<ACT, 1, 4, 4, 2, 1>(a, device, st);
}

template <int ACT, int NT, bool FIRST, bool LAST>
static hipError_t float_narrow_launch_t(const float_narrow_args &a, int nkb, int m_tiles, int n_cu, hipStream_t st)
{
    const int want = (a.n_ct + 3) / 4, most = 4 * n_cu;
    const dim3 grid((unsigned)(want < most ? want : most), (unsigned)(LAST ? m_tiles : 1));
    if (nkb == 2) float_narrow_kernel<ACT, NT, 2, FIRST, LAST><<<grid, 256, 0, st>>>(a);
    else float_narrow_kernel<ACT, NT, 4, FIRST, LAST><<<grid, 256, 0, st>>>(a);
    return hipGetLastError();
}
template <int ACT>
static hipError_t float_narrow_launch(const dhq_float_plan *P, int l, const float_narrow_args &a, hipStream_t st)
{
    const float_lw_layer &Ly = P->lw[l];
    const bool first = (l == 0), last = (l == P->n_layers - 1);
    if (last)
        return first ? float_narrow_launch_t<DHQ_ACT_KIND_NONE, 1, true, true>(a, Ly.nkb, Ly.Mt, P->n_cu, st)
                     : float_narrow_launch_t<DHQ_ACT_KIND_NONE, 1, false, true>(a, Ly.nkb, Ly.Mt, P->n_cu, st);
    if (Ly.Mt == 1)
        return first ? float_narrow_launch_t<ACT, 1, true, false>(a, Ly.nkb, 1, P->n_cu, st)
                     : float_narrow_launch_t<ACT, 1, false, false>(a, Ly.nkb, 1, P->n_cu, st);
    return first ? float_narrow_launch_t<ACT, 2, true, false>(a, Ly.nkb, 1, P->n_cu, st)
                 : float_narrow_launch_t<ACT, 2, false, false>(a, Ly.nkb, 1, P->n_cu, st);
}

hipError_t dhq_float_launch_layerwise(const dhq_float_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    if (!P) return hipErrorInvalidValue;
    const int L = P->n_layers;
    if (n <= 0) return hipSuccess;
    // as few chunks as the buffers allow, of equal size
    const int64_t chunks = (n + P->chunk_rows - 1) / P->chunk_rows, per = (n + chunks - 1) / chunks, step = (per + 255) / 256 * 256;
    for (int64_t start = 0; start < n; start += step) {
        const int64_t rows = (n - start < step) ? n - start : step;
        const int n_ct = (int)((rows + 31) / 32);
        if (P->narrow) {
            for (int l = 0; l < L; ++l) {
                const float_lw_layer &Ly = P->lw[l];
                float_narrow_args a;
                memset(&a, 0, sizeof(a));
                a.in = (l == 0) ? coords + start * Ly.K : reinterpret_cast<const float *>(P->act[l & 1]);
                a.out = (l == L - 1) ? out + start * Ly.M : reinterpret_cast<float *>(P->act[(l + 1) & 1]);
                a.w = Ly.wfrag_dev;
                a.bias = Ly.bias_dev;
                a.n = rows;
                a.n_ct = n_ct;
                a.K = Ly.K;
                a.M = Ly.M;
                a.rev = P->rev;
                a.c2 = P->actf.c2;
                const hipError_t e = P->actf.kind == DHQ_ACT_KIND_WAVELET ? float_narrow_launch<DHQ_ACT_KIND_WAVELET>(P, l, a, st)
                                                                          : float_narrow_launch<DHQ_ACT_KIND_SINE>(P, l, a, st);
                if (e != hipSuccess) return e;
            }
            continue;
        }
        const int64_t n_frag = (int64_t)n_ct * P->lw[0].nkb;
        float_pack_kernel<<<(unsigned)((n_frag + 3) / 4), 256, 0, st>>>(coords + start * P->lw[0].K, rows, P->lw[0].K, P->lw[0].nkb, n_frag,
                                                                        P->act[0]);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        for (int l = 0; l < L; ++l) {
            const float_lw_layer &Ly = P->lw[l];
            if (l == L - 1) {
                const dim3 grid((unsigned)((n_ct + 3) / 4), (unsigned)Ly.Mt);
                float_out_kernel<<<grid, 256, 0, st>>>(P->act[l & 1], Ly.wfrag_dev, Ly.bias_dev, rows, n_ct, Ly.nkb, Ly.M, out + start * Ly.M);
                e = hipGetLastError();
            } else {
                float_layer_args a;
                memset(&a, 0, sizeof(a));
                a.in = P->act[l & 1];
                a.out = P->act[(l + 1) & 1];
                a.w = Ly.wfrag_dev;
                a.bias = Ly.bias_dev;
                a.n_ct = n_ct;
                a.n_ft = Ly.Mt;
                a.nkb = Ly.nkb;
                a.rev = P->rev;
                a.c2 = P->actf.c2;
                e = P->actf.kind == DHQ_ACT_KIND_WAVELET ? float_layer_launch<DHQ_ACT_KIND_WAVELET>(a, P->n_cu, P->device, st)
                                                         : float_layer_launch<DHQ_ACT_KIND_SINE>(a, P->n_cu, P->device, st);
            }
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t dhq_float_launch(const dhq_float_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    if (!P || P->nf == 0) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    // Width 256 has no kernel of its own: one that kept the activations in registers and multiplied on the fp32 matrix
    // instructions was slower than the layer-by-layer kernels at every size.  Measured, that kernel / layer by layer, five
    // hidden layers, us:
    //   rows       1 000     4 096    16 384    65 536      262 144
    //   width 256  142 / 43  142 / 52  151 / 94  304 / 249  1129 / 968
    //   width 128   43 / 31   44 / 34   46 / 54   96 / 125   364 / 429
    //   width 64    16 / 26   16 / 27   17 / 36   33 / 71    119 / 189
    // (At width 128 the line would lie at 8 192 rows; a network's values would then depend in their last bits on how many
    // rows a call brings, so it stays on one path.)
    if (P->nf == 256) return dhq_float_launch_layerwise(P, coords, n, out, st);
    float_args a = P->args;
    a.coords = coords;
    a.out = out;
    a.n = n;
    const int64_t tiles = (n + FLT_TILE - 1) / FLT_TILE;
    const unsigned grid = (unsigned)(tiles < P->n_cu ? tiles : P->n_cu);
    const bool wav = (P->actf.kind == DHQ_ACT_KIND_WAVELET);
    switch (P->nf) {
        case 32:
            if (wav) dhq_float_kernel<32, DHQ_ACT_KIND_WAVELET><<<grid, FLT_THREADS, 0, st>>>(a);
            else dhq_float_kernel<32, DHQ_ACT_KIND_SINE><<<grid, FLT_THREADS, 0, st>>>(a);
            break;
        case 64:
            if (wav) dhq_float_kernel<64, DHQ_ACT_KIND_WAVELET><<<grid, FLT_THREADS, 0, st>>>(a);
            else dhq_float_kernel<64, DHQ_ACT_KIND_SINE><<<grid, FLT_THREADS, 0, st>>>(a);
            break;
        case 128:
            if (wav) dhq_float_kernel<128, DHQ_ACT_KIND_WAVELET><<<grid, FLT_THREADS, 0, st>>>(a);
            else dhq_float_kernel<128, DHQ_ACT_KIND_SINE><<<grid, FLT_THREADS, 0, st>>>(a);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
