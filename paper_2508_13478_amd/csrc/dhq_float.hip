// Forward with floating-point activations (gfx950): the "W32A32" and "W8A32" rows of the paper's comparison (Sec. 1,
// Fig. 1-2, Table 2).  W32A32 is the plain SIREN, y = W a + b, a = sin(omega0 y); W8A32 is the same network run on the weights
// after the offline step and de-quantization, W~ = (s_w Wq) Hn (the caller passes whichever weights apply; the kernels do
// not know the difference).  Weights and activations are fp32 values; the products run on the 16-bit matrix instructions, every
// value as the sum of three bf16 pieces, which hold it without loss.
//
// float_net_kernel runs a whole network, the activations in LDS (float_net_takes).  float_layer_kernel and float_narrow_kernel
// run one layer per launch, activations in device memory between the layers, a chunk of rows at a time: DHQ_LAYERWISE, and the
// networks that the other does not take.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <utility>
#include <vector>

#include "dhq_device.h"
#include "dhq_internal.h"

// Bytes of each of the two activation buffers of the layer-by-layer path: both together stay within the 256 MiB
// memory-side cache, which is worth more than fewer launches (width 512, 262 144 rows: 3.47 ms in chunks of 32 768 rows = 96 MiB
// per buffer, 3.68 ms in chunks of 65 536), while narrower networks take as many rows as fit (width 60: 0.24 ms in chunks of
// 65 536 rows, 0.40 ms in chunks of 32 768).
#define FLT_ACT_BYTES ((int64_t)96 << 20)
// A third of that for the narrow networks, whose rows are short (131 072 rows of 64 features; the launches' latency no longer
// shows), and no more than DHQ_CHUNK rows in the shapes of dhq_float_shape_ok up to 128 wide.
#define FLT_ACT_BYTES_NARROW ((int64_t)32 << 20)

typedef float dhq_v16f __attribute__((ext_vector_type(16)));

// What float_net_kernel needs of a layer and of a network.
struct float_net_layer {
    unsigned w_off, b_off;  // KiB, bytes / 128 in the blob
    unsigned short nkb, Mt;
};
struct float_net_args {
    const float *coords;
    float *out;
    const unsigned char *blob;
    int64_t n;
    int n_blocks, n_layers, k0, m_out;
    int max_kb;  // k blocks of the widest hidden layer's output
    float rev, c2;
    float_net_layer layer[DHQ_MAX_LAYERS];
};

// A layer's weights as fragments of their three bf16 pieces (see float_layer_kernel), biases [feature tile][lane half][16] (times
// omega0 / 2 pi where an activation follows).
struct float_lw_layer {
    const unsigned char *wfrag_dev = nullptr;  // inside the plan's lw_blob_dev, like the biases
    const float *bias_dev = nullptr;
    int K = 0, M = 0, nkb = 0, Mt = 0;
};

struct dhq_float_plan {
    int nf = 0;              // hidden width of the shapes DHQ_FUSED is accepted for, else 0
    int n_cu = 0;
    int n_layers = 0;
    float rev = 0.f;
    dhq_act actf = {DHQ_ACT_KIND_SINE, 0.f};  // what follows every layer but the last
    float_lw_layer lw[DHQ_MAX_LAYERS];
    unsigned char *lw_blob_dev = nullptr;
    unsigned char *act[2] = {nullptr, nullptr};  // chunk_rows rows of fragments of the widest layer
    int64_t chunk_rows = 0;
    float_net_args net;   // the whole-network kernel
    int max_mt = 0;       // feature tiles of the widest hidden layer
    bool narrow = false;  // every layer input up to 64 wide: float_narrow_kernel
    int device = 0;
};

// ----------------------------------------------------------------------------- device code
// ---------------------------------------------------------------- layer by layer, any shape
// One GEMM kernel per layer.  The fp32 MFMA delivers 64 multiply-adds per clock and SIMD, the bf16 one 1024, and three
// bf16 pieces hold an fp32 value without loss: hi = bf16(a), mid = bf16(a - hi), lo = a - hi - mid (rounded to nearest,
// 8 significant bits each, both differences exact).  So every product a w is taken as the six bf16 products whose
// weight is at least 2^-17 of it,
//     hi hi + (hi mid + mid hi) + (hi lo + mid mid + lo hi),
// each exact in the MFMA and summed in fp32.  Left out are mid lo, lo mid and lo lo: at most 2^-24 of |a w| together,
// half an ulp of the product, with a random sign.  (The MFMA takes subnormal pieces as zero: bits of a value below 2^-126.)  A layer then costs 6 / 16 of the fp32 MFMA time.
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
// operands).  The fp32 MFMA form of this kernel took 370 us.  Relative error of the outputs against fp64 (20 000 rows; the same network
// on the fp32 MFMA, which rounds after every two products instead of every sixteen, in brackets): sine, 5 layers of 64 2.1e-7 (2.3e-7),
// of 128 3.2e-7 (3.4e-7), of 512 7.2e-7; wavelet, s0 = 10, 5 layers of 64 6.3e-8 (7.5e-8), of 128 1.1e-7 (1.2e-7).
typedef __bf16 flt_v8b __attribute__((ext_vector_type(8)));
typedef __bf16 flt_v2b __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned flt_pack_bf16(float a, float b)
{
    const flt_v2b p = {(__bf16)a, (__bf16)b};  // one packed conversion, rounded to nearest even
    return __builtin_bit_cast(unsigned, p);
}
// The three bf16 pieces of two values, value 0 in the low halves.  INPUT: coordinates, which may be beyond the largest bf16; the first
// piece of one that would round to infinity is truncated instead (activations are at most 1).
template <bool INPUT = false>
__device__ __forceinline__ void flt_split3(float a0, float a1, unsigned &hi, unsigned &mid, unsigned &lo)
{
// (what is split is an fp32 value: the wavelet's last product must not melt into the subtractions, in one kernel and not in another)
#pragma clang fp contract(off)
    hi = flt_pack_bf16(a0, a1);
    if constexpr (INPUT) {
        const unsigned u0 = __float_as_uint(a0), u1 = __float_as_uint(a1);
        if ((u0 & 0x7fffffffu) - 0x7f7f8000u < 0x8000u) hi = (hi & 0xffff0000u) | u0 >> 16;
        if ((u1 & 0x7fffffffu) - 0x7f7f8000u < 0x8000u) hi = (hi & 0xffffu) | (u1 & 0xffff0000u);
    }
    const float r0 = a0 - __uint_as_float(hi << 16), r1 = a1 - __uint_as_float(hi & 0xffff0000u);
    mid = flt_pack_bf16(r0, r1);
    lo = flt_pack_bf16(r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xffff0000u));
}
// Eight values as a lane's 16 bytes of each of the three fragments.
template <bool INPUT = false>
__device__ __forceinline__ void flt_split(const float (&y)[8], dhq_v4i (&x)[3])
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        unsigned hi, mid, lo;
        flt_split3<INPUT>(y[2 * d], y[2 * d + 1], hi, mid, lo);
        x[0][d] = (int)hi; x[1][d] = (int)mid; x[2][d] = (int)lo;
    }
}
// The fragments at dst, dst + 1 KiB, dst + 2 KiB.
template <bool INPUT = false>
__device__ __forceinline__ void flt_store_pieces(const float (&y)[8], unsigned char *__restrict__ dst)
{
    dhq_v4i x[3];
    flt_split<INPUT>(y, x);
#pragma unroll
    for (int i = 0; i < 3; ++i) *reinterpret_cast<dhq_v4i *>(dst + i * 1024) = x[i];
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

// The activation on any finite argument.  The whole revolutions are taken off by rounding, not by the fractional part: an argument
// of less than half of one stays as it is, where a small negative one's fractional part, 1 + t, is t rounded to 2^-24.
__device__ __forceinline__ float flt_activate(float t, dhq_act act)
{
    const float f = t - __builtin_rintf(t);
    if (act.kind == DHQ_ACT_KIND_WAVELET) {
        const float g = t * act.c2;
        return __builtin_amdgcn_cosf(f) * __builtin_amdgcn_exp2f(-(g * g));
    }
    return __builtin_amdgcn_sinf(f);
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
    flt_store_pieces<true>(y, out + (size_t)w * 3072 + lane * 16);
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
                    y[j] = flt_activate(__builtin_fmaf(R.acc[f][c][8 * b + j], A.rev, bias[8 * b + j]), dhq_act{ACT, A.c2});
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
// are split into pieces by the wave that reads them: the same pieces, products and order of sums as above, so the same bits.
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
                flt_split3<FIRST>(v[kb][2 * d], v[kb][2 * d + 1], hi, mid, lo);
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
                        y[e] = flt_activate(__builtin_fmaf(acc[T][4 * q + e], A.rev, bias[T][4 * q + e]), dhq_act{ACT, A.c2});
                    dst[q * 64] = make_float4(y[0], y[1], y[2], y[3]);
                }
            }
        }
    }
}

// ------------------------------------------------------------- the whole network in one kernel
// A workgroup carries CT = WC TC tiles of 32 coordinates through all layers; their activations lie in LDS, in the fragments
// above ([coordinate tile][k block][piece][lane] x 16 B), and nothing but coordinates and outputs crosses device memory.  The
// WF WC waves split a layer's output: wave (wf, wc) computes feature tiles wf TF .. + TF - 1 of coordinate tiles wc TC ..
// + TC - 1 in its accumulators, takes them through the epilogue, and when all waves have read their inputs the activations'
// pieces take the inputs' place.  A weight fragment is used by one wave (or WC of them) only: it comes from L2 straight into
// registers, a stage (KS k blocks) ahead of its MFMAs.  Biases go through LDS, a layer ahead.
// The sums' order is the layer-by-layer kernels', so the values are theirs bit for bit.
//
// Bound by the matrix unit and, where few coordinates share a weight fragment, by the weights' way into the registers.  Four layers of
// 256, 262 144 rows: 580 us (layer by layer 744) = 1.07 PFLOP/s of bf16 products.  The activations stay in the accumulators until every
// wave has read its inputs and are split then: split before, a tile of 64 x 64 kept 140 bytes a lane in scratch memory.
template <int ACT, int WF, int WC, int TF, int TC, int KS>
__global__ __launch_bounds__(64 * WF * WC, TF * TC <= 4 ? 2 : 1) void float_net_kernel(const float_net_args A)
{
    constexpr int NW = WF * WC, CT = WC * TC, NG = 6 * KS;  // products of a stage
    constexpr int NLW = 3 * KS * TF;                        // weight fragments of a stage and wave
    constexpr bool ALONE = WF == 1 && TF == 1;              // a wave has all of its coordinates' features: no barriers
    constexpr int pw[6] = {0, 2, 1, 0, 1, 0}, px[6] = {2, 0, 1, 1, 0, 0};  // as in flt_mfma6
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wf = wave % WF, wc = wave / WF;
    const int L = A.n_layers, ct_bytes = A.max_kb * 3072;
    unsigned char *act = lds + wc * TC * ct_bytes + lane * 16;
    float *bm = reinterpret_cast<float *>(lds + CT * ct_bytes);  // [feature tile][lane half][16 biases]
    dhq_v16f acc[TF][TC];
    dhq_v4i w[2][KS][TF][3];  // the weights of two stages

    // this thread's share of layer l's biases
    auto fetch_bias = [&](int l) {
        const float4 *src = reinterpret_cast<const float4 *>(A.blob + (size_t)A.layer[l].b_off * 128);
        return tid < A.layer[l].Mt * 8 ? src[tid] : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    auto store_bias = [&](int l, float4 v) {
        if (tid < A.layer[l].Mt * 8) reinterpret_cast<float4 *>(bm)[tid] = v;
    };
    // the weights of the wave's f-th feature tile in layer l (tiles past the last one: the last one's, not used)
    auto weights_of = [&](int l, int f) {
        const int T = wf * TF + f, Tc = T < A.layer[l].Mt ? T : A.layer[l].Mt - 1;
        return A.blob + ((size_t)A.layer[l].w_off + (size_t)Tc * A.layer[l].nkb * 3) * 1024;
    };
    const unsigned voff = lane * 16;

    float4 own[4];  // ALONE: the lane's biases
    auto fetch_own = [&](int l) {
#pragma unroll
        for (int i = 0; i < 4; ++i) own[i] = reinterpret_cast<const float4 *>(A.blob + (size_t)A.layer[l].b_off * 128)[h * 4 + i];
    };

    float4 bias_next;
    if constexpr (!ALONE) bias_next = fetch_bias(0);
    for (int block = blockIdx.x; block < A.n_blocks; block += gridDim.x) {
        const int64_t row0 = (int64_t)block * (CT * 32);
        if constexpr (ALONE) fetch_own(0);
        else store_bias(0, bias_next);
#pragma unroll
        for (int f = 0; f < TF; ++f)
#pragma unroll
            for (int t = 0; t < TC; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[f][t][v] = 0.f;
        // the input layer: coordinates in natural k order
        if (wf * TF < A.layer[0].Mt) {
            const int nkb = A.layer[0].nkb;
            const dhq_v4i *w0 = reinterpret_cast<const dhq_v4i *>(A.blob + (size_t)A.layer[0].w_off * 1024) + lane;
            for (int kb = 0; 16 * kb < A.k0; ++kb) {
                dhq_v4i x[TC][3];
#pragma unroll
                for (int t = 0; t < TC; ++t) {
                    const int64_t row = row0 + (wc * TC + t) * 32 + c;
                    const int kk = 16 * kb + 8 * h;
                    float y[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) y[j] = (row < A.n && kk + j < A.k0) ? A.coords[row * A.k0 + kk + j] : 0.f;
                    flt_split<true>(y, x[t]);
                }
#pragma unroll
                for (int f = 0; f < TF; ++f) {
                    const int T = wf * TF + f, Tc = T < A.layer[0].Mt ? T : A.layer[0].Mt - 1;
                    dhq_v4i wk[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) wk[p] = w0[((size_t)Tc * nkb + kb) * 192 + p * 64];
#pragma unroll
                    for (int t = 0; t < TC; ++t) acc[f][t] = flt_mfma6(wk, x[t], acc[f][t]);
                }
            }
        }
        if constexpr (!ALONE) __syncthreads();  // the input layer's biases are in place
        for (int l = 0; l < L - 1; ++l) {
            // here: layer l's sums in the accumulators of the waves that have tiles in it
            const int Mt = A.layer[l].Mt, ns = 2 * Mt / KS;  // stages of the next layer
            const bool busy = wf * TF < Mt;
            const int ln = l + 1 < L - 1 ? l + 1 : 0;  // whose biases come next
            if constexpr (!ALONE) bias_next = fetch_bias(ln);
            const unsigned char *wp[TF];
            if (l + 1 < L - 1) {
#pragma unroll
                for (int f = 0; f < TF; ++f) {
                    wp[f] = weights_of(l + 1, f);
#pragma unroll
                    for (int k = 0; k < KS; ++k)
#pragma unroll
                        for (int p = 0; p < 3; ++p) w[0][k][f][p] = *reinterpret_cast<const dhq_v4i *>(wp[f] + voff + (k * 3 + p) * 1024);
                }
            }
            if (busy) {  // the activations, in the sums' place
#pragma unroll
                for (int f = 0; f < TF; ++f) {
                    const int T = wf * TF + f, Tc = T < Mt ? T : Mt - 1;
                    const float4 *bp = reinterpret_cast<const float4 *>(bm + (Tc * 2 + h) * 16);
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        float bias[8];
#pragma unroll
                        for (int i = 0; i < 2; ++i) *reinterpret_cast<float4 *>(&bias[4 * i]) = ALONE ? own[2 * b + i] : bp[2 * b + i];
#pragma unroll
                        for (int t = 0; t < TC; ++t)
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                acc[f][t][8 * b + j] = flt_activate(__builtin_fmaf(acc[f][t][8 * b + j], A.rev, bias[j]), dhq_act{ACT, A.c2});
                    }
                }
            }
            if constexpr (!ALONE) __syncthreads();  // every wave has read layer l's inputs and its biases
            if (busy) {
#pragma unroll
                for (int f = 0; f < TF; ++f) {
                    const int T = wf * TF + f;
                    if (T < Mt) {
#pragma unroll
                        for (int t = 0; t < TC; ++t)
#pragma unroll
                            for (int b = 0; b < 2; ++b) {
                                float y[8];
#pragma unroll
                                for (int j = 0; j < 8; ++j) y[j] = acc[f][t][8 * b + j];
                                flt_store_pieces(y, act + t * ct_bytes + (2 * T + b) * 3072);
                            }
                    }
                }
            }
            if constexpr (ALONE) {
                if (l + 1 < L - 1) fetch_own(l + 1);
            } else {
                store_bias(ln, bias_next);
                __syncthreads();
            }
            if (l + 1 == L - 1 || wf * TF >= A.layer[l + 1].Mt) continue;
            // layer l + 1's sums
#pragma unroll
            for (int f = 0; f < TF; ++f)
#pragma unroll
                for (int t = 0; t < TC; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[f][t][v] = 0.f;
            dhq_v4i x[2][TC][3];
#pragma unroll
            for (int t = 0; t < TC; ++t)
#pragma unroll
                for (int p = 0; p < 3; ++p) x[0][t][p] = *reinterpret_cast<const dhq_v4i *>(act + t * ct_bytes + p * 1024);
            auto stage = [&](auto B, int s) {
                constexpr int wb = decltype(B)::value;
                const int sn = s + 1 < ns ? s + 1 : s;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const int k = g / 6, i = g % 6, xb = (wb * KS + k) & 1;
                    // the next stage's weights, spread over the first two thirds of the groups
#pragma unroll
                    for (int q = 0; q < NLW; ++q)
                        if (q * (4 * KS) / NLW == g) {
                            const int k2 = q / (3 * TF), f = (q / 3) % TF, p = q % 3;
                            w[wb ^ 1][k2][f][p] = *reinterpret_cast<const dhq_v4i *>(wp[f] + (size_t)sn * (KS * 3072) + voff + (k2 * 3 + p) * 1024);
                        }
                    if (i == 0) {  // the next k block's activations
                        const int kn = k + 1 < KS ? s * KS + k + 1 : sn * KS;
#pragma unroll
                        for (int t = 0; t < TC; ++t)
#pragma unroll
                            for (int p = 0; p < 3; ++p) x[xb ^ 1][t][p] = *reinterpret_cast<const dhq_v4i *>(act + t * ct_bytes + (kn * 3 + p) * 1024);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int f = 0; f < TF; ++f)
#pragma unroll
                        for (int t = 0; t < TC; ++t)
                            acc[f][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(flt_v8b, w[wb][k][f][pw[i]]),
                                                                                __builtin_bit_cast(flt_v8b, x[xb][t][px[i]]), acc[f][t], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // ahead of the other workgroup's epilogue on the SIMD, which fills what the products leave
            __builtin_amdgcn_s_setprio(3);
            int s = 0;
            for (; s + 1 < ns; s += 2) {
                stage(std::integral_constant<int, 0>{}, s);
                stage(std::integral_constant<int, 1>{}, s + 1);
            }
            if (s < ns) stage(std::integral_constant<int, 0>{}, s);
            __builtin_amdgcn_s_setprio(0);
        }
        // the output layer: tiles of 32 outputs x 32 coordinates dealt over the waves
        {
            const int Mt = A.layer[L - 1].Mt, nkb = A.layer[L - 1].nkb;
            for (int job = ALONE ? 0 : wave; job < (ALONE ? TC : CT) * Mt; job += ALONE ? 1 : NW) {
                const int t = ALONE ? wave * TC + job % TC : job % CT, T = job / (ALONE ? TC : CT);
                const dhq_v4i *wo = reinterpret_cast<const dhq_v4i *>(A.blob + (size_t)A.layer[L - 1].w_off * 1024) + (size_t)T * nkb * 192 + lane;
                const dhq_v4i *xo = reinterpret_cast<const dhq_v4i *>(lds + t * ct_bytes) + lane;
                dhq_v16f o;
#pragma unroll
                for (int v = 0; v < 16; ++v) o[v] = 0.f;
                for (int kb0 = 0; kb0 < nkb; kb0 += 2) {  // (an even number of k blocks)
                    dhq_v4i wk[2][3], xk[2][3];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int p = 0; p < 3; ++p) {
                            wk[k][p] = wo[((kb0 + k) * 3 + p) * 64];
                            xk[k][p] = xo[((kb0 + k) * 3 + p) * 64];
                        }
#pragma unroll
                    for (int k = 0; k < 2; ++k) o = flt_mfma6(wk[k], xk[k], o);
                }
                const int64_t row = row0 + t * 32 + c;
                if (row < A.n) {
                    const float *bo = reinterpret_cast<const float *>(A.blob + (size_t)A.layer[L - 1].b_off * 128) + (T * 2 + h) * 16;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int f = 32 * T + 8 * (v >> 2) + 4 * h + (v & 3);
                        if (f < A.m_out) A.out[row * A.m_out + f] = o[v] + bo[v];
                    }
                }
            }
        }
        // (the next block's first write to the activations comes behind two barriers)
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
    P->nf = dhq_float_shape_ok(dims, L) ? dims[1] : 0;
    const int rc = float_create_layerwise(P, dims, L, rev, W, b);
    if (rc != DHQ_OK) {
        dhq_float_destroy(P);
        return rc;
    }
    *plan_out = P;
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
    memset(&P->net, 0, sizeof(P->net));
    for (int l = 0; l < L; ++l) {
        P->net.layer[l].w_off = (unsigned)(w_off[l] / 1024);
        P->net.layer[l].b_off = (unsigned)(b_off[l] / 128);
        P->net.layer[l].nkb = (unsigned short)P->lw[l].nkb;
        P->net.layer[l].Mt = (unsigned short)P->lw[l].Mt;
        if (l < L - 1) P->max_mt = std::max(P->max_mt, P->lw[l].Mt);
    }
    P->net.blob = P->lw_blob_dev;
    P->net.n_layers = L;
    P->net.k0 = dims[0];
    P->net.m_out = dims[L];
    P->net.max_kb = 2 * P->max_mt;
    P->net.rev = P->rev;
    P->net.c2 = P->actf.c2;
    // bytes of 32 rows of the widest hidden layer: fragments, or floats in the narrow networks
    const int max_mt = std::max(P->max_mt, 1);
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

// Whether float_net_kernel takes a network and n rows (the values are the same).  Its tiles hold six bytes a hidden feature and coordinate
// in LDS: two of 32 coordinates up to 13 feature tiles, one beyond, where the weights' way into the registers takes longer than the
// layer-by-layer kernels' way through memory, except in the few rows that leave those short of workgroups.  Every wave of a tile
// loads and splits its coordinates for itself, and an output tile is one wave's, which large fan-ins and fan-outs make the
// longest part.  Whole forwards in us, here / layer by layer, by rows:
//                          100          1 000        5 000        20 000       65 536       262 144
//   2 x 400 (six layers)   88 / 77      87 / 81      86 / 127     294 / 291    614 / 713    2411 / 3206
//   64 x 256 x 256 x 3     17 / 22      18 / 23      18 / 31      37 / 53      90 / 111     346 / 418
//   256 x 256 x 256 x 256  37 / 32      37 / 34      38 / 51      87 / 93      230 / 204    870 / 841
//   512 x 128 x 128 x 3    42 / 25      43 / 27      43 / 38      127 / 66     247 / 172    1005 / 778
//   512 x 64 x 64 x 3      43 / 22      43 / 24      43 / 34      77 / 59      126 / 154    511 / 707
//   512 x 32 x 32 x 3      22 / 21      23 / 23      22 / 32      39 / 55      75 / 145     289 / 663
//   2 x 256 x 256 x 512    35 / 25      36 / 25      40 / 44      74 / 151     193 / 456    767 / 1823
//   2 x 128 x 128 x 300    20 / 19      21 / 20      22 / 26      47 / 78      100 / 161    415 / 691
//   2 x 64 x 64 x 512      40 / 13      43 / 13      44 / 20      53 / 49      110 / 105    565 / 428
// With nine to eleven feature tiles and few rows one launch saves 2.5 us against one per layer where 32 rows are all there is, 6.5 us
// beyond, and its weights' way into the registers takes about one more for every tile beyond eight of every hidden layer but the
// first, and one for every 16 inputs beyond the first 16 (a fit over 1 to 6 hidden layers, fan-ins of 2, 40 and 64, sine and
// wavelet; where the rule is wrong, it is by 10 % at most).  Three layers of 352, fan-in 40, sine: 1 row 32.5 / 27.8, 64 rows 35.7 / 33.3, 300 rows 36.0 / 36.5;
// six of 257, fan-in 2: 1 row 48.3 / 46.5, 64 rows 49.7 / 51.1.
// With nine to thirteen tiles a round of the chip takes as long for one coordinate tile as for all: beyond two rounds both ways' times in us,
// fitted over 257 to 416 features, 1, 2 and 4 hidden layers and fan-ins of 2 to 64 (rms 10 %), say which is faster.  257 features, two
// hidden layers: fan-in 2, 51 200 rows (a fourth round with an eighth of its tiles) at 0.89 of the layer kernels' rate; fan-in 64 0.69.
// One hidden layer behind a large fan-in: 64 x 128 x 3, 81 920 rows at 0.81; 64 x 64 x 3 at 0.90; 64 x 200 x 3, 51 200 rows at 0.91.
static bool float_net_takes(const dhq_float_plan *P, int64_t n)
{
    const int64_t round = 32 * (int64_t)P->n_cu;
    const int L = P->n_layers, K = P->lw[0].K, mt = P->max_mt;
    if (L < 2) return false;
    if (mt > 13 ? n <= round / 4 || n > round : mt > 11 && n <= round / 4) return false;
    if (mt > 8 && n <= round / 16 && (mt - 8) * (L - 2) + (K + 15) / 16 - 1 > (n <= 32 ? 2 : 6)) return false;
    const int kb = (K + 15) / 16;
    if (mt > 8 && n > 2 * round) {
        const double x = (double)n / (2 * round);  // rounds of tiles of 64
        const double here = ceil(x) * (7.7 + 3.8 * kb + 1.94 * (L - 2) * mt), layers = 12 + x * (1.25 * (L - 1) * mt + 1.35 * kb + 0.087 * (L - 2) * mt * mt);
        if (1.03 * here > layers) return false;
    }
    if (mt <= 8 && L == 2 && (mt <= 2 ? K > 16 && n > (K > 48 ? 2 : 8) * round : K > 48 && n > 6 * round)) return false;
    if (K > 64 && !(mt == 1 && (K <= 256 || n > 1024)) && !(mt == 2 && n > 4 * round)) return false;
    return P->lw[L - 1].Mt == 1 || (mt > 2 && n > round / 2);
}

template <int ACT, int WF, int WC, int TF, int TC, int KS>
static hipError_t float_net_launch_t(const dhq_float_plan *P, float_net_args a, int waves_per_cu, hipStream_t st)
{
    static_assert(64 * WF * WC >= 8 * WF * TF, "a thread carries one float4 of a layer's biases");
    auto kern = float_net_kernel<ACT, WF, WC, TF, TC, KS>;
    const size_t lds = (size_t)WC * TC * a.max_kb * 3072 + (size_t)P->max_mt * 128;
    if (P->max_mt > WF * TF || lds > 160 * 1024) return hipErrorInvalidValue;
    const hipError_t e = dhq_lds_limit_once(kern, 160 * 1024, P->device);
    if (e != hipSuccess) return e;
    const int64_t rows = 32 * WC * TC, blocks = (a.n + rows - 1) / rows;
    const int per_cu = std::max(1, std::min((int)(160 * 1024 / lds), waves_per_cu / (WF * WC)));
    a.n_blocks = (int)blocks;
    const int64_t most = (int64_t)P->n_cu * per_cu;
    kern<<<(unsigned)(blocks < most ? blocks : most), 64 * WF * WC, lds, st>>>(a);
    return hipGetLastError();
}
// The tile of a workgroup, by the widest hidden layer's feature tiles and the rows: few rows take small tiles, as long as the
// launch is one round of the chip (`round`: rows of a tile of 32 per CU); beyond, more coordinates share a weight fragment.
// Whole forwards in us, four hidden layers (512: five), by the rows of a tile, and layer by layer in brackets:
//   rows          4 096               16 384                65 536                  262 144
//   width 32    6.8 (16)            7.2 (16)              8.7 (21)                26 (84)
//   width 64    32: 9.6 (20)        32: 10.0 (21)         32: 20.6, 64: 16 (36)   32: 76, 64: 59 (144)
//   width 128   32: 12, 64: 16 (29) 32: 15, 64: 17 (44)   32: 51, 64: 46 (92)     64: 165, 96: 158 (371)
//   width 256   23 (43)             43 (73)               150 (187)               584 (744); 96 with eight waves: 580
//   width 300   32: 38, 64: 62 (60) 32: 76, 64: 67 (106)  32: 299, 64: 259 (358)  32: 1155, 64: 1003 (1491)
//   width 400   32: 52, 64: 88 (76) 32: 116, 64: 97 (138) 32: 434, 64: 378 (452)  32: 1678, 64: 1476 (1820)
//   width 512   91 (106)            206 (213)             812 (727)               3164 (2895)
template <int ACT>
static hipError_t float_net_launch(const dhq_float_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    float_net_args a = P->net;
    a.coords = coords;
    a.out = out;
    a.n = n;
    const int64_t round = 32 * (int64_t)P->n_cu;
    if (P->max_mt > 8)
        return n <= round || P->max_mt > 13 ? float_net_launch_t<ACT, 8, 1, 2, 1, 1>(P, a, 8, st) : float_net_launch_t<ACT, 8, 1, 2, 2, 1>(P, a, 8, st);
    if (P->max_mt > 4) return float_net_launch_t<ACT, 4, 1, 2, 1, 1>(P, a, 12, st);
    if (P->max_mt > 2)
        return n <= 2 * round   ? float_net_launch_t<ACT, 4, 1, 1, 1, 2>(P, a, 8, st)
               : n <= 8 * round ? float_net_launch_t<ACT, 4, 1, 1, 2, 2>(P, a, 12, st)
                                : float_net_launch_t<ACT, 4, 1, 1, 3, 1>(P, a, 8, st);
    if (P->max_mt > 1)
        return n <= 4 * round ? float_net_launch_t<ACT, 2, 2, 1, 1, 2>(P, a, 8, st) : float_net_launch_t<ACT, 2, 2, 1, 2, 2>(P, a, 8, st);
    return float_net_launch_t<ACT, 1, 1, 1, 1, 2>(P, a, 12, st);
}

hipError_t dhq_float_launch(const dhq_float_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    if (!P) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    if (!float_net_takes(P, n)) return dhq_float_launch_layerwise(P, coords, n, out, st);
    return P->actf.kind == DHQ_ACT_KIND_WAVELET ? float_net_launch<DHQ_ACT_KIND_WAVELET>(P, coords, n, out, st)
                                                : float_net_launch<DHQ_ACT_KIND_SINE>(P, coords, n, out, st);
}
