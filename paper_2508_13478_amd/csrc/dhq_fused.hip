// Whole-network fused DHQ forward for gfx950 (paper Sec. 3.3 pipeline: input layer, linear
// layers with a quantization module between them, output layer -- here one kernel).
//
// Every wave owns 32 coordinates and carries them through all layers without their
// activations ever leaving registers; device-memory traffic is the coordinates in and the
// signal values out.  The only shared state is the current layer's weights in LDS.
//
// Data layout.  The GEMM runs "features x coordinates": the int8 weights are the A operand
// of v_mfma_i32_32x32x32_i8 (32 output features x 32 k), the activation codes the B operand
// (32 k x 32 coordinates).  With that orientation lane l of a wave holds, for coordinate
// l % 32, accumulator rows 8g + 4h + e (g = 0..3, h = l / 32, e = 0..3) of every 32-row
// tile T: half of the feature vector of one coordinate, in registers R = 16T + 4g + e.
// The Walsh-Hadamard transform over the feature index (Eq. 3) factors as H_NF = H_NT (x) H_32
// and is done in two parts:
//   - H_32 over the 32 rows of each tile on the matrix unit (see fused_gemm_sine_hm below):
//     the tile's activations are already laid out as an MFMA B operand, H_32 is the A operand;
//   - log2(NT) butterfly stages over the tile index, i.e. over bits 4.. of R: plain register
//     add/sub, no lane traffic.
// After the last stage register s of lane half u holds rotated feature j(s, u) (hm_index in
// dhq_fused_common.h); quantizing register s into byte s % 4 of dword s / 4 makes four consecutive dwords
// exactly the B operand of k block s / 16.  The contraction index of an MFMA can be enumerated
// in any order as long as both operands agree, so the weights are packed offline with their k
// positions permuted by j(s, u) and nothing is ever shuffled at run time.
//
// The first layer (fan-in <= 4) and the output layer (fan-out <= 32) use the same
// machinery with the k block / the M tile zero-padded.
//
// Weights: each layer's A fragments ([tile][k block][lane] x 16 B) followed by its biases
// form one contiguous block; while layer l computes, the block of layer l+1 is copied from
// device memory (L2-resident) straight into the other LDS buffer with 16-byte
// global->LDS loads, so the copy costs no registers and no VALU work.
//
// Two-sided rotation (Eq. 4 with both factors): the layer's output in the rotated basis is multiplied by H once more, exactly, in
// int32.  That product is linear in the weights, z = (q W'^T) H = q (H W')^T, so these kernels multiply by U = H W' and have no
// un-rotation.  An entry of U is a sum of up to 256 codes of 127, at most 32 512 = two int8 digits, 256 u1 + u0
// (DHQ_TWO_DIGITS): twice the int8 MFMAs and a shift against eight integer butterfly stages and a lane exchange per value.  Five
// layers, 262 144 rows, butterflies / digits in us: width 32 25.9 / 22.0, 64 (wavelet) 55.9 / 48.6, 128 90.3 / 75.8, 256 197.7 /
// 194.2 (there the digits' products load the matrix unit as much as the epilogue does the vector ALU); 1 000 rows of 256,
// which the kernel for few rows now takes as well, 49.9 / 13.3.
// Row r of a tile is the feature whose index in the tile is r with bits 0 and 2 exchanged, which is where the lane exchange of the
// butterflies left it: the products with H_32 then add a tile's activations in the same order as behind them, and the values are
// theirs bit for bit.
#include <math.h>
#include <string.h>

#include <vector>

#include "dhq_device.h"
#include "dhq_fused_common.h"
#include "dhq_internal.h"

#define FUSED_WAVES 8            // waves per workgroup, two per SIMD
#define FUSED_THREADS (FUSED_WAVES * 64)
#define FUSED_TILE (FUSED_WAVES * 32)  // coordinates per workgroup pass

struct fused_layer_desc {
    uint32_t blob_off;   // byte offset of the layer's block in the packed weight blob
    uint32_t chunks;     // block size in KiB (1 KiB = what one wave copies per instruction)
    float c1;            // sine layers: s_a s_w omega0 / (2 pi); output layer: s_a s_w
    float inv_in;        // 1 / (s_a sqrt(Kp)) of this layer's input quantizer (divided by `scale` behind split activations)
};

struct fused_args {
    const float *coords;
    float *out;
    const unsigned char *blob;
    int64_t n;
    int n_layers;
    int k0, k0p;   // fan-in of the first layer and its power-of-two padding (<= 4)
    int m_out;     // fan-out of the output layer (<= 32)
    int qmax;
    float c2;      // wavelet activation: 2 pi s0 sqrt(log2 e) / omega0
    fused_layer_desc layer[DHQ_MAX_LAYERS];
    float scale;   // padded networks: what the activations are multiplied by before they are split (last: with the layers four
                   // bytes on in the argument block a one-pass forward took 1 % longer, 28.6 against 28.35 us)
    int kb0;       // k blocks of the input layer
    const int8_t *codes0;  // its codes, where the fan-in is above 4 (DHQ_CODES_IN)
};

struct dhq_fused_plan {
    int nf = 0;                      // hidden width
    int act_kind = DHQ_ACT_KIND_SINE;
    bool padded = false;             // the network's own hidden widths are smaller, padded to nf
    int digits = 1;                  // int8 digits of a weight: two in two-sided models
    int skip = 0;                    // tiles of 32 features that are all padding
    unsigned char *blob_dev = nullptr;
    size_t blob_bytes = 0;
    fused_args args;
    size_t lds_bytes = 0;
    int n_cu = 0;
    int device = 0;
};

// ---- the in-tile part of the transform on the matrix unit ------------------------------------
// The 32 features of an M tile are one factor of the Sylvester matrix, H_NF = H_NT (x) H_32, so
// the five butterfly stages over the within-tile index (four over register bits, one over the
// lane half) are the product H_32 * (tile of activations): a 32 x 32 x 32 contraction whose B
// operand the lanes already hold.  The matrix unit has no fp32 input at a useful rate, so an
// activation a (|a| <= 1) is split into two binary16 pieces, hi = a rounded toward zero and
// lo = (a - hi) rounded toward zero (a - hi is exact in fp32), which carry a to within 2^-21 |a|
// (2^-24 absolute below 2^-10, where lo is subnormal; v_mfma_f32_32x32x16_f16 takes subnormal
// inputs as they are).  That is up to four units in the last place of a, still below the error
// of the sine that produced a, and the rotated activations come out with about the same error
// as from fp32 butterflies (1.3e-6 against 0.9e-6 rms at width 256, un-normalised).  The
// products with +-1 are exact and the sum is accumulated in fp32 like
// the butterflies' sums.  Per tile: 8 + 8 packed conversions, 16 mixed-precision subtractions
// and 4 MFMAs replace 80 add/sub and 8 lane swaps.  The three stages over the tile index stay
// on the vector ALU.  Afterwards register s of lane half u holds rotated feature hm_index(s, u).
// KB: MFMAs of a tile; DS: steps its drain is spread over.
template <int NT, int KB, int DS>
struct hm_sched {
    static constexpr bool STAGGER = (NT >= 2 && KB >= 2);
    static constexpr int STEPS = (STAGGER ? ((NT + 1) / 2) * 2 * KB + KB + 1 : NT * KB) + DS + 6;
    static constexpr int NM = NT * KB;
    int tile[STEPS], kb[STEPS], seq[STEPS];   // GEMM MFMA issued at this step (tile -1: none)
    int drain[STEPS], drain_pos[STEPS];       // tile drained at this step and which slice of it
    int hm_n[STEPS], hm_tile[STEPS][4], hm_k[STEPS][4];  // transform MFMAs issued at this step
    int seq_tile[NM], seq_kb[NM];
    int last;                                 // last step with any work
    constexpr hm_sched()
        : tile(), kb(), seq(), drain(), drain_pos(), hm_n(), hm_tile(), hm_k(), seq_tile(), seq_kb(), last(0)
    {
        int done[NT > 0 ? NT : 1] = {};
        for (int g = 0; g < STEPS; ++g) { tile[g] = -1; kb[g] = 0; seq[g] = -1; drain[g] = -1; drain_pos[g] = 0; hm_n[g] = 0; }
        for (int t = 0; t < NT; ++t) {
            const int i = t / 2;
            const int base = (t & 1) ? 2 * KB * i + KB + 1 : 2 * KB * i;
            for (int k = 0; k < KB; ++k) {
                const int g = STAGGER ? base + 2 * k : t * KB + k;
                tile[g] = t; kb[g] = k; done[t] = g;
            }
        }
        int m = 0;
        for (int g = 0; g < STEPS; ++g)
            if (tile[g] >= 0) { seq[g] = m; seq_tile[m] = tile[g]; seq_kb[m] = kb[g]; ++m; }
        for (int t = 0; t < NT; ++t) {
            int at[DS + 3] = {};
            int g = done[t] + 1;
            for (int k = 0; k < DS; ++k) {
                while (drain[g] >= 0) ++g;
                drain[g] = t; drain_pos[g] = k; at[k] = g;
                ++g;
            }
            at[DS] = at[DS - 1] + 1; at[DS + 1] = at[DS - 1] + 2;
            // pieces of block 0 (accumulators 0..7) are complete after slice DS/2 - 1, of block 1 after the last
            int when[4] = {at[DS], at[DS], at[DS], at[DS]};
            if (DS >= 4) { when[0] = at[DS / 2]; when[1] = at[DS / 2 + 1]; when[2] = at[DS]; when[3] = at[DS + 1]; }
            for (int k = 0; k < 4; ++k) {
                const int w = when[k];
                hm_tile[w][hm_n[w]] = t; hm_k[w][hm_n[w]] = k; ++hm_n[w];
                if (w > last) last = w;
            }
        }
    }
};

// One layer's GEMM with the dequantize + bias + sine epilogue, the split into binary16 pieces and
// the H_32 products, software-pipelined by hand according to hm_sched.  On return xt[T][v]
// holds, for this lane's coordinate, row 8 (v / 4) + 4 h + v % 4 of H_32 * (activations of tile T).
// ACTK: the activation (sine, or the wavelet with envelope constant c2), plus DHQ_SPLIT_RN where the activations are scaled
// before they are split and hi rounds to nearest (xt then comes out times `scale`).  With DHQ_PLAIN xt[T][v] is the activation
// itself, any finite argument.  With DHQ_TWO_DIGITS a tile takes the products with the upper digits, shifts its sums by eight
// bits and takes the products with the lower ones into the same accumulators (wrapping, the exact int32).
template <int NT, int KB, int NCD, int ACTK = DHQ_ACT_KIND_SINE>
__device__ __forceinline__ void fused_gemm_sine_hm(const dhq_v4i *__restrict__ wA, const float4 *__restrict__ wB,
                                                   const dhq_v4i (&cd)[NCD], float c1, dhq_v16f (&xt)[NT],
                                                   const dhq_v4i (&hA)[2], int lane, int h, float c2 = 0.f, float scale = 1.f)
{
    constexpr int RT = NT - DHQ_SKIP(ACTK);  // tiles that are not all padding
    constexpr int KM = KB * DHQ_DIGITS(ACTK);  // MFMAs of a tile
    constexpr hm_sched<RT, KM, KB> S{};
    // the multiplier in a vector register: a multiply-add whose operands are all vector registers issues in about
    // 3 clocks per wave, one with a scalar operand in about 4.5 (measured with a register-only loop)
    asm volatile("" : "+v"(c1));
    if constexpr ((ACTK & DHQ_SPLIT_RN) != 0) asm volatile("" : "+v"(scale));
    constexpr int LAST = S.last;
    constexpr int NM = RT * KM;
    constexpr int EPS = 16 / KB;  // accumulators drained per step (KB <= 8: an even number)
    constexpr int PF = (NM >= 4) ? 4 : (NM >= 2 ? 2 : 1);  // LDS prefetch distance in MFMAs
    dhq_v4i fr[PF + 1];
    float4 bq[3][4];
    dhq_v16i acc[3];
    unsigned hp[2][8], lp[2][8];  // packed pieces of the tile being drained (and of the one before)
#pragma unroll
    for (int m = 0; m < PF; ++m)
        if (m < NM) fr[m % (PF + 1)] = wA[(S.seq_tile[m] * KM + S.seq_kb[m]) * 64 + lane];
    constexpr int GB = 8;
#pragma unroll
    for (int g0 = 0; g0 <= LAST; g0 += GB) {
#pragma unroll
      for (int g1 = 0; g1 < GB; ++g1) {
        const int g = g0 + g1;
        if (g > LAST) continue;
        const int T = S.tile[g];
        if (T >= 0) {
            const int m = S.seq[g], kb = S.kb[g];
            if (m + PF < NM) {
                fr[(m + PF) % (PF + 1)] = wA[(S.seq_tile[m + PF] * KM + S.seq_kb[m + PF]) * 64 + lane];
                __builtin_amdgcn_sched_barrier(0);  // keep the prefetch at the top of the step
            }
#pragma unroll
            for (int gg = 0; gg < 4; ++gg)
                if ((gg * KM) / 4 == kb) bq[T % 3][gg] = wB[(T * 4 + gg) * 2 + h];
            if (kb == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[T % 3][v] = 0;
            }
            if (KM > KB && kb == KB) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[T % 3][v] = (int)((unsigned)acc[T % 3][v] << 8);
            }
            acc[T % 3] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[m % (PF + 1)], cd[kb % KB], acc[T % 3], 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((ACTK & DHQ_PLAIN) == 0 && q < S.hm_n[g]) {
                const int Th = S.hm_tile[g][q], k = S.hm_k[g][q];
                const int blk = k >> 1;
                dhq_v4i b;  // small pieces first
#pragma unroll
                for (int d = 0; d < 4; ++d) b[d] = (int)((k & 1) ? hp[Th & 1][4 * blk + d] : lp[Th & 1][4 * blk + d]);
                dhq_v16f d;
                if (k == 0) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) d[v] = 0.f;
                } else {
                    d = xt[Th];
                }
                xt[Th] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(dhq_v8h, hA[blk]),
                                                                __builtin_bit_cast(dhq_v8h, b), d, 0, 0, 0);
            }
        }
        const int Td = S.drain[g];
        if (Td >= 0) {
#pragma unroll
            for (int j = 0; j < EPS; j += 2) {
                const int v = S.drain_pos[g] * EPS + j;
                const float4 bb = bq[Td % 3][v >> 2];
                const float bias0 = (v & 2) ? bb.z : bb.x, bias1 = (v & 2) ? bb.w : bb.y;
                // accumulators v, v + 1 (v even) are neighbouring features 2m, 2m + 1: the pair the complex wavelet takes
                const float t0 = __builtin_fmaf((float)acc[Td % 3][v], c1, bias0), t1 = __builtin_fmaf((float)acc[Td % 3][v + 1], c1, bias1);
                float a0, a1;
                if constexpr ((ACTK & DHQ_PLAIN) != 0) {
                    if constexpr (DHQ_KIND(ACTK) == DHQ_ACT_KIND_WAVELET_COMPLEX) {
                        dhq_activate_pair_rev<true>(t0, t1, c2, a0, a1);
                    } else {
                        a0 = dhq_activate_rev_any(t0, dhq_act{DHQ_KIND(ACTK), c2});
                        a1 = dhq_activate_rev_any(t1, dhq_act{DHQ_KIND(ACTK), c2});
                    }
                    asm volatile("" : "+v"(a0), "+v"(a1));  // (a wavelet's product is rounded before anything is added to it)
                    xt[Td][v] = a0;
                    xt[Td][v + 1] = a1;
                    continue;
                }
                if constexpr (DHQ_KIND(ACTK) == DHQ_ACT_KIND_WAVELET_COMPLEX) {
                    dhq_activate_pair_rev<false>(t0, t1, c2, a0, a1, hm_scaled<ACTK>(1.f, scale));
                } else {
                    a0 = hm_scaled<ACTK>(dhq_activate_rev(t0, dhq_act{DHQ_KIND(ACTK), c2}), scale);
                    a1 = hm_scaled<ACTK>(dhq_activate_rev(t1, dhq_act{DHQ_KIND(ACTK), c2}), scale);
                }
                hm_split_pair<ACTK>(a0, a1, hp[Td & 1][v >> 1], lp[Td & 1][v >> 1]);
            }
        }
        if (T >= 0 || Td >= 0 || S.hm_n[g] > 0) __builtin_amdgcn_sched_barrier(0);
      }
    }
}

// The stages of the transform over the tile index: plain register add/sub.  The last SKIP tiles are zero (and not written yet);
// before stage s a tile still is if all tiles that differ from it in lower bits only are.
template <int NT, int SKIP = 0>
__device__ __forceinline__ void fused_tile_stages(dhq_v16f (&xt)[NT])
{
#pragma unroll
    for (int s = 1; s < NT; s <<= 1) {
#pragma unroll
        for (int T = 0; T < NT; ++T) {
            if ((T & s) == 0 && (T & -s) < NT - SKIP) {
                if (((T | s) & -s) >= NT - SKIP) {
                    xt[T | s] = xt[T];
                    continue;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float a = xt[T][v], b = xt[T | s][v];
                    xt[T][v] = a + b;
                    xt[T | s][v] = a - b;
                }
            }
        }
    }
}

// The whole transform in fp32, with the additions of the layer-by-layer kernels in their order (wht_butterflies: index bits
// 0, 1, then 6, 7 where there are any, then 2, 3, 4, 5), so the same bits.  Index bits 0, 1, 3, 4 are bits of v, 2 is the lane
// half, 5 .. the tile.  The stage over the lane half works on pairs of registers: v_permlane32_swap brings both operands
// of one register's stage into one lane half, those of the other's into the other.  With four tiles or more the pairs are tiles
// T, T | 2, which no later stage combines; lane half and that bit stay swapped until fused_plain_codes has four values in a
// dword.  Below, v and v + 1 are swapped back at once.
// The last SKIP tiles are zero, as in fused_tile_stages (`done`: the tile-index bits whose stages are behind).
template <int NT, int SKIP = 0>
__device__ __forceinline__ void fused_butterflies(dhq_v16f (&x)[NT])
{
    auto zero = [](int T, int done) { return (T & ~done) >= NT - SKIP; };
    auto over_v = [&](int b, int done) {
#pragma unroll
        for (int T = 0; T < NT; ++T) {
            if (zero(T, done)) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if ((v & b) == 0) {
                    const float p = x[T][v], q = x[T][v | b];
                    x[T][v] = p + q;
                    x[T][v | b] = p - q;
                }
        }
    };
    auto over_tiles = [&](int b, int done) {
#pragma unroll
        for (int T = 0; T < NT; ++T)
            if ((T & b) == 0 && !zero(T, done)) {
                if (zero(T | b, done)) {
                    x[T | b] = x[T];
                    continue;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float p = x[T][v], q = x[T | b][v];
                    x[T][v] = p + q;
                    x[T | b][v] = p - q;
                }
            }
    };
    constexpr int high = NT > 4 ? 6 : NT > 2 ? 2 : 0;  // the tile-index bits that come before the lane half
    over_v(1, 0);
    over_v(2, 0);
    if constexpr (NT > 2) over_tiles(2, 0);
    if constexpr (NT > 4) over_tiles(4, 2);
#pragma unroll
    for (int T = 0; T < NT; ++T) {
        if ((NT > 2 && (T & 2) != 0) || zero(T, high)) continue;
#pragma unroll
        for (int v = 0; v < 16; v += NT > 2 ? 1 : 2) {
            const int T2 = NT > 2 ? (T | 2) % NT : T, v2 = NT > 2 ? v : (v + 1) % 16;
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[T][v]), __float_as_uint(x[T2][v2]), false, false);
            const float s = __uint_as_float(r[0]) + __uint_as_float(r[1]), d = __uint_as_float(r[0]) - __uint_as_float(r[1]);
            if constexpr (NT > 2) {
                x[T][v] = s;
                x[T2][v2] = d;
            } else {
                const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(d), false, false);
                x[T][v] = __uint_as_float(o[0]);
                x[T2][v2] = __uint_as_float(o[1]);
            }
        }
    }
    over_v(4, high);
    over_v(8, high);
    if constexpr (NT > 1) over_tiles(1, high);
}
// The codes of what fused_butterflies leaves (quantized by fused_quantize), in their places.
template <int NT>
__device__ __forceinline__ void fused_plain_codes(dhq_v4i (&cd)[NT])
{
    if constexpr (NT > 2) {
#pragma unroll
        for (int T = 0; T < NT; ++T)
            if ((T & 2) == 0) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)cd[T][g], (unsigned)cd[T | 2][g], false, false);
                    cd[T][g] = (int)r[0];
                    cd[T | 2][g] = (int)r[1];
                }
            }
    }
}

// The quantizer: register s = 16 T + v becomes byte s % 4 of dword s / 4 of the codes.
template <int NT>
__device__ __forceinline__ void fused_quantize(const dhq_v16f (&xt)[NT], dhq_v4i (&cd)[NT], float inv, int qlo, int qhi)
{
    asm volatile("" : "+v"(inv));  // a vector-register multiplier, as in fused_gemm_sine_hm
#pragma unroll
    for (int w = 0; w < NT * 4; ++w) {
        const int v = 4 * (w & 3);
        cd[w / 4][w % 4] = (int)fused_quant4(xt[w >> 2][v], xt[w >> 2][v + 1], xt[w >> 2][v + 2], xt[w >> 2][v + 3], inv, qlo, qhi);
    }
}

// The output layer: one zero-padded M tile, no sine.
template <int NKB, int DIGITS = 1>
__device__ __forceinline__ void fused_output_layer(const dhq_v4i *__restrict__ wA, const float *__restrict__ wB,
                                                   const dhq_v4i (&cd)[NKB], float c1, float *__restrict__ out, int64_t ci,
                                                   bool valid, int m_out, int lane, int h)
{
    dhq_v16i acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
    for (int kb = 0; kb < NKB * DIGITS; ++kb) {
        if (DIGITS > 1 && kb == NKB) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = (int)((unsigned)acc[v] << 8);
        }
        const dhq_v4i a = wA[kb * 64 + lane];
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, cd[kb % NKB], acc, 0, 0, 0);
    }
    if (valid) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = 8 * (v >> 2) + 4 * h + (v & 3);
            if (row < m_out) out[ci * m_out + row] = __builtin_fmaf((float)acc[v], c1, wB[((v >> 2) * 2 + h) * 4 + (v & 3)]);
        }
    }
}

// A hidden layer's block: fragments [tile][digit][k block] KiB, then one KiB of biases.  Two digits at width 256 are 128 KiB of
// fragments, which the two buffers of the whole-network kernel take as two blocks of half the tiles each.
template <int NT, int KB, int ACTK>
constexpr int fused_halves = NT * KB * DHQ_DIGITS(ACTK) > 64 ? 2 : 1;
template <int NT, int KB, int ACTK>
constexpr int fused_block_kib = NT * KB * DHQ_DIGITS(ACTK) / fused_halves<NT, KB, ACTK> + 1;
// The GEMM of one of them (HALF), and of a whole layer in LDS.
template <int NT, int KB, int NCD, int ACTK, int HALF>
__device__ __forceinline__ void fused_half(const unsigned char *blk, const dhq_v4i (&cd)[NCD], float c1, dhq_v16f (&xt)[NT],
                                           const dhq_v4i (&hA)[2], int lane, int h, float c2, float scale)
{
    constexpr int TH = NT / fused_halves<NT, KB, ACTK>;
    fused_gemm_sine_hm<TH, KB, NCD, ACTK>(reinterpret_cast<const dhq_v4i *>(blk),
                                          reinterpret_cast<const float4 *>(blk + (fused_block_kib<NT, KB, ACTK> - 1) * 1024), cd, c1,
                                          reinterpret_cast<dhq_v16f(&)[TH]>(xt[HALF * TH]), hA, lane, h, c2, scale);
}
template <int NT, int KB, int NCD, int ACTK>
__device__ __forceinline__ void fused_layer_gemm(const unsigned char *blk, const dhq_v4i (&cd)[NCD], float c1, dhq_v16f (&xt)[NT],
                                                 const dhq_v4i (&hA)[2], int lane, int h, float c2, float scale = 1.f)
{
    fused_half<NT, KB, NCD, ACTK, 0>(blk, cd, c1, xt, hA, lane, h, c2, scale);
    if constexpr (fused_halves<NT, KB, ACTK> > 1)
        fused_half<NT, KB, NCD, ACTK, 1>(blk + fused_block_kib<NT, KB, ACTK> * 1024, cd, c1, xt, hA, lane, h, c2, scale);
}

// ROWS: which rows a wave takes, and whether it has to look.
//   FUSED_DEALT  32-row tiles go to wave 0 of every workgroup, then to wave 1 and so on, so that a last pass with too few of
//     them for all waves leaves the higher waves of every workgroup without one (they only help to copy the weights in)
//     rather than some workgroups: waves w and w + 4 share a SIMD, and one that has it alone needs about two thirds of the time.
//   FUSED_WHOLE  the same where every wave has a tile in every pass; the test for it costs 0.5 % of a forward.
//   FUSED_IN_A_ROW  a workgroup takes FUSED_TILE rows in a row, and waves beyond the end repeat the last one: for a last pass
//     that more than half of the waves have a tile in, where dealing gains nothing and CUs without work leave the others a
//     higher clock (100 003 rows, 3 layers of 64 and of 256 features: 12.0 and 38.9 us, dealt 12.2 and 39.8).
enum { FUSED_DEALT, FUSED_WHOLE, FUSED_IN_A_ROW };
template <int NF, int ACTK, int ROWS>
__global__ __launch_bounds__(FUSED_THREADS) void dhq_fused_kernel(const fused_args A)
{
    constexpr int NT = NF / 32;   // M tiles of a hidden layer
    constexpr int NKB = NF / 32;  // k blocks of a hidden layer
    constexpr int BLK = fused_block_kib<NT, NKB, ACTK> * 1024;  // LDS bytes per weight buffer
    constexpr bool HALVES = fused_halves<NT, NKB, ACTK> > 1;
    constexpr int INPUT_KB = (ACTK & DHQ_CODES_IN) != 0 && NKB > 1 ? 2 : 1;  // most k blocks of the input layer

    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int L = A.n_layers;
    constexpr bool IN_A_ROW = (ROWS == FUSED_IN_A_ROW);
    const int64_t n_tiles = IN_A_ROW ? (A.n + FUSED_TILE - 1) / FUSED_TILE : (A.n + 31) / 32;
    const int64_t stride = IN_A_ROW ? gridDim.x : (int64_t)gridDim.x * FUSED_WAVES;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;

    dhq_v4i hA[2];
    fused_h32_operand<(ACTK & DHQ_TWO_DIGITS) != 0>(c, h, hA);

    int p = 0;  // LDS buffer holding the layer about to run
    if ((int64_t)blockIdx.x < n_tiles)
        fused_issue_copy(A.blob + A.layer[0].blob_off, lds, (int)A.layer[0].chunks, wave, lane, FUSED_WAVES);

    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += stride) {
        const int64_t wave_tile = tile + (int64_t)__builtin_amdgcn_readfirstlane(wave) * gridDim.x;  // (dealt)
        const bool active = ROWS != FUSED_DEALT || wave_tile < n_tiles;
        const int64_t ci = IN_A_ROW ? tile * FUSED_TILE + wave * 32 + c : wave_tile * 32 + c;
        const bool valid = ci < A.n;
        const int64_t cl = valid ? ci : A.n - 1;

        dhq_v4i cd[NKB];  // activation codes: the B operands of the next GEMM
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
        if constexpr ((ACTK & DHQ_CODES_IN) != 0) fused_load_codes(A.codes0, cl, A.k0p, h, cd);
        else cd[0][0] = fused_input_codes(A.coords, cl, A.k0, A.k0p, A.layer[0].inv_in, A.qmax);

        dhq_v16f xt[NT];
        for (int l = 0; l < L - 1; ++l) {
            // weights of layer l have landed; everyone is done with the other buffer
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            const fused_layer_desc &nx = A.layer[l + 1];
            const unsigned char *const next = A.blob + nx.blob_off;
            const int next_kib = HALVES && l + 1 < L - 1 ? BLK / 1024 : (int)nx.chunks;
            const float c1 = A.layer[l].c1;
            if (HALVES && l > 0) {
                fused_issue_copy(A.blob + A.layer[l].blob_off + BLK, lds + (p ^ 1) * BLK, BLK / 1024, wave, lane, FUSED_WAVES);
                if (active) fused_half<NT, NKB, NKB, ACTK, 0>(lds + p * BLK, cd, c1, xt, hA, lane, h, A.c2, A.scale);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                fused_issue_copy(next, lds + p * BLK, next_kib, wave, lane, FUSED_WAVES);
                if (active) fused_half<NT, NKB, NKB, ACTK, HALVES ? 1 : 0>(lds + (p ^ 1) * BLK, cd, c1, xt, hA, lane, h, A.c2, A.scale);
                p ^= 1;
            } else {
                fused_issue_copy(next, lds + (p ^ 1) * BLK, next_kib, wave, lane, FUSED_WAVES);
                if (!active) {
                } else if (INPUT_KB > 1 && l == 0 && A.kb0 == 2)
                    fused_layer_gemm<NT, INPUT_KB, NKB, ACTK>(lds + p * BLK, cd, c1, xt, hA, lane, h, A.c2, A.scale);
                else if (l == 0)
                    fused_layer_gemm<NT, 1, NKB, ACTK>(lds + p * BLK, cd, c1, xt, hA, lane, h, A.c2, A.scale);
                else if constexpr (!HALVES)
                    fused_layer_gemm<NT, NKB, NKB, ACTK>(lds + p * BLK, cd, c1, xt, hA, lane, h, A.c2, A.scale);
            }
            // The two waves of a SIMD overlap well while both feed the matrix unit or both
            // do vector work, but a wave in its vector phase starves the MFMA chain of the
            // other; keep the phases aligned across the workgroup.
            __syncthreads();
            if (active) {
                if constexpr ((ACTK & DHQ_PLAIN) != 0) fused_butterflies<NT, DHQ_SKIP(ACTK)>(xt);
                else fused_tile_stages<NT, DHQ_SKIP(ACTK)>(xt);
                fused_quantize<NT>(xt, cd, A.layer[l + 1].inv_in, qlo, qhi);
                if constexpr ((ACTK & DHQ_PLAIN) != 0) fused_plain_codes<NT>(cd);
            }
            p ^= 1;
        }

        // output layer: one zero-padded M tile, no sine
        {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tile + stride < n_tiles)
                fused_issue_copy(A.blob + A.layer[0].blob_off, lds + (p ^ 1) * BLK, (int)A.layer[0].chunks, wave, lane, FUSED_WAVES);
            if (active)
                fused_output_layer<NKB, DHQ_DIGITS(ACTK)>(reinterpret_cast<const dhq_v4i *>(lds + p * BLK),
                                        reinterpret_cast<const float *>(lds + p * BLK + NKB * DHQ_DIGITS(ACTK) * 1024), cd, A.layer[L - 1].c1, A.out, ci,
                                        valid, A.m_out, lane, h);
            p ^= 1;
        }
    }
}

// ---- few rows: the features of 32 coordinates split over the waves of a workgroup --------------
// In the kernel above a wave carries 32 coordinates alone, and a pass takes the time of two waves per SIMD going through
// every feature (5.5 us per 256-wide layer) however few rows there are.  Here a workgroup of NT waves carries 32 coordinates
// and each wave one M tile: its GEMM, epilogue and H_32 products.  For the stages over the tile index the work is
// re-split by rows through LDS (wave w takes rows 16 w / NT .. of every tile), and the codes are joined in LDS, from where
// every wave reads the whole B operand, as the two waves of a pair do at width 512.  The weights are not staged: a fragment is
// read by one wave only, straight from device memory, while the layer before is in its epilogue.  Same operations in the
// same order per value, hence the same bits as the kernel above; what a layer takes is latency: a forward of
// five 256-wide layers on 1 000 rows 31.7 -> 11.0 us.  (Two accumulator chains of every other k block: unchanged.)
template <int NF, int ACTK>
__global__ __launch_bounds__(NF * 2, DHQ_DIGITS(ACTK) > 1 ? 2 : 4) void dhq_fused_split_kernel(const fused_args A)
{
    constexpr int NT = NF / 32, NKB = NF / 32, RPW = 16 / NT, D = DHQ_DIGITS(ACTK);
    constexpr int BLK = fused_block_kib<NT, NKB, ACTK> * 1024, TH = NT / fused_halves<NT, NKB, ACTK>;  // a hidden layer's blocks
    __shared__ float4 xs[NT * 4 * 64];    // [tile][row group g][lane]: rows 4 g .. 4 g + 3 of the lane's coordinate
    __shared__ dhq_v4i codes[NKB * 64];   // [k block][lane]: the next layer's B operand
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 31, h = lane >> 5;
    const int L = A.n_layers;
    const int n_tiles = (int)((A.n + 31) / 32);  // fewer than a full pass of the kernel above has
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;
    dhq_v4i hA[2];
    fused_h32_operand<(ACTK & DHQ_TWO_DIGITS) != 0>(c, h, hA);
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t ci = (int64_t)tile * 32 + c;
        const bool valid = ci < A.n;
        const int64_t cl = valid ? ci : A.n - 1;
        dhq_v4i fr[D * NKB];  // [digit][k block]
        float4 bias[4];
        {
            const unsigned char *blk = A.blob + A.layer[0].blob_off;
#pragma unroll
            for (int d = 0; d < D; ++d) fr[d] = reinterpret_cast<const dhq_v4i *>(blk)[(wave * D + d) * 64 + lane];
#pragma unroll
            for (int g = 0; g < 4; ++g) bias[g] = reinterpret_cast<const float4 *>(blk + NT * D * 1024)[(wave * 4 + g) * 2 + h];
        }
        dhq_v16i acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0;
        {
            const dhq_v4i cd = {fused_input_codes(A.coords, cl, A.k0, A.k0p, A.layer[0].inv_in, A.qmax), 0, 0, 0};
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[0], cd, acc, 0, 0, 0);
            if constexpr (D > 1) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = (int)((unsigned)acc[v] << 8);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[1], cd, acc, 0, 0, 0);
            }
        }
        for (int l = 0; l < L - 1; ++l) {
            const float c1 = A.layer[l].c1;
            float4 b[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) b[g] = bias[g];
            // the next layer's fragments and biases, in time for its GEMM (the output layer: one tile, wave 0's)
            {
                const unsigned char *blk = A.blob + A.layer[l + 1].blob_off + wave / TH * BLK;
                const bool last = (l + 1 == L - 1);
                if (!last || wave == 0) {
                    const int t = wave % TH;  // (wave 0: 0)
#pragma unroll
                    for (int kb = 0; kb < D * NKB; ++kb) fr[kb] = reinterpret_cast<const dhq_v4i *>(blk)[(t * D * NKB + kb) * 64 + lane];
                    const float4 *wB = reinterpret_cast<const float4 *>(blk + (last ? 1 : TH) * D * NKB * 1024);
#pragma unroll
                    for (int g = 0; g < 4; ++g) bias[g] = wB[(t * 4 + g) * 2 + h];
                }
            }
            unsigned hp[8], lp[8];
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                const float4 bb = b[v >> 2];
                const float bias0 = (v & 2) ? bb.z : bb.x, bias1 = (v & 2) ? bb.w : bb.y;
                const float t0 = __builtin_fmaf((float)acc[v], c1, bias0), t1 = __builtin_fmaf((float)acc[v + 1], c1, bias1);
                float a0, a1;
                if constexpr (DHQ_KIND(ACTK) == DHQ_ACT_KIND_WAVELET_COMPLEX) {
                    dhq_activate_pair_rev<false>(t0, t1, A.c2, a0, a1, hm_scaled<ACTK>(1.f, A.scale));
                } else {
                    a0 = hm_scaled<ACTK>(dhq_activate_rev(t0, dhq_act{DHQ_KIND(ACTK), A.c2}), A.scale);
                    a1 = hm_scaled<ACTK>(dhq_activate_rev(t1, dhq_act{DHQ_KIND(ACTK), A.c2}), A.scale);
                }
                hm_split_pair<ACTK>(a0, a1, hp[v >> 1], lp[v >> 1]);
            }
            dhq_v16f x;
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                dhq_v4i p;  // small pieces first
#pragma unroll
                for (int d = 0; d < 4; ++d) p[d] = (int)((k & 1) ? hp[4 * (k >> 1) + d] : lp[4 * (k >> 1) + d]);
                x = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(dhq_v8h, hA[k >> 1]), __builtin_bit_cast(dhq_v8h, p), x, 0, 0, 0);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) xs[(wave * 4 + g) * 64 + lane] = make_float4(x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]);
            __syncthreads();
            float z[NT][RPW];
#pragma unroll
            for (int T = 0; T < NT; ++T) {
                if constexpr (RPW == 2) {
                    const float2 p = reinterpret_cast<const float2 *>(xs)[((T * 4 + (wave >> 1)) * 64 + lane) * 2 + (wave & 1)];
                    z[T][0] = p.x; z[T][1] = p.y;
                } else {
#pragma unroll
                    for (int i = 0; i < RPW; i += 4) {
                        const float4 p = xs[(T * 4 + wave * (RPW / 4) + i / 4) * 64 + lane];
                        z[T][i] = p.x; z[T][i + 1] = p.y; z[T][i + 2] = p.z; z[T][i + 3] = p.w;
                    }
                }
            }
#pragma unroll
            for (int s = 1; s < NT; s <<= 1) {
#pragma unroll
                for (int T = 0; T < NT; ++T) {
                    if ((T & s) == 0) {
#pragma unroll
                        for (int i = 0; i < RPW; ++i) {
                            const float p = z[T][i], q = z[T | s][i];
                            z[T][i] = p + q;
                            z[T | s][i] = p - q;
                        }
                    }
                }
            }
            const float inv = A.layer[l + 1].inv_in;
#pragma unroll
            for (int T = 0; T < NT; ++T) {
                if constexpr (RPW == 2) {
                    if ((T & 1) == 0) {
                        const unsigned w = fused_quant4(z[T][0], z[T][1], z[T + 1][0], z[T + 1][1], inv, qlo, qhi);
                        unsigned short *d = reinterpret_cast<unsigned short *>(codes) + lane * 8 + wave;
                        d[T * 512] = (unsigned short)w;
                        d[(T + 1) * 512] = (unsigned short)(w >> 16);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < RPW; i += 4)
                        reinterpret_cast<unsigned *>(codes)[(T * 64 + lane) * 4 + wave * (RPW / 4) + i / 4] =
                            fused_quant4(z[T][i], z[T][i + 1], z[T][i + 2], z[T][i + 3], inv, qlo, qhi);
                }
            }
            __syncthreads();
            if (l + 1 < L - 1 || wave == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
                for (int kb = 0; kb < D * NKB; ++kb) {
                    if (D > 1 && kb == NKB) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[v] = (int)((unsigned)acc[v] << 8);
                    }
                    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[kb], codes[kb % NKB * 64 + lane], acc, 0, 0, 0);
                }
            }
        }
        if (wave == 0 && valid) {
            const float c1 = A.layer[L - 1].c1;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                const float4 bb = bias[v >> 2];
                const float bv = (v & 3) == 0 ? bb.x : (v & 3) == 1 ? bb.y : (v & 3) == 2 ? bb.z : bb.w;
                if (row < A.m_out) A.out[ci * A.m_out + row] = __builtin_fmaf((float)acc[v], c1, bv);
            }
        }
    }
}

// ---- one launch per layer: the dynamic quantization module (Sec. 3.3) ------------------------
// With scales measured on line, a layer's quantizer needs max |x^| over the whole batch before
// it can emit a single code, so the network cannot stay in registers from end to end.  These
// kernels cut the fused kernel at exactly that point: the launch of layer l folds the maxima the previous launch's
// workgroups left into this layer's constants (every workgroup for itself: a few hundred floats and three fp64
// operations cost less than a launch in between), quantizes its input x^ with them, runs the layer (GEMM, epilogue,
// transform) and leaves each workgroup's max |x^| of the result.  How x^ gets from one launch to the next:
//   - as floats (dhq_fused_layer_xhat_kernel): written by the launch that made them, four bytes a feature in each
//     direction;
//   - not at all (dhq_fused_layer_kernel): a launch runs the layer below again, from that layer's input codes, which the
//     previous launch stored (they could only be quantized after the launch that made them), or from the coordinates, and
//     stores the codes it makes of the result for the next launch.  One byte a feature in each direction, and every
//     hidden layer computed twice.
// The same operations on the same values, so the same bits.  The floats are bound by memory from about half a pass of the
// chip on; the second computation costs its latency however few rows there are.  Five hidden layers of 256, floats / codes:
// 1 000 rows 65 / 82 us, 262 144 rows 561 (5.2 TB/s) / 324 us (bound by vector instruction issue as the whole-network kernel
// is); fused_pass_floats draws the line.  Everything crosses memory in the lanes' register order ([wave tile][k block][lane] x 16 B
// codes, [wave tile][float4][lane]: every access of a wave is 1 KiB contiguous); a wave overwrites the codes it has read
// itself, so one buffer of them serves all layers, while the floats take two in turn.
//   MODE 0  input layer (no layer below)   MODE 1  hidden layer   MODE 2  output layer: signal values out
struct fusedl_args {
    const float *coords;
    dhq_v4i *codes;            // MODE 1, 2: in (unless the layer below is the input layer); MODE 1: out
    const float4 *xin;         // floats, MODE 1, 2: in
    float4 *xout;              // floats, MODE 0, 1: out (not the buffer xin points to)
    float *out;                // MODE 2
    const unsigned char *blk;  // this layer's block of the packed weights (fragments, then biases)
    const unsigned char *blk_below;  // codes, MODE 1, 2: the block of the layer below
    const float *partial_in;   // max |x^| of this layer's input, one float per workgroup of the launch before
    int partial_count;
    int kp;                    // length of this layer's rotated input
    double c1_over_sa;         // epilogue multiplier divided by the activation scale
    float *dyn;                // this layer's {1 / (s_a sqrt(Kp)), epilogue multiplier, s_a}: written by workgroup 0
    const float *dyn_below;    // codes, MODE 1, 2: those of the layer below, written by the launch before
    float *partial;            // MODE 0, 1: max |x^| of the output per workgroup (not the buffer partial_in points to)
    int64_t n;
    int chunks, chunks_below;  // block sizes in KiB
    int k0, k0p, m_out, qmax;
    int dealt;                 // codes: which rows a wave takes (FUSED_DEALT or FUSED_IN_A_ROW)
    float c2;                  // wavelet activation: 2 pi s0 sqrt(log2 e) / omega0
    float scale, unscale;      // what the activations are multiplied by before they are split (padded networks), and 1 over it
};

// This layer's constants from the maxima of its input.
__device__ __forceinline__ void fusedl_constants(const fusedl_args &A, float (&red_in)[FUSED_WAVES], int wave, int lane, float &inv, float &c1)
{
    float mi = 0.f, s_a;
    for (int i = threadIdx.x; i < A.partial_count; i += FUSED_THREADS) mi = fmaxf(mi, A.partial_in[i]);
#pragma unroll
    for (int m = 1; m < 64; m *= 2) mi = fmaxf(mi, __shfl_xor(mi, m, 64));
    if (lane == 0) red_in[wave] = mi;
    __syncthreads();
    mi = red_in[0];
#pragma unroll
    for (int w = 1; w < FUSED_WAVES; ++w) mi = fmaxf(mi, red_in[w]);
    dhq_dyn_constants(mi, A.kp, A.qmax, A.c1_over_sa, inv, c1, s_a);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.dyn[0] = inv; A.dyn[1] = c1; A.dyn[2] = s_a;
    }
}
// Each workgroup's maximum of its lanes' mw.
__device__ __forceinline__ void fusedl_store_max(const fusedl_args &A, float (&red)[FUSED_WAVES], int wave, int lane, float mw)
{
#pragma unroll
    for (int m = 1; m < 64; m *= 2) mw = fmaxf(mw, __shfl_xor(mw, m, 64));
    if (lane == 0) red[wave] = mw;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = red[0];
#pragma unroll
        for (int w = 1; w < FUSED_WAVES; ++w) r = fmaxf(r, red[w]);
        A.partial[blockIdx.x] = r * A.unscale;
    }
}

// x^ between the launches as floats.  ACTK: the activation of the hidden layers (MODE 0, 1).
template <int NF, int MODE, int ACTK>
__global__ __launch_bounds__(FUSED_THREADS) void dhq_fused_layer_xhat_kernel(const fusedl_args A)
{
    constexpr int NT = NF / 32, NKB = NF / 32, NR = NF / 2;
    constexpr int KB = (MODE == 0) ? 1 : NKB;      // k blocks of this layer's GEMM
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ float red_in[FUSED_WAVES], red[FUSED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int64_t n_tiles = (A.n + FUSED_TILE - 1) / FUSED_TILE;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;
    dhq_v4i hA[2];
    fused_h32_operand<(ACTK & DHQ_TWO_DIGITS) != 0>(c, h, hA);
    fused_issue_copy(A.blk, lds, A.chunks, wave, lane, FUSED_WAVES);
    float inv, c1;
    fusedl_constants(A, red_in, wave, lane, inv, c1);
    const float inv_x = inv * A.unscale;
    float mx = 0.f;
    bool landed = false;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t ci = tile * FUSED_TILE + wave * 32 + c;
        const bool valid = ci < A.n;
        const int64_t cl = valid ? ci : A.n - 1;  // lanes past the end repeat the last coordinate: no effect on the maximum
        const size_t slot = ((size_t)tile * FUSED_WAVES + wave) * (NR / 4) * 64 + lane;
        dhq_v4i cd[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
        if constexpr (MODE == 0) {
            cd[0][0] = fused_input_codes(A.coords, cl, A.k0, A.k0p, inv, A.qmax);
        } else {
#pragma unroll
            for (int q = 0; q < NR / 4; ++q) {
                const float4 x = A.xin[slot + (size_t)q * 64];
                cd[q / 4][q % 4] = (int)fused_quant4(x.x, x.y, x.z, x.w, inv_x, qlo, qhi);
            }
        }
        if (!landed) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();  // the weights are in LDS
            landed = true;
        }
        if constexpr (MODE == 2) {
            fused_output_layer<NKB, DHQ_DIGITS(ACTK)>(reinterpret_cast<const dhq_v4i *>(lds),
                                    reinterpret_cast<const float *>(lds + KB * DHQ_DIGITS(ACTK) * 1024), cd, c1, A.out, ci, valid, A.m_out,
                                    lane, h);
        } else {
            dhq_v16f xt[NT];
            fused_layer_gemm<NT, KB, NKB, ACTK>(lds, cd, c1, xt, hA, lane, h, A.c2, A.scale);
            fused_tile_stages<NT>(xt);
#pragma unroll
            for (int q = 0; q < NR / 4; ++q) {
                const float4 x = make_float4(xt[q >> 2][4 * (q & 3)], xt[q >> 2][4 * (q & 3) + 1], xt[q >> 2][4 * (q & 3) + 2],
                                             xt[q >> 2][4 * (q & 3) + 3]);
                mx = fmaxf(fmaxf(mx, fmaxf(fabsf(x.x), fabsf(x.y))), fmaxf(fabsf(x.z), fabsf(x.w)));
                A.xout[slot + (size_t)q * 64] = x;
            }
        }
    }
    if constexpr (MODE != 2) fusedl_store_max(A, red, wave, lane, mx);
}

// Codes between the launches, the layer below computed again.
// BELOW0: the layer below is the input layer.  ACTK: the activation of the hidden layers.
template <int NF, int MODE, bool BELOW0, int ACTK>
__global__ __launch_bounds__(FUSED_THREADS) void dhq_fused_layer_kernel(const fusedl_args A)
{
    constexpr int NT = NF / 32, NKB = NF / 32;
    constexpr int KB = (MODE == 0) ? 1 : NKB;      // k blocks of this layer's GEMM
    constexpr int KBB = BELOW0 ? 1 : NKB;          // k blocks of the layer below
    constexpr int MT = (MODE == 2) ? 1 : NT;       // M tiles of this layer's GEMM
    extern __shared__ __align__(16) unsigned char lds[];  // this layer's block, then that of the layer below
    __shared__ float red_in[FUSED_WAVES], red[FUSED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int64_t n_tiles = A.dealt ? (A.n + 31) / 32 : (A.n + FUSED_TILE - 1) / FUSED_TILE;
    const int64_t stride = A.dealt ? (int64_t)gridDim.x * FUSED_WAVES : gridDim.x;
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;
    dhq_v4i hA[2];
    fused_h32_operand<(ACTK & DHQ_TWO_DIGITS) != 0>(c, h, hA);
    fused_issue_copy(A.blk, lds, A.chunks, wave, lane, FUSED_WAVES);
    const unsigned char *lds_below = lds + (MT * KB + 1) * 1024;
    float inv_below = 0.f, c1_below = 0.f;
    if constexpr (MODE != 0) {
        fused_issue_copy(A.blk_below, lds + (MT * KB + 1) * 1024, A.chunks_below, wave, lane, FUSED_WAVES);
        inv_below = A.dyn_below[0];
        c1_below = A.dyn_below[1];
    }
    float inv, c1;
    if ((ACTK & DHQ_PLAIN) != 0 && A.partial_count == 0) {  // an earlier launch has left them
        inv = A.dyn[0];
        c1 = A.dyn[1];
    } else {
        fusedl_constants(A, red_in, wave, lane, inv, c1);
    }
    const dhq_v4i *wA = reinterpret_cast<const dhq_v4i *>(lds);
    float mx[4] = {0.f, 0.f, 0.f, 0.f};  // four chains of three-operand maxima
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // the weights are in LDS
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += stride) {
        const int64_t wave_tile = A.dealt ? tile + (int64_t)uwave * gridDim.x : tile * FUSED_WAVES + uwave;
        const bool active = wave_tile * 32 < A.n;
        const int64_t ci = wave_tile * 32 + c;
        const bool valid = ci < A.n;
        const int64_t cl = valid ? ci : A.n - 1;  // lanes past the end repeat the last coordinate: no effect on the maximum
        dhq_v4i *const codes = A.codes + (size_t)wave_tile * NKB * 64 + lane;
        dhq_v4i cd[NKB];
        dhq_v16f xt[NT];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
        if (!active) {
        } else if constexpr (MODE == 0 || BELOW0) {
            cd[0][0] = fused_input_codes(A.coords, cl, A.k0, A.k0p, MODE == 0 ? inv : inv_below, A.qmax);
        } else {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) cd[kb] = codes[kb * 64];
        }
        if constexpr (MODE != 0) {
            if (active)
                fused_gemm_sine_hm<NT, KBB, NKB, ACTK>(reinterpret_cast<const dhq_v4i *>(lds_below),
                                                   reinterpret_cast<const float4 *>(lds_below + NT * KBB * 1024), cd, c1_below, xt, hA,
                                                   lane, h, A.c2, A.scale);
            __syncthreads();  // keeps the two waves of a SIMD in the same phase, as in the whole-network kernel
            if (active) {
                if constexpr ((ACTK & DHQ_PLAIN) != 0) fused_butterflies<NT, DHQ_SKIP(ACTK)>(xt);
                else fused_tile_stages<NT, DHQ_SKIP(ACTK)>(xt);
                fused_quantize<NT>(xt, cd, hm_scaled<ACTK>(inv, A.unscale), qlo, qhi);
                if constexpr ((ACTK & DHQ_PLAIN) != 0) fused_plain_codes<NT>(cd);
                if constexpr (MODE == 1) {
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb) codes[kb * 64] = cd[kb];
                }
            }
        }
        if ((ACTK & DHQ_PLAIN) != 0 && !A.partial) continue;  // only the codes are wanted
        if constexpr (MODE == 2) {
            if (active) fused_output_layer<NKB>(wA, reinterpret_cast<const float *>(lds + MT * KB * 1024), cd, c1, A.out, ci, valid, A.m_out,
                                    lane, h);
        } else {
            if (active)
                fused_gemm_sine_hm<NT, KB, NKB, ACTK>(wA, reinterpret_cast<const float4 *>(lds + MT * KB * 1024), cd, c1, xt, hA, lane, h,
                                                      A.c2, A.scale);
            __syncthreads();
            if (active) {
                if constexpr ((ACTK & DHQ_PLAIN) != 0) fused_butterflies<NT, DHQ_SKIP(ACTK)>(xt);
                else fused_tile_stages<NT, DHQ_SKIP(ACTK)>(xt);
#pragma unroll
                for (int T = 0; T < NT; ++T) {
#pragma unroll
                    for (int v = 0; v < 16; v += 2) mx[(v >> 1) & 3] = fmaxf(fmaxf(fabsf(xt[T][v]), fabsf(xt[T][v + 1])), mx[(v >> 1) & 3]);
                }
            }
        }
    }
    if ((ACTK & DHQ_PLAIN) != 0 && !A.partial) return;
    if constexpr (MODE != 2) fusedl_store_max(A, red, wave, lane, fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])));
}

// The feature of row r of a two-digit layer (its own inverse).
constexpr __host__ __device__ int two_digit_feature(int r) { return (r & ~5) | (r & 1) << 2 | (r >> 2 & 1); }

// ---- test hook: one layer of the whole-network kernel on caller-supplied codes ---------------
// The layer body is the code dhq_fused_kernel runs (fused_gemm_sine_hm, fused_tile_stages,
// fused_quant4 on the same packed weights); only the way in and out differs: the input codes
// are gathered from a row-major n x Kp array into the lanes' register order, and the
// un-normalised transform x^ of the layer's output and the codes the next layer's quantizer
// makes of it are scattered back to row-major n x NF arrays in rotated-feature order.  The
// integer accumulators come from a second, plain MFMA loop over the same fragments and codes.  Two digits: those are the
// un-rotated ones, z = H acc' over the outputs, which fusedd_rotate_kernel takes back to the rotated ones, acc' = H z / NF.
struct fusedd_args {
    const int8_t *codes_in;    // n x kp_in, rotated-feature order
    const unsigned char *blk;  // the layer's block of the packed weights
    float *xhat;               // n x NF or null
    int8_t *codes_out;         // n x NF or null
    int32_t *acc;              // n x NF or null
    int64_t n;
    int chunks, kp_in, qmax;
    float c1, inv_next, c2;
};

template <int NF, bool FIRST, int ACTK>
__global__ __launch_bounds__(FUSED_THREADS) void dhq_fused_debug_kernel(const fusedd_args A)
{
    constexpr int NT = NF / 32, NKB = NF / 32, NR = NF / 2;
    constexpr int KB = FIRST ? 1 : NKB;
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;
    dhq_v4i hA[2];
    fused_h32_operand<(ACTK & DHQ_TWO_DIGITS) != 0>(c, h, hA);
    fused_issue_copy(A.blk, lds, A.chunks, wave, lane, FUSED_WAVES);
    const int64_t ci = (int64_t)blockIdx.x * FUSED_TILE + wave * 32 + c;
    const bool valid = ci < A.n;
    const int64_t cl = valid ? ci : A.n - 1;
    dhq_v4i cd[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
    if constexpr (FIRST) {
        // the input layer's (<= 4) codes sit in bytes 0.. of dword 0, whichever lane half
        unsigned w = 0;
        for (int k = 0; k < A.kp_in; ++k) w |= (unsigned)(uint8_t)A.codes_in[cl * A.kp_in + k] << (8 * k);
        cd[0][0] = (int)w;
    } else {
#pragma unroll
        for (int s = 0; s < NR; ++s) {
            const int f = 32 * (s >> 4) + 8 * ((s >> 2) & 3) + 4 * h + (s & 3);  // rotated feature of register s
            const unsigned byte = (unsigned)(uint8_t)A.codes_in[cl * A.kp_in + f];
            cd[s >> 4][(s >> 2) & 3] |= (int)(byte << (8 * (s & 3)));
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (A.acc) {
        constexpr int D = DHQ_DIGITS(ACTK), TH = NT / fused_halves<NT, KB, ACTK>;  // tiles of a block
#pragma unroll
        for (int T = 0; T < NT; ++T) {
            const dhq_v4i *wA = reinterpret_cast<const dhq_v4i *>(lds + T / TH * (fused_block_kib<NT, KB, ACTK> * 1024)) + T % TH * D * KB * 64 + lane;
            dhq_v16i acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
            for (int kb = 0; kb < D * KB; ++kb) {
                if (D > 1 && kb == KB) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[v] = (int)((unsigned)acc[v] << 8);
                }
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wA[kb * 64], cd[kb % KB], acc, 0, 0, 0);
            }
            if (valid) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                    A.acc[ci * NF + 32 * T + (D > 1 ? two_digit_feature(row) : row)] = acc[v];
                }
            }
        }
    }
    dhq_v16f xt[NT];
    fused_layer_gemm<NT, KB, NKB, ACTK>(lds, cd, A.c1, xt, hA, lane, h, A.c2);
    __syncthreads();
    fused_tile_stages<NT>(xt);
    fused_quantize<NT>(xt, cd, A.inv_next, qlo, qhi);
    if (valid) {
#pragma unroll
        for (int s = 0; s < NR; ++s) {
            const int f = 32 * (s >> 4) + 8 * ((s >> 2) & 3) + 4 * h + (s & 3);
            if (A.xhat) A.xhat[ci * NF + f] = xt[s >> 4][s & 15];
            if (A.codes_out) A.codes_out[ci * NF + f] = (int8_t)(((unsigned)cd[s >> 4][(s >> 2) & 3] >> (8 * (s & 3))) & 0xffu);
        }
    }
}

// One row per workgroup of NF threads, in place.  (A sum that NF does not divide is no product with the rotated weights.)
__global__ void fusedd_rotate_kernel(int32_t *acc)
{
    __shared__ int32_t z[256];
    int32_t *const row = acc + (size_t)blockIdx.x * blockDim.x;
    const int j = threadIdx.x, n = blockDim.x;
    z[j] = row[j];
    __syncthreads();
    long long s = 0;
    for (int k = 0; k < n; ++k) s += (__builtin_popcount(j & k) & 1) ? -(long long)z[k] : z[k];
    row[j] = s % n == 0 ? (int32_t)(s / n) : INT32_MIN;
}

// ------------------------------------------------------------------------------- host code
// `padded`: hidden widths that are no kernel's width, or differ, but all round up to the same one's.
// Two-sided models: whole-network kernels for the exact widths only.  Fan-ins above 4: with the padded plans, exact widths too.
static bool fused_shape_ok(const dhq_model *m, bool padded, int *nf_out)
{
    const int L = m->n_layers;
    if (L < 2) return false;
    if (m->dims[L] > 32) return false;
    const int nf = dhq_padded_width(m->dims, L);
    if (nf != 32 && nf != 64 && nf != 128 && nf != 256) return false;
    if (m->dims[0] > 4) {
        if (!padded || m->layer[0].Kp > dhq_most_input_codes(nf / 32)) return false;
    } else if (dhq_all_hidden_are(m->dims, L, nf) == padded) {
        return false;
    }
    if (padded && !dhq_pad_act_ok(m->act_kind, dhq_hidden_act(m).c2)) return false;
    *nf_out = nf;
    return true;
}

int dhq_fused_create(const dhq_model *m, bool padded, dhq_fused_plan **plan_out)
{
    *plan_out = nullptr;
    int nf = 0;
    if (!fused_shape_ok(m, padded, &nf)) return DHQ_OK;
    const int L = m->n_layers;
    const int NT = nf / 32, NKB = nf / 32;

    dhq_fused_plan *P = new (std::nothrow) dhq_fused_plan();
    if (!P) return DHQ_ENOMEM;
    P->nf = nf;
    P->act_kind = m->act_kind;
    P->padded = padded;
    P->digits = m->rot_out ? 2 : 1;
    const int D = P->digits, halves = NT * NKB * D > 64 ? 2 : 1;
    int widest = 0;
    for (int l = 1; l < L; ++l) widest = m->dims[l] > widest ? m->dims[l] : widest;
    P->skip = NT - (widest + 31) / 32;
    memset(&P->args, 0, sizeof(P->args));
    P->args.scale = padded && m->dims[0] <= 4 ? ldexpf(1.f, dhq_piece_scale_log2(m->act_kind, dhq_hidden_act(m).c2)) : 1.f;

    // block sizes: fragments [Mt][digit][Kb] KiB + one KiB of biases; hidden layers in `halves` such blocks
    std::vector<unsigned char> blob;
    for (int l = 0; l < L; ++l) {
        const dhq_layer &Ly = m->layer[l];
        const int Mt = (l == L - 1) ? 1 : NT;
        const int Kb = (l == 0) ? (Ly.Kp + 31) / 32 : NKB;
        const int H = (l == 0 || l == L - 1) ? 1 : halves, th = Mt / H;  // blocks, tiles of a block
        const size_t off = blob.size(), block = (size_t)(th * D * Kb + 1) * 1024;
        blob.resize(off + H * block, 0);
        // rotated-index order: the codes (M x Kp), or their product with H over the outputs (Mp x Kp), of which the outputs' rows
        const int8_t *wq = Ly.wq_host.data();
        const int32_t *u2 = Ly.u_host.data();
        // position of byte jj of lane half u in k block kb: the input layer's codes sit in natural order, 16 to a lane half
        int pos[2 * 32 * 8];
        for (int kb = 0; kb < Kb; ++kb)
            for (int u = 0; u < 2; ++u)
                for (int jj = 0; jj < 16; ++jj) pos[(kb * 2 + u) * 16 + jj] = l == 0 ? 32 * kb + 16 * u + jj : hm_index(16 * kb + jj, u);
        for (int T = 0; T < Mt; ++T)
            for (int ln = 0; ln < 64; ++ln) {
                const int u = ln >> 5, row = 32 * T + (D == 2 && l < L - 1 ? two_digit_feature(ln & 31) : ln & 31);
                if (row >= Ly.M) continue;
                int8_t *frag = reinterpret_cast<int8_t *>(blob.data() + off + (T / th) * block) + ((size_t)(T % th) * D * Kb * 64 + ln) * 16;
                for (int kb = 0; kb < Kb; ++kb, frag += 1024) {
                    const int *k = pos + (kb * 2 + u) * 16;
                    if (D == 1) {
                        for (int jj = 0; jj < 16; ++jj)
                            if (k[jj] < Ly.Kp) frag[jj] = wq[(size_t)row * Ly.Kp + k[jj]];
                    } else {
                        for (int jj = 0; jj < 16; ++jj)
                            if (k[jj] < Ly.Kp) {
                                const int32_t w = u2[(size_t)row * Ly.Kp + k[jj]], w0 = ((w + 128) & 255) - 128;
                                frag[jj] = (int8_t)((w - w0) / 256);
                                frag[(size_t)Kb * 1024 + jj] = (int8_t)w0;
                            }
                    }
                }
            }
        // the bias blocks: [T][g][h][e], in revolutions for the sine layers
        {
            const std::vector<float> &src = (l == L - 1) ? Ly.bias_host : Ly.bias_rev_host;
            const int F = (l == L - 1) ? Ly.M : nf;
            for (int r = 0; r < F; ++r) {
                const int f = D == 2 && l < L - 1 ? two_digit_feature(r) : r;
                float *bias = reinterpret_cast<float *>(blob.data() + off + (r / 32 / th) * block + block - 1024);
                bias[bias_slot(r % (32 * th))] = f < Ly.M ? src[f] : dhq_pad_bias(m->act_kind, f);
            }
        }
        P->args.layer[l].blob_off = (uint32_t)off;
        P->args.layer[l].chunks = (uint32_t)(H * block / 1024);
    }
    P->blob_bytes = blob.size();
    if (hipMalloc((void **)&P->blob_dev, P->blob_bytes) != hipSuccess) {
        delete P;
        return DHQ_ENOMEM;
    }
    if (hipMemcpy(P->blob_dev, blob.data(), P->blob_bytes, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(P->blob_dev);
        delete P;
        return DHQ_EHIP;
    }
    P->args.blob = P->blob_dev;
    P->args.n_layers = L;
    P->args.k0 = m->dims[0];
    P->args.k0p = m->layer[0].Kp;
    P->args.kb0 = (m->layer[0].Kp + 31) / 32;
    P->args.m_out = m->dims[L];
    P->args.qmax = m->qmax_a;
    P->lds_bytes = (size_t)2 * (NT * NKB * D / halves + 1) * 1024;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, m->device) != hipSuccess) {
        (void)hipFree(P->blob_dev);
        delete P;
        return DHQ_EHIP;
    }
    P->n_cu = prop.multiProcessorCount;
    P->device = m->device;
    *plan_out = P;
    return DHQ_OK;
}

void dhq_fused_destroy(dhq_fused_plan *plan)
{
    if (!plan) return;
    if (plan->blob_dev) (void)hipFree(plan->blob_dev);
    delete plan;
}

// Refreshes the per-layer constants after the activation scales changed.
int dhq_fused_update_scales(const dhq_model *m, dhq_fused_plan *P)
{
    if (!P) return DHQ_OK;
    for (int l = 0; l < m->n_layers; ++l) {
        const dhq_layer &Ly = m->layer[l];
        P->args.layer[l].c1 = dhq_c1(m, l);
        P->args.layer[l].inv_in = (float)(1.0 / ((double)Ly.s_a * sqrt((double)Ly.Kp)));
        if (l > 0) P->args.layer[l].inv_in /= P->args.scale;  // a power of two
    }
    return DHQ_OK;
}

// The most 32-row tiles per CU that the split kernel takes: alone, or as the rest after full passes (a launch more).  Whole
// forwards of five hidden layers in us, split kernel / higher waves idle / all waves of fewer workgroups:
//   tiles per CU     1                  2                  3                  4
//   width 256 alone  12.2 / 24.1 / 32   18.9 / 25.4 / 33   27.5 / 26.5 / 34   34.2 / 27.7 / 34
//   width 256 rest   52.9 / 59.7 / 67   60.6 / 60.3 / 67   67.4 / 63.6 / 67   75.3 / 66.0 / 68
//   width 128 alone   9.2 / 12.3 / 16    9.5 / 12.8 / 17   11.7 / 13.1 / 17   14.1 / 13.5 / 17
//   width 128 rest   26.8 / 29.2 / 33   27.7 / 29.4 / 32   29.7 / 29.3 / 32   32.3 / 29.3 / 32
// Width 64 (six layers) alone 9.2 against 11.6 for all waves of fewer workgroups; as a rest it gains nothing over the launch.
// Two digits, split kernel / all waves of fewer workgroups, tiles per CU 2, 3, 4, 5, 6: width 256 alone 25/45 36/45 47/45, rest
// 76/91 86/91 97/91; width 128 alone 9.9/20 13/20 15/20 19/20 22/20, rest 31/39 33/39 35/39 41/38; width 64 alone 9.8/11.3 at 5,
// 11.5/11.3 at 6.
static int fused_split_most(int nf, int digits, bool rest)
{
    if (digits == 2) return nf == 256 ? 3 : nf == 128 ? (rest ? 4 : 5) : (rest ? 0 : 5);
    return nf == 256 ? (rest ? 1 : 2) : nf == 128 ? (rest ? 2 : 3) : (rest ? 0 : 4);
}
// A call's rows go to full passes of dhq_fused_kernel (FUSED_WAVES wave tiles of 32 rows per CU); what is left of a last
// pass runs on dhq_fused_split_kernel where that is faster than the pass.
template <int NF, int ACTK>
static hipError_t fused_launch_act(const dhq_fused_plan *P, fused_args &a, hipStream_t st)
{
    const int64_t tiles = (a.n + 31) / 32, pass = (int64_t)P->n_cu * FUSED_WAVES, rest = tiles % pass;
    int64_t head = a.n;  // rows for the full passes
    constexpr bool SPLIT = NF >= 64 && (ACTK & DHQ_PLAIN) == 0;
    if constexpr (SPLIT) {
        if (rest != 0 && rest <= (int64_t)fused_split_most(NF, DHQ_DIGITS(ACTK), tiles > pass) * P->n_cu) head = (tiles - rest) * 32;
    }
    const int64_t n = a.n;
    if (head > 0) {
        a.n = head;
        // Up to four waves of each workgroup have a SIMD each; more than that and fewer workgroups with all their waves
        // are as fast and use less power (width 256, 49 152 rows: 37.8 us against 39.2).  After many passes the test for an idle
        // wave has cost more than the last one gains.  Dealt / in a row, us, a last pass of 20 000 rows after 5, 10 and 20
        // full ones: 2 x 64 features 23.4 / 23.5, 41.5 / 41.3, 78.9 / 76.9; 3 x 256 115 / 119, 215 / 219, 416 / 419; of 35 000
        // rows after 1, 5 and 29: 3 x 64 wavelets 15.8 / 15.5, 42.3 / 41.5, 205 / 200; 2 x 32 features, where in a row is never
        // ahead, 6.6 / 6.7, 16.0 / 16.2, 73.4 / 73.7.
        constexpr bool ROWS_MATTER = NF >= 64 || DHQ_KIND(ACTK) != DHQ_ACT_KIND_SINE;
        const int64_t head_tiles = (head + 31) / 32, last = head_tiles % pass;
        // (With two digits the dealt form does not fit the registers: 676 bytes of scratch.)
        constexpr bool NO_DEALING = DHQ_DIGITS(ACTK) > 1;
        const bool most = NO_DEALING || last > 4 * (int64_t)P->n_cu, in_a_row = ROWS_MATTER && (most || head_tiles > 11 * pass);
        const int64_t want = most ? (head_tiles + FUSED_WAVES - 1) / FUSED_WAVES : head_tiles;
        const unsigned grid = (unsigned)(want < P->n_cu ? want : P->n_cu);
        auto kern = last == 0                ? dhq_fused_kernel<NF, ACTK, FUSED_WHOLE>
                    : in_a_row || NO_DEALING ? dhq_fused_kernel<NF, ACTK, FUSED_IN_A_ROW>
                                             : dhq_fused_kernel<NF, ACTK, NO_DEALING ? FUSED_IN_A_ROW : FUSED_DEALT>;
        hipError_t e = dhq_lds_limit_once(kern, P->lds_bytes, P->device);
        if (e != hipSuccess) return e;
        kern<<<grid, FUSED_THREADS, P->lds_bytes, st>>>(a);
        e = hipGetLastError();
        if (e != hipSuccess || head == n) return e;
    }
    if constexpr (SPLIT) {
        a.coords += head * a.k0;
        a.out += head * a.m_out;
        a.n = n - head;
        dhq_fused_split_kernel<NF, ACTK & 0xff><<<(unsigned)rest, NF * 2, 0, st>>>(a);
    }
    return hipGetLastError();
}
// The instance of a padded network: of the tiles that are all padding up to two are left out at width 256, one at 128 (the others
// have none).  Whole forwards of four hidden layers in us, all tiles / without those:
// 200 features, 65 536 rows 29.8 / 27.6; 140 (wavelet) 35.8 / 29.2; 180, on-line scales 84.1 / 71.4; 90, 131 072 rows 27.0 / 23.1;
// 200, 150 001 rows with calibration 271 / 255.
template <int NF, typename F>
static hipError_t fused_with_skip(int skip, F f)
{
    if constexpr (NF >= 256) {
        if (skip >= 2) return f(std::integral_constant<int, DHQ_SKIPPING(2)>{});
    }
    if constexpr (NF >= 128) {
        if (skip >= 1) return f(std::integral_constant<int, DHQ_SKIPPING(1)>{});
    }
    return f(std::integral_constant<int, 0>{});
}
template <int NF>
static hipError_t fused_launch_t(const dhq_fused_plan *P, fused_args &a, int act_kind, hipStream_t st)
{
    auto padded = [&](auto flags) {
        constexpr int S = decltype(flags)::value;
        if (act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) return fused_launch_act<NF, DHQ_ACT_KIND_WAVELET_COMPLEX | S>(P, a, st);
        return act_kind == DHQ_ACT_KIND_WAVELET ? fused_launch_act<NF, DHQ_ACT_KIND_WAVELET | S>(P, a, st)
                                                : fused_launch_act<NF, DHQ_ACT_KIND_SINE | S>(P, a, st);
    };
    if (a.codes0)
        return fused_with_skip<NF>(P->skip, [&](auto skip) {
            return padded(std::integral_constant<int, DHQ_PLAIN | DHQ_CODES_IN | decltype(skip)::value>{});
        });
    if (P->padded)
        return fused_with_skip<NF>(P->skip, [&](auto skip) { return padded(std::integral_constant<int, DHQ_SPLIT_RN | decltype(skip)::value>{}); });
    if (P->digits == 2)
        return act_kind == DHQ_ACT_KIND_WAVELET ? fused_launch_act<NF, DHQ_ACT_KIND_WAVELET | DHQ_TWO_DIGITS>(P, a, st)
                                                : fused_launch_act<NF, DHQ_ACT_KIND_SINE | DHQ_TWO_DIGITS>(P, a, st);
    if (act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) return fused_launch_act<NF, DHQ_ACT_KIND_WAVELET_COMPLEX>(P, a, st);
    return act_kind == DHQ_ACT_KIND_WAVELET ? fused_launch_act<NF, DHQ_ACT_KIND_WAVELET>(P, a, st)
                                            : fused_launch_act<NF, DHQ_ACT_KIND_SINE>(P, a, st);
}

hipError_t dhq_fused_launch(const dhq_model *m, const dhq_fused_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    if (!P) return hipErrorInvalidValue;
    // A fan-in above 4: the rotation and quantizer of the input are the layer-by-layer path's kernel, whose codes the whole-network
    // kernel reads (a launch more, n x Kp bytes of the model's workspace), a workspace full of rows at a time.  Its transform is
    // the calibration's (DHQ_PLAIN), so that the values are the layer-by-layer path's bit for bit.  4 hidden layers, 65 536 rows,
    // layer by layer / this way in us: 5 x 30 features 52.7 / 9.7, 12 x 90 (wavelet) 105 / 23.8, 40 x 60 69.1 / 18.3, 5 x 200 174 / 41.8,
    // 40 x 200 153 / 47.0; 12 x 200 on 700 rows 70.3 / 23.9; 12 x 300 325 / 131, 5 x 512 349 / 132 (dhq_pair2_launch).
    const bool wide_input = m->dims[0] > 4;
    const int64_t pass = (int64_t)P->n_cu * FUSED_TILE, room = DHQ_CHUNK * (int64_t)m->max_kp / P->args.k0p;
    const int64_t step = wide_input ? (room >= pass ? room / pass * pass : room) : n;
    for (int64_t off = 0; off < n; off += step) {
        fused_args a = P->args;
        a.coords = coords + off * a.k0;
        a.out = out + off * a.m_out;
        a.n = n - off < step ? n - off : step;
        a.c2 = dhq_hidden_act(m).c2;
        if (wide_input) {
            const dhq_layer &Ly = m->layer[0];
            const hipError_t e = dhq_launch_wht_quant(a.coords, a.n, Ly.K, Ly.Kp, a.layer[0].inv_in, m->qmax_a, m->codes, nullptr, st);
            if (e != hipSuccess) return e;
            a.codes0 = m->codes;
        }
        hipError_t e;
        switch (P->nf) {
            case 32: e = fused_launch_t<32>(P, a, m->act_kind, st); break;
            case 64: e = fused_launch_t<64>(P, a, m->act_kind, st); break;
            case 128: e = fused_launch_t<128>(P, a, m->act_kind, st); break;
            case 256: e = fused_launch_t<256>(P, a, m->act_kind, st); break;
            default: return hipErrorInvalidValue;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Whether the launches of a dynamic call on n rows pass floats (see the kernels).  The codes' time goes by whole passes of the
// chip (FUSED_TILE rows per CU), the floats' by rows, so the floats are ahead in a pass that few CUs take part in: at most these
// 256ths of them, in the first, the second and the third pass.  Measured, floats / codes in us, four or five hidden
// layers (one, complex), by CUs in use:
//                     16         64         96        128        256        264        304
//   sine 32         26 /  28    27 /  28    28 /  28    30 /  29    32 /  29    38 /  36    38 /  36
//   sine 64         30 /  33    32 /  34    33 /  35    37 /  35    48 /  36    57 /  49    57 /  49
//   sine 128        41 /  46    48 /  47    51 /  48    55 /  49    78 /  51    95 /  76    98 /  76
//   sine 256        67 /  84    80 /  85    88 /  86    97 /  88   139 /  99   176 / 155   179 / 153
//   wavelet 32      23 /  25    24 /  26    25 /  26    26 /  26    28 /  27    33 /  34    33 /  35
//   wavelet 64      28 /  32    29 /  33    30 /  33    33 /  33    42 /  35    50 /  48    51 /  49
//   wavelet 128     38 /  46    43 /  47    47 /  48    50 /  49    68 /  50    84 /  78    86 /  79
//   wavelet 256     64 /  84    73 /  85    81 /  86    88 /  87   115 /  93   147 / 152   153 / 154
//   complex 64      11 /  12    11 /  12    11 /  12    12 /  12    13 /  12    15 /  16    16 /  16
//   complex 256     19 /  23    20 /  23    21 /  23    23 /  23    32 /  23    41 /  37    41 /  37
// (The codes' times follow the clock the card sustains, 7 % up or down from one card to the next; the floats' do not.)
static bool fused_pass_floats(const dhq_fused_plan *P, int64_t n)
{
    static const short most[4][3][3] = {
        {{104, 0, 0}, {176, 192, 32}, {176, 160, 200}},  // width 32: sine, wavelet, complex wavelet
        {{120, 0, 0}, {136, 0, 0}, {200, 48, 0}},        // 64
        {{62, 0, 0}, {110, 0, 0}, {168, 0, 0}},          // 128
        {{80, 0, 0}, {120, 112, 0}, {128, 0, 0}},        // 256
    };
    const int64_t tiles = (n + FUSED_TILE - 1) / FUSED_TILE, pass = (tiles - 1) / P->n_cu, in_last = tiles - pass * P->n_cu;
    const int w = P->nf == 32 ? 0 : P->nf == 64 ? 1 : P->nf == 128 ? 2 : 3;
    const int k = P->act_kind == DHQ_ACT_KIND_WAVELET ? 1 : P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX ? 2 : 0;
    if (P->digits == 2) return n > 0;  // the layer below again would need its weights in LDS as well
    return n > 0 && pass < 3 && in_last * 256 <= (int64_t)most[w][k][pass] * P->n_cu;
}

// The dynamic mode on the per-layer kernels above.  ws[0], ws[1]: two buffers of ws_bytes each, at least
// dhq_fused_dynamic_bytes (rows rounded up to whole workgroup tiles); the codes take the first one, the floats both;
// partial: room for 2 x DHQ_ABSMAX_PARTIALS floats (two sets of per-workgroup maxima, used alternately: a layer's slower
// workgroups still read one set while its faster ones already write the other); dyn: three floats per layer.
size_t dhq_fused_dynamic_rows(int64_t n) { return (size_t)((n + FUSED_TILE - 1) / FUSED_TILE) * FUSED_TILE; }
// What any call of up to n rows takes of each buffer: its codes, or the floats of the most rows up to n that pass them.
size_t dhq_fused_dynamic_bytes(const dhq_fused_plan *P, int64_t n)
{
    const int64_t last = (int64_t)3 * P->n_cu * FUSED_TILE;
    int64_t floats = n < last || P->digits == 2 ? n : last;
    while (floats > 0 && !fused_pass_floats(P, floats)) floats -= FUSED_TILE;
    const size_t codes = dhq_fused_dynamic_rows(n) * (size_t)P->nf;
    const size_t xhat = floats > 0 ? dhq_fused_dynamic_rows(floats) * (size_t)P->nf * sizeof(float) : 0;
    return codes > xhat ? codes : xhat;
}

// Whether the launches that pass codes deal 32-row tiles over all workgroups: a last pass that at most half of the waves have a
// tile in, as in the whole-network kernel.
static bool fused_deal(const dhq_fused_plan *P, int64_t n)
{
    const int64_t waves = (int64_t)P->n_cu * FUSED_WAVES, tiles = (n + 31) / 32, last = tiles % waves;
    return tiles > waves && last > 0 && 2 * last <= waves;
}

template <int NF, int MODE, bool BELOW0, int ACTK>
static hipError_t fusedl_launch_t(const fusedl_args &a, unsigned grid, int device, hipStream_t st)
{
    auto kern = dhq_fused_layer_kernel<NF, MODE, BELOW0, ACTK>;
    const size_t lds = (size_t)(a.chunks + a.chunks_below) * 1024;
    hipError_t e = dhq_lds_limit_once(kern, lds, device);
    if (e != hipSuccess) return e;
    kern<<<grid, FUSED_THREADS, lds, st>>>(a);
    return hipGetLastError();
}
template <int NF, int MODE, int ACTK>
static hipError_t fusedl_launch_xhat(const fusedl_args &a, unsigned grid, int device, hipStream_t st)
{
    auto kern = dhq_fused_layer_xhat_kernel<NF, MODE, ACTK>;
    const size_t lds = (size_t)a.chunks * 1024;
    hipError_t e = dhq_lds_limit_once(kern, lds, device);
    if (e != hipSuccess) return e;
    kern<<<grid, FUSED_THREADS, lds, st>>>(a);
    return hipGetLastError();
}
template <int NF, int ACTK>
static hipError_t fusedl_launch_layer(int layer, int n_layers, const fusedl_args &a, unsigned grid, int device, hipStream_t st)
{
    // the complex wavelet has a bound on its arguments with on-line scales for one hidden layer only, which the caller checks
    constexpr bool ONE_HIDDEN = (DHQ_KIND(ACTK) == DHQ_ACT_KIND_WAVELET_COMPLEX);
    if (ONE_HIDDEN && n_layers != 2) return hipErrorInvalidValue;
    const bool last = (layer == n_layers - 1);
    if (a.xout) {  // floats; the output layer has no activation
        if (layer == 0) return fusedl_launch_xhat<NF, 0, ACTK & 0xff>(a, grid, device, st);
        if (last) return fusedl_launch_xhat<NF, 2, DHQ_ACT_KIND_NONE | (ACTK & DHQ_TWO_DIGITS)>(a, grid, device, st);
        if constexpr (!ONE_HIDDEN) return fusedl_launch_xhat<NF, 1, ACTK & 0xff>(a, grid, device, st);
    } else if constexpr (DHQ_DIGITS(ACTK) == 1) {
        if (layer == 0) return fusedl_launch_t<NF, 0, false, ACTK>(a, grid, device, st);
        if (last && layer == 1) return fusedl_launch_t<NF, 2, true, ACTK>(a, grid, device, st);
        if constexpr (!ONE_HIDDEN) {
            if (last) return fusedl_launch_t<NF, 2, false, ACTK>(a, grid, device, st);
            return layer == 1 ? fusedl_launch_t<NF, 1, true, ACTK>(a, grid, device, st) : fusedl_launch_t<NF, 1, false, ACTK>(a, grid, device, st);
        }
    }
    return hipErrorInvalidValue;
}
template <int NF>
static hipError_t fusedl_launch_nf(const dhq_fused_plan *P, int layer, int L, const fusedl_args &a, unsigned grid, hipStream_t st)
{
    if (P->padded)
        return fused_with_skip<NF>(P->skip, [&](auto skip) {
            constexpr int S = DHQ_SPLIT_RN | decltype(skip)::value;
            if (P->act_kind == DHQ_ACT_KIND_WAVELET) return fusedl_launch_layer<NF, DHQ_ACT_KIND_WAVELET | S>(layer, L, a, grid, P->device, st);
            if (P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) return fusedl_launch_layer<NF, DHQ_ACT_KIND_WAVELET_COMPLEX | S>(layer, L, a, grid, P->device, st);
            return fusedl_launch_layer<NF, DHQ_ACT_KIND_SINE | S>(layer, L, a, grid, P->device, st);
        });
    if (P->digits == 2)
        return P->act_kind == DHQ_ACT_KIND_WAVELET ? fusedl_launch_layer<NF, DHQ_ACT_KIND_WAVELET | DHQ_TWO_DIGITS>(layer, L, a, grid, P->device, st)
                                                   : fusedl_launch_layer<NF, DHQ_ACT_KIND_SINE | DHQ_TWO_DIGITS>(layer, L, a, grid, P->device, st);
    if (P->act_kind == DHQ_ACT_KIND_WAVELET) return fusedl_launch_layer<NF, DHQ_ACT_KIND_WAVELET>(layer, L, a, grid, P->device, st);
    if (P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) return fusedl_launch_layer<NF, DHQ_ACT_KIND_WAVELET_COMPLEX>(layer, L, a, grid, P->device, st);
    return fusedl_launch_layer<NF, DHQ_ACT_KIND_SINE>(layer, L, a, grid, P->device, st);
}

hipError_t dhq_fused_dynamic_launch(const dhq_model *m, const dhq_fused_plan *P, const float *coords, int64_t n, float *out,
                                    void *const (&ws)[2], size_t ws_bytes, float *partial, float *dyn, hipStream_t st)
{
    if (!P) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    const int L = m->n_layers;
    const int64_t tiles = (n + FUSED_TILE - 1) / FUSED_TILE;
    const unsigned grid = (unsigned)(tiles < P->n_cu ? tiles : P->n_cu);
    // (buffers sized for the layer-by-layer path, whose rows are narrower than a padded network's, may be too small for floats)
    if (dhq_fused_dynamic_rows(n) * (size_t)P->nf > ws_bytes) return hipErrorInvalidValue;
    const bool floats = fused_pass_floats(P, n) && dhq_fused_dynamic_rows(n) * (size_t)P->nf * sizeof(float) <= ws_bytes;
    // the input layer's scale: max over the rotated coordinates, left as per-workgroup maxima
    float *pbuf[2] = {partial, partial + DHQ_ABSMAX_PARTIALS};
    int count = 0;
    hipError_t e = dhq_launch_wht_absmax_partials(coords, n, m->layer[0].K, m->layer[0].Kp, pbuf[0], &count, st);
    if (e != hipSuccess) return e;
    for (int l = 0; l < L; ++l) {
        fusedl_args a;
        memset(&a, 0, sizeof(a));
        a.coords = coords;
        a.codes = reinterpret_cast<dhq_v4i *>(ws[0]);
        if (floats) {
            a.xin = reinterpret_cast<const float4 *>(ws[(l + 1) & 1]);
            a.xout = reinterpret_cast<float4 *>(ws[l & 1]);
        }
        a.out = out;
        a.blk = P->blob_dev + P->args.layer[l].blob_off;
        a.chunks = (int)P->args.layer[l].chunks;
        if (l > 0) {
            a.blk_below = P->blob_dev + P->args.layer[l - 1].blob_off;
            a.chunks_below = (int)P->args.layer[l - 1].chunks;
            a.dyn_below = dyn + 3 * (l - 1);
        }
        a.partial_in = pbuf[l & 1];
        a.partial_count = count;
        a.kp = m->layer[l].Kp;
        a.c1_over_sa = dhq_c1_over_sa(m, l);
        a.dyn = dyn + 3 * l;
        a.partial = pbuf[(l + 1) & 1];
        a.n = n;
        a.dealt = fused_deal(P, n);
        a.k0 = P->args.k0; a.k0p = P->args.k0p; a.m_out = P->args.m_out; a.qmax = P->args.qmax;
        a.c2 = dhq_hidden_act(m).c2;
        a.scale = P->args.scale;
        a.unscale = 1.f / P->args.scale;
        switch (P->nf) {
            case 32: e = fusedl_launch_nf<32>(P, l, L, a, grid, st); break;
            case 64: e = fusedl_launch_nf<64>(P, l, L, a, grid, st); break;
            case 128: e = fusedl_launch_nf<128>(P, l, L, a, grid, st); break;
            case 256: e = fusedl_launch_nf<256>(P, l, L, a, grid, st); break;
            default: e = hipErrorInvalidValue;
        }
        if (e != hipSuccess) return e;
        count = (int)grid;
    }
    return hipSuccess;
}

// ---- calibration ------------------------------------------------------------------------------
// The scales of all layers, with the layer-by-layer kernels' bits: dhq_fused_layer_kernel with the transform in fp32
// (DHQ_PLAIN), one launch per hidden layer: it computes the layer below once more from its codes, stores the codes that this makes,
// computes the layer and leaves the maximum of its transform.  Bound by vector issue like the whole-network kernel (eight
// add/sub stages in place of the products with H_32).  Four layers of 200 on 150 001 rows, forward included: 782 us with a
// GEMM, a transform and a maximum over memory each, twice a layer; this way 255 us (24 of the
// difference by a copy of the scales into pinned memory, 16 by leaving out the padding's tile).  buf_bytes of codes in each of two buffers: calls with more rows
// run in groups, and those beyond two groups make their codes again from the coordinates for every layer (hipErrorInvalidValue beyond eight groups: too many maxima).
template <int NF, int ACTK>
static hipError_t fused_measure_layer(int layer, const fusedl_args &a, unsigned grid, int device, hipStream_t st)
{
    if (layer == 0) return fusedl_launch_t<NF, 0, false, ACTK | DHQ_PLAIN>(a, grid, device, st);
    return layer == 1 ? fusedl_launch_t<NF, 1, true, ACTK | DHQ_PLAIN>(a, grid, device, st)
                      : fusedl_launch_t<NF, 1, false, ACTK | DHQ_PLAIN>(a, grid, device, st);
}
template <int NF>
static hipError_t fused_measure_nf(const dhq_fused_plan *P, int layer, const fusedl_args &a, unsigned grid, hipStream_t st)
{
    return fused_with_skip<NF>(P->skip, [&](auto skip) {
        constexpr int S = decltype(skip)::value;
        if (P->act_kind == DHQ_ACT_KIND_WAVELET) return fused_measure_layer<NF, DHQ_ACT_KIND_WAVELET | S>(layer, a, grid, P->device, st);
        if (P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) return fused_measure_layer<NF, DHQ_ACT_KIND_WAVELET_COMPLEX | S>(layer, a, grid, P->device, st);
        return fused_measure_layer<NF, DHQ_ACT_KIND_SINE | S>(layer, a, grid, P->device, st);
    });
}
hipError_t dhq_fused_measure_launch(const dhq_model *m, const dhq_fused_plan *P, const float *coords, int64_t n, void *const (&buf)[2],
                                    size_t buf_bytes, float *partial, float *dyn, hipStream_t st)
{
    const int L = m->n_layers;
    const int64_t pass = (int64_t)P->n_cu * FUSED_TILE, room = (int64_t)(buf_bytes / (size_t)P->nf) / FUSED_TILE * FUSED_TILE;
    const int64_t step = room >= pass ? room / pass * pass : room, groups = step > 0 ? (n + step - 1) / step : 9;
    if (n <= 0 || groups > DHQ_ABSMAX_PARTIALS / P->n_cu || groups > 8) return hipErrorInvalidValue;
    float *pbuf[2] = {partial, partial + DHQ_ABSMAX_PARTIALS};
    int count = 0;
    hipError_t e = dhq_launch_wht_absmax_partials(coords, n, m->layer[0].K, m->layer[0].Kp, pbuf[0], &count, st);
    for (int l = 0; l < L - 1 && e == hipSuccess; ++l) {
        int left = 0;  // maxima of this layer's launches
        for (int64_t g = 0; g < groups && e == hipSuccess; ++g) {
            const int64_t rows = n - g * step < step ? n - g * step : step, tiles = (rows + FUSED_TILE - 1) / FUSED_TILE;
            const unsigned grid = (unsigned)(tiles < P->n_cu ? tiles : P->n_cu);
            for (int k = groups > 2 && l > 1 ? 1 : l; k <= l && e == hipSuccess; ++k) {
                fusedl_args a;
                memset(&a, 0, sizeof(a));
                a.coords = coords + g * step * m->dims[0];
                a.codes = reinterpret_cast<dhq_v4i *>(buf[g & 1]);
                a.blk = P->blob_dev + P->args.layer[k].blob_off;
                a.chunks = (int)P->args.layer[k].chunks;
                if (k > 0) {
                    a.blk_below = P->blob_dev + P->args.layer[k - 1].blob_off;
                    a.chunks_below = (int)P->args.layer[k - 1].chunks;
                    a.dyn_below = dyn + 3 * (k - 1);
                }
                if (k == l) {
                    a.partial_in = pbuf[l & 1];
                    a.partial_count = count;
                    a.partial = pbuf[(l + 1) & 1] + left;
                }
                a.kp = m->layer[k].Kp;
                a.c1_over_sa = dhq_c1_over_sa(m, k);
                a.dyn = dyn + 3 * k;
                a.n = rows;
                a.dealt = fused_deal(P, rows);
                a.k0 = P->args.k0; a.k0p = P->args.k0p; a.m_out = P->args.m_out; a.qmax = P->args.qmax;
                a.c2 = dhq_hidden_act(m).c2;
                a.scale = a.unscale = 1.f;
                switch (P->nf) {
                    case 32: e = fused_measure_nf<32>(P, k, a, grid, st); break;
                    case 64: e = fused_measure_nf<64>(P, k, a, grid, st); break;
                    case 128: e = fused_measure_nf<128>(P, k, a, grid, st); break;
                    case 256: e = fused_measure_nf<256>(P, k, a, grid, st); break;
                    default: e = hipErrorInvalidValue;
                }
            }
            left += (int)grid;
        }
        count = left;
    }
    if (e != hipSuccess) return e;
    return dhq_launch_absmax_finish(pbuf[(L - 1) & 1], count, m->layer[L - 1].Kp, m->qmax_a, dhq_c1_over_sa(m, L - 1), dyn + 3 * (L - 1), st);
}

// Test hook behind dhq_forward_debug_fused: layer `layer` (one that ends in an activation) of the
// whole-network kernel on the caller's codes.
template <int NF, bool FIRST, int ACTK>
static hipError_t fusedd_launch_t(const fusedd_args &a, unsigned grid, int device, hipStream_t st)
{
    auto kern = dhq_fused_debug_kernel<NF, FIRST, ACTK>;
    const size_t lds = (size_t)a.chunks * 1024;
    hipError_t e = dhq_lds_limit_once(kern, lds, device);
    if (e != hipSuccess) return e;
    kern<<<grid, FUSED_THREADS, lds, st>>>(a);
    return hipGetLastError();
}
template <int NF>
static hipError_t fusedd_launch_nf(bool first, int digits, int act_kind, const fusedd_args &a, unsigned grid, int device, hipStream_t st)
{
    const bool wav = (act_kind == DHQ_ACT_KIND_WAVELET);
    if (digits == 2) {
        constexpr int W = DHQ_ACT_KIND_WAVELET | DHQ_TWO_DIGITS, N = DHQ_ACT_KIND_SINE | DHQ_TWO_DIGITS;
        if (first) return wav ? fusedd_launch_t<NF, true, W>(a, grid, device, st) : fusedd_launch_t<NF, true, N>(a, grid, device, st);
        return wav ? fusedd_launch_t<NF, false, W>(a, grid, device, st) : fusedd_launch_t<NF, false, N>(a, grid, device, st);
    }
    if (act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX)
        return first ? fusedd_launch_t<NF, true, DHQ_ACT_KIND_WAVELET_COMPLEX>(a, grid, device, st)
                     : fusedd_launch_t<NF, false, DHQ_ACT_KIND_WAVELET_COMPLEX>(a, grid, device, st);
    if (first) return wav ? fusedd_launch_t<NF, true, DHQ_ACT_KIND_WAVELET>(a, grid, device, st) : fusedd_launch_t<NF, true, DHQ_ACT_KIND_SINE>(a, grid, device, st);
    return wav ? fusedd_launch_t<NF, false, DHQ_ACT_KIND_WAVELET>(a, grid, device, st) : fusedd_launch_t<NF, false, DHQ_ACT_KIND_SINE>(a, grid, device, st);
}

hipError_t dhq_fused_debug_launch(const dhq_model *m, const dhq_fused_plan *P, int layer, const int8_t *codes_in, int64_t n, float *xhat,
                                  int8_t *codes_out, int32_t *acc, hipStream_t st)
{
    if (!P || layer < 0 || layer >= m->n_layers - 1) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    fusedd_args a;
    memset(&a, 0, sizeof(a));
    a.codes_in = codes_in;
    a.blk = P->blob_dev + P->args.layer[layer].blob_off;
    a.chunks = (int)P->args.layer[layer].chunks;
    a.xhat = xhat;
    a.codes_out = codes_out;
    a.acc = acc;
    a.n = n;
    a.kp_in = m->layer[layer].Kp;
    a.qmax = P->args.qmax;
    a.c1 = P->args.layer[layer].c1;
    a.inv_next = P->args.layer[layer + 1].inv_in;
    a.c2 = dhq_hidden_act(m).c2;
    const unsigned grid = (unsigned)((n + FUSED_TILE - 1) / FUSED_TILE);
    hipError_t e;
    switch (P->nf) {
        case 32: e = fusedd_launch_nf<32>(layer == 0, P->digits, m->act_kind, a, grid, P->device, st); break;
        case 64: e = fusedd_launch_nf<64>(layer == 0, P->digits, m->act_kind, a, grid, P->device, st); break;
        case 128: e = fusedd_launch_nf<128>(layer == 0, P->digits, m->act_kind, a, grid, P->device, st); break;
        case 256: e = fusedd_launch_nf<256>(layer == 0, P->digits, m->act_kind, a, grid, P->device, st); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess || P->digits != 2 || !acc) return e;
    fusedd_rotate_kernel<<<(unsigned)n, P->nf, 0, st>>>(acc);
    return hipGetLastError();
}
