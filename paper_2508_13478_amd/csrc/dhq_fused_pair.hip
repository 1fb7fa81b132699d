// Whole-network fused DHQ forward for hidden width 512, two waves per SIMD (gfx950).
//
// Same arithmetic, same data layout inside a wave and the same packed weight fragments as
// dhq_fused_wide.hip (features are the MFMA M dimension, a lane holds half of one coordinate's
// feature vector, the 32-point factor of the Walsh-Hadamard transform of Eq. 3 runs on the matrix
// unit over binary16 pieces, the factor over the tile index as register butterflies).  What
// differs is who holds what.  A 512-wide layer gives a lane 256 activations, which leaves room
// for one wave per SIMD only; such a lone wave pays the latency of every dependent instruction
// and cannot overlap its own matrix and vector instruction issue.  Here two waves share 32
// coordinates and split the output features of every layer:
//
//   wave role 0 computes M tiles 0..7, role 1 tiles 8..15 (half of the GEMM, of the epilogue, of
//   the split into binary16 pieces and of the H_32 products each); both hold all 512 input codes;
//
//   the transform over the tile index needs tile T and tile T + 8 together.  Its stages never mix
//   the rows of a tile, so the work is re-split by rows: of every pair (T, T + 8) role 0 finishes
//   rows 0..7 and role 1 rows 8..15.  Each wave therefore hands half of its H_32 results (8 of
//   the 16 values per tile and lane) to its partner through LDS and receives as many, then runs
//   all four stages on 16 tiles x 8 rows and quantizes them;
//
//   the two code dwords per k block that a wave produces and the two its partner produces are
//   joined in LDS, from where both read the whole B operand of the next layer.
//
// So that both roles run the same instructions on the same register numbers, role 1 takes the
// rows of H_32 in the order "16..31, 0..15" as the A operand of its H_32 products: the rows it
// keeps then sit in registers 0..7 of a tile like role 0's, and it sends registers 8..15 like
// role 0.  Its difference "own - partner" is minus the true one (it owns T + 8), which a negated
// quantizer multiplier for that half undoes.  Everything that tells the roles apart is a
// wave-uniform run-time value: an LDS or fragment offset, the H_32 operand, one sign.
//
// LDS: two 32 KiB weight buffers (a 512 x 512 layer is streamed in eight chunks, one M tile per
// role each, copied straight from device memory into LDS by all eight waves while the previous
// chunk is consumed), a 64 KiB exchange area and three 2 KiB bias blocks (the input layer's, and
// those of the hidden / output layers by layer parity, each copied in while the layer before runs).
#include <math.h>
#include <string.h>

#include <new>
#include <utility>
#include <vector>

#include "dhq_device.h"
#include "dhq_fused_common.h"
#include "dhq_internal.h"

#define PAIR_WAVES 8
#define PAIR_THREADS (PAIR_WAVES * 64)
#define PAIR_TILE 128          // coordinates per workgroup pass: four groups of 32
#define PAIR_NT 8              // M tiles per wave
#define PAIR_KB 16             // k blocks of a hidden layer
#define PAIR_BUF 32768         // bytes per weight buffer = bytes per chunk
#define PAIR_X 65536           // exchange area
#define PAIR_BIAS (2 * PAIR_BUF + PAIR_X)  // LDS offset of the bias blocks, 2 KiB each: [layer parity 0, 1, input layer]
#define PAIR_PF 2              // LDS prefetch distance of the A fragments, in MFMAs
#define PAIR_EARLY 4           // tiles whose outgoing rows leave during the GEMM phase

#define PAIR2_MAX_U 32639      // largest entry that two int8 digits hold: 256 * 127 + 127

struct pair_args {
    const float *coords;
    float *out;
    const unsigned char *blob;
    int64_t n;
    int n_layers;
    int k0, k0p;
    int m_out;
    int qmax;
    int n_chunks;              // weight chunks a coordinate pass goes through, in a cycle (the whole network: the input layer's, rt
                               // (padded 5 .. 8, exact 8; two-sided 16) for each further hidden layer, the output layer's; an odd count
                               // puts a pass's first chunk into the other buffer: buffers go by the running count)
    int chunk_base;            // first of them: 0 (the whole network), or a single layer's first chunk
    uint32_t bias_off;         // byte offset of the bias table in the blob: [layer][512] floats, bias_slot order per tile
    float c2;                  // wavelet activation: 2 pi s0 sqrt(log2 e) / omega0
    float c1[DHQ_MAX_LAYERS];
    float inv_in[DHQ_MAX_LAYERS];  // (behind split activations divided by `scale`)
    float scale;               // padded networks: what the activations are multiplied by before they are split
    const int8_t *codes0;      // the input layer's codes, where the fan-in is above 4 (DHQ_CODES_IN)
};

struct dhq_pair_plan {
    int act_kind = DHQ_ACT_KIND_SINE;
    bool padded = false;       // the network's own hidden widths are smaller, padded to 512
    int rt = PAIR_NT;          // tiles of each role that are not all padding
    unsigned char *blob_dev = nullptr;
    size_t blob_bytes = 0;
    pair_args args;
    size_t lds_bytes = 0;
    int n_cu = 0;
    int device = 0;
};

// ----------------------------------------------------------------------------- device code
struct pair_stream {
    const pair_args *A;
    unsigned char *lds;        // buffer 0, buffer 1, exchange area
    int wave, lane, role, grp;
    const unsigned char *cp_src;  // chunk being copied in: this wave's first block (uniform)
    unsigned cp_dst;              // LDS address of that block in the buffer it goes to (uniform)
    unsigned voff;                // lane * 16
};

__device__ __forceinline__ unsigned pair_lds_addr(const unsigned char *p)
{
    return (unsigned)(size_t)(__attribute__((address_space(3))) const unsigned char *)p;
}

// One KiB from device memory straight into LDS: lane i's 16 bytes go to LDS address dst + 16 i
// (dst travels in M0).  Inline assembly for the reason given at fused_issue_copy: the kernel orders
// these copies itself -- a destination is never read between the load and the "s_waitcnt vmcnt(0)" +
// barrier that precedes its first use -- and loads the compiler does not know about can only make its
// own vmcnt waits longer, never shorter.
__device__ __forceinline__ void pair_copy_kib(const pair_stream &S, const unsigned char *src, unsigned dst)
{
    // the source is wave-uniform; its halves go through readfirstlane so that the operand is a scalar register pair
    // whatever the compiler knows about it
    const unsigned long long a = (unsigned long long)src;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    const unsigned long long sa = ((unsigned long long)hi << 32) | lo;
    const unsigned m0v = __builtin_amdgcn_readfirstlane(dst);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(S.voff), "s"(sa), "s"(m0v) : "memory", "m0");
}

// LDS block of layer l's biases.
__device__ __forceinline__ int pair_bias_slot(int l) { return l == 0 ? 2 : (l & 1); }
// Layer l's biases (2 KiB) into their block: waves 0 and 1 move one KiB each.
__device__ __forceinline__ void pair_copy_bias(const pair_stream &S, int l)
{
    if (S.wave < 2)
        pair_copy_kib(S, S.A->blob + S.A->bias_off + (size_t)l * 2048 + S.wave * 1024,
                      pair_lds_addr(S.lds) + PAIR_BIAS + pair_bias_slot(l) * 2048 + S.wave * 1024);
}

// Entering chunk `cc` (a running count; chunk cc lives in buffer cc & 1): every wave has written
// its share of it (the wait, then the barrier) and nobody reads chunk cc - 1 any more, so chunk
// cc + 1 may overwrite that one.
__device__ __forceinline__ void pair_enter_chunk(pair_stream &S, int cc)
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    const int j = S.A->chunk_base + (cc + 1) % S.A->n_chunks;
    S.cp_src = S.A->blob + (size_t)j * PAIR_BUF + S.wave * 1024;
    S.cp_dst = pair_lds_addr(S.lds) + ((cc + 1) & 1) * PAIR_BUF + S.wave * 1024;
}

// Slot i of a chunk's copy moves the 1 KiB block wave + 8 i (i = 0..3: 32 blocks, eight waves).
template <int I>
__device__ __forceinline__ void pair_copy_slot(const pair_stream &S)
{
    pair_copy_kib(S, S.cp_src + I * 8192, S.cp_dst + I * 8192);
}

// Where wave w parks the outgoing half of tile t (slot t & 3), as two float4 per lane.
__device__ __forceinline__ float4 *pair_x_slot(const pair_stream &S, int w, int t)
{
    return reinterpret_cast<float4 *>(S.lds + 2 * PAIR_BUF + w * 8192 + (t & 3) * 2048) + S.lane;
}

// RT: the wave's tiles that are not all padding (exact networks: all eight).  The chunks, products and additions of the others
// are left out: their activations are zero.
template <int ACTK, int RT>
struct pair_ctx {
    pair_stream &S;
    dhq_v4i (&cd)[PAIR_KB];       // codes of the layer input: the B operands
    dhq_v16f (&y)[PAIR_NT];       // H_32 products of this wave's tiles
    const dhq_v4i (&hA)[2];       // H_32 (rows in this role's order) as an MFMA A operand, two k blocks
    const unsigned char *bufs[2];
    const float4 *bias;           // this layer's biases in LDS, this wave's first tile, lane half folded in
    int cc, layer;
    float c1, c2;
    float scale;                  // padded networks: what the activations are multiplied by before they are split
    dhq_v4i fr[PAIR_PF + 1];
    float4 bq[3];
    float4 bq0[4];
    dhq_v16i acc[2];
    unsigned hp[2][8], lp[2][8];  // binary16 pieces of the tile being drained and of the one before
    float ex, ey, et;             // et: the complex wavelet's real-part argument, waiting for the imaginary one
    float ar[4];
    float er[2];
    __device__ __forceinline__ pair_ctx(pair_stream &S_, dhq_v4i (&cd_)[PAIR_KB], dhq_v16f (&y_)[PAIR_NT], const dhq_v4i (&hA_)[2])
        : S(S_), cd(cd_), y(y_), hA(hA_)
    {
    }
};

__device__ __forceinline__ float pair_comp(const float4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// H_32 product K (0: low pieces of block 0, 1: high pieces of block 0, 2, 3: block 1) of tile T.
template <int T, int K, int ACTK, int RT>
__device__ __forceinline__ void pair_h32(pair_ctx<ACTK, RT> &C)
{
    constexpr int blk = K >> 1;
    dhq_v4i b;
#pragma unroll
    for (int d = 0; d < 4; ++d) b[d] = (int)((K & 1) ? C.hp[T & 1][4 * blk + d] : C.lp[T & 1][4 * blk + d]);
    dhq_v16f d;
    if constexpr (K == 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] = 0.f;
    } else {
        d = C.y[T];
    }
    C.y[T] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(dhq_v8h, C.hA[blk]), __builtin_bit_cast(dhq_v8h, b), d, 0, 0, 0);
}

// The outgoing half of tile T (registers 8..15) to this wave's exchange slot.
template <int T, int ACTK, int RT>
__device__ __forceinline__ void pair_send(pair_ctx<ACTK, RT> &C)
{
    float4 *dst = pair_x_slot(C.S, C.S.wave, T);
    dst[0] = make_float4(C.y[T][8], C.y[T][9], C.y[T][10], C.y[T][11]);
    dst[64] = make_float4(C.y[T][12], C.y[T][13], C.y[T][14], C.y[T][15]);
}

// The weight copy that runs while a hidden layer's chunk is consumed, by steps since the chunk was
// entered.
template <int REL, int ACTK, int RT>
__device__ __forceinline__ void pair_copy_rel(pair_ctx<ACTK, RT> &C)
{
    if constexpr (REL == 1) pair_copy_slot<0>(C.S);
    if constexpr (REL == 3) pair_copy_slot<1>(C.S);
    if constexpr (REL == 5) pair_copy_slot<2>(C.S);
    if constexpr (REL == 7) pair_copy_slot<3>(C.S);
}

// One step of a hidden layer's GEMM + epilogue + H_32 pipeline (every step is its own template
// instance, so all register indices are compile-time constants):
//   step G   MFMA (tile G / 16, k block G % 16); its A fragment was fetched PF steps earlier, and
//            when that prefetch crosses into the next chunk the chunk is entered first;
//            accumulator e = G - 16 is converted, e - 1 gets its multiply-add with the bias,
//            e - 2 its activation; the split of a finished pair of activations into binary16
//            pieces takes three more steps, and the four H_32 products of a tile issue one per
//            step once their pieces exist (two after the tile's 8th value, two after its 16th);
//            the outgoing halves of the first tiles leave for the exchange area once complete.
template <int G, int ACTK, int RT>
__device__ __forceinline__ void pair_step(pair_ctx<ACTK, RT> &C)
{
    constexpr int NM = RT * PAIR_KB, NE = RT * 16, PF = PAIR_PF;
    if constexpr (G >= 0 && G < NM) {
        constexpr int pf = G + PF;
        if constexpr (pf < NM) {
            if constexpr (pf % PAIR_KB == 0) pair_enter_chunk(C.S, C.cc + pf / PAIR_KB);
            C.fr[pf % (PF + 1)] = reinterpret_cast<const dhq_v4i *>(C.bufs[(pf / PAIR_KB) & 1])[(pf % PAIR_KB) * 64 + C.S.lane];
        }
    }
    if constexpr (G + PF >= 0 && G + PF < NM) pair_copy_rel<(G + PF) % PAIR_KB>(C);
    if constexpr (G == 9) pair_copy_bias(C.S, C.layer + 1);  // the next layer's biases; in place long before its first step
    if constexpr (G >= 0 && G < NM) {
        constexpr int t = G / PAIR_KB, kb = G % PAIR_KB;
        if constexpr (kb == 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) C.acc[t & 1][v] = 0;
        }
        C.acc[t & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(C.fr[G % (PF + 1)], C.cd[kb], C.acc[t & 1], 0, 0, 0);
    }
    if constexpr (G >= 0) {
        constexpr int e0 = G - PAIR_KB, e1 = e0 - 1, e2 = e0 - 2;
        constexpr int hq = e2 - 11;  // 16 t + {0, 1, 8, 9} -> product 0, 1, 2, 3 of tile t
        if constexpr (hq >= 0 && hq / 16 < RT) {
            constexpr int Th = hq / 16, r = hq % 16;
            if constexpr (r == 0) pair_h32<Th, 0>(C);
            if constexpr (r == 1) pair_h32<Th, 1>(C);
            if constexpr (r == 8) pair_h32<Th, 2>(C);
            if constexpr (r == 9) pair_h32<Th, 3>(C);
            if constexpr (r == 12 && Th < PAIR_EARLY) pair_send<Th>(C);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr ((e2 & 1) == 0) {
            constexpr int pl = (e2 - 4) / 2, ph = (e2 - 2) / 2;  // pairs whose low / high pieces are packed now
            if constexpr (e2 >= 4 && pl < NE / 2) C.lp[(pl / 8) & 1][pl % 8] = hm_pack_half2(C.er[0], C.er[1]);
            if constexpr (e2 >= 2 && ph < NE / 2) C.hp[(ph / 8) & 1][ph % 8] = hm_pack_hi<ACTK>(C.ar[(e2 - 2) & 3], C.ar[(e2 - 1) & 3]);
        } else {
            constexpr int pm = (e2 - 3) / 2;  // pair whose remainders are taken now
            if constexpr (e2 >= 3 && pm < NE / 2)
                hm_remainders(C.ar[(e2 - 3) & 3], C.ar[(e2 - 2) & 3], C.hp[(pm / 8) & 1][pm % 8], C.er[0], C.er[1]);
        }
        if constexpr (e2 >= 0 && e2 < NE) {
            if constexpr (DHQ_KIND(ACTK) == DHQ_ACT_KIND_WAVELET_COMPLEX) {
                // accumulators e2 - 1, e2 (e2 odd) are the features 2m, 2m + 1 = (Re, Im) of one complex feature; both
                // results are consumed from the step after this one on (the packing of the high pieces)
                if constexpr ((e2 & 1) == 0) C.et = C.ey;
                else dhq_activate_pair_rev<false>(C.et, C.ey, C.c2, C.ar[(e2 - 1) & 3], C.ar[e2 & 3], hm_scaled<ACTK>(1.f, C.scale));
            } else {
                C.ar[e2 & 3] = hm_scaled<ACTK>(dhq_activate_rev(C.ey, dhq_act{DHQ_KIND(ACTK), C.c2}), C.scale);
            }
        }
        if constexpr (e1 >= 0 && e1 < NE) C.ey = __builtin_fmaf(C.ex, C.c1, pair_comp(C.bq[(e1 / 4) % 3], e1 % 4));
        if constexpr (e0 >= 0 && e0 < NE) C.ex = (float)C.acc[(e0 / 16) & 1][e0 % 16];
        if constexpr (e0 + 8 >= 0 && (e0 + 8) % 4 == 0 && e0 + 8 < NE) {
            // biases of values e0 + 8 .. e0 + 11 (tile ge / 4, row group ge % 4), from device memory; the ring
            // slot's previous tenant, group ge - 3, had its last use in the multiply-add just above
            constexpr int ge = (e0 + 8) / 4;
            C.bq[ge % 3] = C.bias[ge * 2];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int ACTK, int RT, int... Gs>
__device__ __forceinline__ void pair_steps(pair_ctx<ACTK, RT> &C, std::integer_sequence<int, Gs...>)
{
    (pair_step<Gs - PAIR_PF>(C), ...);  // steps -PF (the copy's first steps) .. NSTEPS - 1
}

// A hidden layer: reads the input codes the transform left in the exchange area, then the GEMM
// pipeline over this wave's eight tiles.  cc is the running chunk count and is advanced.
template <int ACTK, int RT = PAIR_NT>
__device__ __forceinline__ void pair_hidden(pair_stream &S, int &cc, int layer, float c1, dhq_v4i (&cd)[PAIR_KB],
                                            dhq_v16f (&y)[PAIR_NT], const dhq_v4i (&hA)[2], int h)
{
    // last step with work: the send after the fourth H_32 product of the last tile would be
    // e2 - 11 = 16 (RT - 1) + 12, the product itself 16 (RT - 1) + 9
    constexpr int NSTEPS = 16 * (RT - 1) + 9 + 11 + 2 + PAIR_KB + 1;
    pair_ctx<ACTK, RT> C(S, cd, y, hA);
    C.cc = cc;
    C.c1 = c1;
    C.c2 = S.A->c2;
    C.scale = S.A->scale;
    if constexpr ((ACTK & DHQ_SPLIT_RN) != 0) asm volatile("" : "+v"(C.scale));
    C.ex = C.ey = C.et = 0.f;
    C.layer = layer;
    C.bias = reinterpret_cast<const float4 *>(S.lds + PAIR_BIAS + pair_bias_slot(layer) * 2048) + S.role * 64 + h;
    pair_enter_chunk(S, cc);
    {
        const dhq_v4i *src = reinterpret_cast<const dhq_v4i *>(S.lds + 2 * PAIR_BUF + S.grp * 16384) + S.lane;
#pragma unroll
        for (int T = 0; T < PAIR_KB; ++T) cd[T] = src[T * 64];
    }
    C.bufs[0] = S.lds + (cc & 1) * PAIR_BUF + S.role * 16384;
    C.bufs[1] = S.lds + ((cc + 1) & 1) * PAIR_BUF + S.role * 16384;
#pragma unroll
    for (int m = 0; m < PAIR_PF; ++m) C.fr[m % (PAIR_PF + 1)] = reinterpret_cast<const dhq_v4i *>(C.bufs[0])[m * 64 + S.lane];
    pair_steps<ACTK, RT>(C, std::make_integer_sequence<int, NSTEPS + PAIR_PF>{});
    cc += RT;
}

// The input layer (fan-in <= 4: one k block, one chunk with all sixteen tiles): step G issues the
// MFMA of tile G and the four H_32 products of tile G - 1, then drains tile G.
template <int G, int ACTK, int RT>
__device__ __forceinline__ void pair_step0(pair_ctx<ACTK, RT> &C, int h)
{
    constexpr int PF = PAIR_PF;
    if constexpr (G + PF < RT) C.fr[(G + PF) % (PF + 1)] = reinterpret_cast<const dhq_v4i *>(C.bufs[0])[(G + PF) * 64 + C.S.lane];
    if constexpr (G == 0) pair_copy_slot<0>(C.S);
    if constexpr (G == 1) pair_copy_slot<1>(C.S);
    if constexpr (G == 2) pair_copy_slot<2>(C.S);
    if constexpr (G == 3) pair_copy_slot<3>(C.S);
    if constexpr (G == 4) pair_copy_bias(C.S, 1);
    if constexpr (G < RT) {
#pragma unroll
        for (int v = 0; v < 16; ++v) C.acc[0][v] = 0;
        C.acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(C.fr[G % (PF + 1)], C.cd[0], C.acc[0], 0, 0, 0);
    }
    if constexpr (G >= 1 && G <= RT) {
        pair_h32<G - 1, 0>(C);
        pair_h32<G - 1, 1>(C);
        pair_h32<G - 1, 2>(C);
        pair_h32<G - 1, 3>(C);
    }
    if constexpr (G >= 2 && G - 2 < PAIR_EARLY) pair_send<G - 2>(C);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (G < RT) {
        float x[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = (float)C.acc[0][v];
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = __builtin_fmaf(x[v], C.c1, pair_comp(C.bq0[v >> 2], v & 3));
        if constexpr (DHQ_KIND(ACTK) == DHQ_ACT_KIND_WAVELET_COMPLEX) {
#pragma unroll
            for (int d = 0; d < 8; ++d)
                dhq_activate_pair_rev<false>(x[2 * d], x[2 * d + 1], C.c2, x[2 * d], x[2 * d + 1], hm_scaled<ACTK>(1.f, C.scale));
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = hm_scaled<ACTK>(dhq_activate_rev(x[v], dhq_act{DHQ_KIND(ACTK), C.c2}), C.scale);
        }
#pragma unroll
        for (int d = 0; d < 8; ++d) hm_split_pair<ACTK>(x[2 * d], x[2 * d + 1], C.hp[G & 1][d], C.lp[G & 1][d]);
    }
    if constexpr (G + 1 < RT) {
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) C.bq0[gg] = C.bias[((G + 1) * 4 + gg) * 2];
    }
    __builtin_amdgcn_sched_barrier(0);
}
template <int ACTK, int RT, int... Gs>
__device__ __forceinline__ void pair_steps0(pair_ctx<ACTK, RT> &C, int h, std::integer_sequence<int, Gs...>)
{
    (pair_step0<Gs>(C, h), ...);
}

template <int ACTK, int RT = PAIR_NT>
__device__ __forceinline__ void pair_input_layer(pair_stream &S, int &cc, float c1, dhq_v4i (&cd)[PAIR_KB], dhq_v16f (&y)[PAIR_NT],
                                                 const dhq_v4i (&hA)[2], int h)
{
    pair_ctx<ACTK, RT> C(S, cd, y, hA);
    C.cc = cc;
    C.c1 = c1;
    C.c2 = S.A->c2;
    C.scale = S.A->scale;
    if constexpr ((ACTK & DHQ_SPLIT_RN) != 0) asm volatile("" : "+v"(C.scale));
    C.layer = 0;
    C.bias = reinterpret_cast<const float4 *>(S.lds + PAIR_BIAS + pair_bias_slot(0) * 2048) + S.role * 64 + h;
    pair_enter_chunk(S, cc);
    C.bufs[0] = S.lds + (cc & 1) * PAIR_BUF + S.role * 8192;  // fragments [tile 0..15], 1 KiB each
    C.bufs[1] = C.bufs[0];
#pragma unroll
    for (int m = 0; m < PAIR_PF; ++m) C.fr[m % (PAIR_PF + 1)] = reinterpret_cast<const dhq_v4i *>(C.bufs[0])[m * 64 + S.lane];
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) C.bq0[gg] = C.bias[gg * 2];
    pair_steps0<ACTK, RT>(C, h, std::make_integer_sequence<int, RT + 1>{});
    cc += 1;
}

// What the partner parked for tile T, combined with the kept half of this wave's tile T:
// zl = own + partner (tile T of the stage over tile-index bit 3), zh = own - partner (tile T + 8;
// minus that for role 1, which owns T + 8).  PADDED: the two as they are, own in zl, the partner's in zh.
template <int T, int RT = PAIR_NT, bool PADDED = false>
__device__ __forceinline__ void pair_recv(const pair_stream &S, const dhq_v16f (&y)[PAIR_NT], float (&zl)[PAIR_NT][8],
                                          float (&zh)[PAIR_NT][8])
{
    if constexpr (T >= RT) return;  // zeros, which pair_transform leaves out
    const float4 *src = pair_x_slot(S, S.wave ^ 4, T);
    const float4 p0 = src[0], p1 = src[64];
    const float p[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        zl[T][i] = PADDED ? y[T][i] : y[T][i] + p[i];
        zh[T][i] = PADDED ? p[i] : y[T][i] - p[i];
    }
}

// The outgoing half of a tile that did not leave during the GEMM phase.
template <int T, int RT>
__device__ __forceinline__ void pair_send_late(const pair_stream &S, const dhq_v16f (&y)[PAIR_NT])
{
    if constexpr (T >= RT) return;
    float4 *d = pair_x_slot(S, S.wave, T);
    d[0] = make_float4(y[T][8], y[T][9], y[T][10], y[T][11]);
    d[64] = make_float4(y[T][12], y[T][13], y[T][14], y[T][15]);
}

__device__ __forceinline__ void pair_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
}

// The rest of the transform: on return zl[T][i] / zh[T][i] hold the un-normalised x^ of rotated features
// 32 T + 8 (i / 4 + 2 role) + 4 h + i % 4 and 256 + the same (zh of role 1 with its sign flipped), and
// the exchange area is free.
// PADDED networks, whose role r holds tiles 2 t + r (pair_tile): zl[t] is tile 2 t, zh[t] tile 2 t + 1.  The stages come in the same
// order over the tile index, bits 3, 0, 1, 2, so that a value's sum does not depend on who holds it: bit 3 is then bit 2 of
// t, and the stage between the two roles is the second.
template <bool AFTER_INPUT_LAYER, int RT = PAIR_NT, bool PADDED = false>
__device__ __forceinline__ void pair_transform(pair_stream &S, dhq_v16f (&y)[PAIR_NT], float (&zl)[PAIR_NT][8], float (&zh)[PAIR_NT][8])
{
    // the halves sent during the GEMM phase are in place: a hidden layer's last sends (step 16 * 3 + 12 + 29) precede its last
    // chunk's barrier (step 16 (RT - 1) - PAIR_PF) from seven tiles on, the input layer has none
    if constexpr (AFTER_INPUT_LAYER || 16 * (RT - 1) - PAIR_PF <= 16 * (PAIR_EARLY - 1) + 12 + 29) pair_barrier();
    pair_recv<0, RT, PADDED>(S, y, zl, zh);
    pair_recv<1, RT, PADDED>(S, y, zl, zh);
    pair_recv<2, RT, PADDED>(S, y, zl, zh);
    pair_recv<3, RT, PADDED>(S, y, zl, zh);
    pair_barrier();  // everyone has read them: the slots are free again
    pair_send_late<4, RT>(S, y);
    pair_send_late<5, RT>(S, y);
    pair_send_late<6, RT>(S, y);
    pair_send_late<7, RT>(S, y);
    pair_barrier();
    pair_recv<4, RT, PADDED>(S, y, zl, zh);
    pair_recv<5, RT, PADDED>(S, y, zl, zh);
    pair_recv<6, RT, PADDED>(S, y, zl, zh);
    pair_recv<7, RT, PADDED>(S, y, zl, zh);
    pair_barrier();  // the exchange area is free for the codes
    if constexpr (PADDED) {
        // a padding tile t | 4 is zero, so that tiles t and t | 4 are then the same, and so are the sums that the next stages make of
        // them, which the compiler takes once
        static_assert(RT >= 4, "tiles 0 .. 3 are written");
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = zl[t][i], b = zh[t][i];
                zl[t][i] = t + 4 < RT ? a + zl[t + 4][i] : a;
                zh[t][i] = t + 4 < RT ? b + zh[t + 4][i] : b;
                zl[t + 4][i] = t + 4 < RT ? a - zl[t + 4][i] : a;
                zh[t + 4][i] = t + 4 < RT ? b - zh[t + 4][i] : b;
            }
        }
#pragma unroll
        for (int t = 0; t < PAIR_NT; ++t) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = zl[t][i], b = zh[t][i];
                zl[t][i] = a + b;
                zh[t][i] = a - b;
            }
        }
    }
    // the other stages within each half
#pragma unroll
    for (int s = 1; s < (PADDED ? 4 : PAIR_NT); s <<= 1) {
#pragma unroll
        for (int t = 0; t < PAIR_NT; ++t) {
            if ((t & s) == 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float a = zl[t][i], b = zl[t | s][i];
                    zl[t][i] = a + b;
                    zl[t | s][i] = a - b;
                    const float a2 = zh[t][i], b2 = zh[t | s][i];
                    zh[t][i] = a2 + b2;
                    zh[t | s][i] = a2 - b2;
                }
            }
        }
    }
}

// The rest of the transform and the next layer's quantizer.  On return the exchange area holds,
// per coordinate group, the next layer's whole B operand ([k block][lane] x 16 B); it may be read
// after the next barrier.  xrow (test hook): where this lane's coordinate keeps its row of x^.
template <bool DUMP, bool AFTER_INPUT_LAYER = true, int RT = PAIR_NT, bool PADDED = false>
__device__ __forceinline__ void pair_transform_quant(pair_stream &S, dhq_v16f (&y)[PAIR_NT], float inv, int qlo, int qhi, int h,
                                                     float *xrow = nullptr, int *crow = nullptr)
{
    float zl[PAIR_NT][8], zh[PAIR_NT][8];
    pair_transform<AFTER_INPUT_LAYER, RT, PADDED>(S, y, zl, zh);
    const float inv_hi = S.role ? -inv : inv;
    if constexpr (DUMP) {
        // rotated feature of zl[T][i]: 32 T + 8 (i / 4 + 2 role) + 4 h + i % 4; zh: tile T + 8, sign as above
        const float sg = S.role ? -1.f : 1.f;
#pragma unroll
        for (int T = 0; T < PAIR_NT; ++T) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float *p = xrow + 32 * T + 8 * (q + 2 * S.role) + 4 * h;
                *reinterpret_cast<float4 *>(p) = make_float4(zl[T][4 * q], zl[T][4 * q + 1], zl[T][4 * q + 2], zl[T][4 * q + 3]);
                *reinterpret_cast<float4 *>(p + 256) =
                    make_float4(sg * zh[T][4 * q], sg * zh[T][4 * q + 1], sg * zh[T][4 * q + 2], sg * zh[T][4 * q + 3]);
            }
        }
    }
    // this wave's two dwords of every k block: bytes 8 role .. 8 role + 7 of the lane's 16
    unsigned char *dst = S.lds + 2 * PAIR_BUF + S.grp * 16384 + S.lane * 16 + S.role * 8;
#pragma unroll
    for (int T = 0; T < PAIR_NT; ++T) {
        const unsigned a0 = fused_quant4(zl[T][0], zl[T][1], zl[T][2], zl[T][3], inv, qlo, qhi);
        const unsigned a1 = fused_quant4(zl[T][4], zl[T][5], zl[T][6], zl[T][7], inv, qlo, qhi);
        const unsigned b0 = fused_quant4(zh[T][0], zh[T][1], zh[T][2], zh[T][3], inv_hi, qlo, qhi);
        const unsigned b1 = fused_quant4(zh[T][4], zh[T][5], zh[T][6], zh[T][7], inv_hi, qlo, qhi);
        *reinterpret_cast<uint2 *>(dst + T * 1024) = make_uint2(a0, a1);
        *reinterpret_cast<uint2 *>(dst + (T + 8) * 1024) = make_uint2(b0, b1);
        if constexpr (DUMP) {
            int *c = crow + 8 * T + 2 * (2 * S.role) + h;  // dwords of 4 codes: feature / 4
            c[0] = (int)a0; c[2] = (int)a1; c[64] = (int)b0; c[66] = (int)b1;
        }
    }
}

__device__ __forceinline__ void pair_h32_operand(int c, int h, int role, dhq_v4i (&hA)[2])
{
    fused_h32_operand(c ^ (role << 4), h, hA);
}

__device__ __forceinline__ void pair_stream_init(pair_stream &S, const pair_args *A, unsigned char *lds, int wave, int lane)
{
    S.A = A;
    S.lds = lds;
    S.wave = __builtin_amdgcn_readfirstlane(wave);
    S.lane = lane;
    S.role = S.wave >> 2;
    S.grp = S.wave & 3;
    S.cp_src = A->blob;
    S.cp_dst = pair_lds_addr(lds);
    S.voff = (unsigned)lane * 16;
}

// Copies chunk j into buffer `buf` right now (the first chunk of a kernel has nobody to copy it in the background).
__device__ __forceinline__ void pair_copy_now(const pair_stream &S, int j, int buf)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int q = S.wave + 8 * i;
        reinterpret_cast<dhq_v4i *>(S.lds + buf * PAIR_BUF)[q * 64 + S.lane] =
            reinterpret_cast<const dhq_v4i *>(S.A->blob + (size_t)j * PAIR_BUF)[q * 64 + S.lane];
    }
}

template <int ACTK, int RT>
__global__ __launch_bounds__(PAIR_THREADS) void dhq_fused_pair_kernel(const pair_args A)
{
    constexpr bool PADDED = (ACTK & DHQ_SPLIT_RN) != 0;
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int L = A.n_layers;
    const int64_t n_tiles = (A.n + PAIR_TILE - 1) / PAIR_TILE;
    if ((int64_t)blockIdx.x >= n_tiles) return;
    const int my_tiles = (int)((n_tiles - 1 - blockIdx.x) / gridDim.x) + 1;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;

    pair_stream S;
    pair_stream_init(S, &A, lds, wave, lane);
    int cc = 0;
    pair_copy_now(S, 0, 0);
    pair_copy_bias(S, 0);

    dhq_v4i hA[2];
    pair_h32_operand(c, h, S.role, hA);

    for (int it = 0; it < my_tiles; ++it) {
        const int64_t tile = (int64_t)blockIdx.x + (int64_t)it * gridDim.x;
        // the codes of a layer's input: the input layer uses k block 0 only (and of it only k positions 0..3, the
        // rest of its fragments being zero), every hidden layer reads all sixteen from the exchange area first
        dhq_v4i cd[PAIR_KB];
#pragma unroll
        for (int kb = 0; kb < PAIR_KB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
        {
            // (the lane's coordinate from the thread index afresh in every pass, like the output layer below: a
            // loop-invariant per-lane address would be carried through all layers in registers it spills)
            unsigned tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int64_t ci = tile * PAIR_TILE + S.grp * 32 + (tid & 31);
            const int64_t cl = ci < A.n ? ci : A.n - 1;  // lanes past the end repeat the last coordinate and store nothing
            cd[0][0] = fused_input_codes(A.coords, cl, A.k0, A.k0p, A.inv_in[0], A.qmax);
        }

        dhq_v16f y[PAIR_NT];
        pair_input_layer<ACTK, RT>(S, cc, A.c1[0], cd, y, hA, h);
        pair_transform_quant<false, true, RT, PADDED>(S, y, A.inv_in[1], qlo, qhi, h);
        for (int l = 1; l < L - 1; ++l) {
            pair_hidden<ACTK, RT>(S, cc, l, A.c1[l], cd, y, hA, h);
            pair_transform_quant<false, false, RT, PADDED>(S, y, A.inv_in[l + 1], qlo, qhi, h);
        }

        // output layer: one zero-padded M tile, no activation; role 0 computes it while all waves
        // copy in the next pass's first chunk
        {
            pair_enter_chunk(S, cc);
            const unsigned char *buf = lds + (cc & 1) * PAIR_BUF;
            pair_copy_slot<0>(S); pair_copy_slot<1>(S); pair_copy_slot<2>(S); pair_copy_slot<3>(S);
            pair_copy_bias(S, 0);
            if (S.role == 0) {
                // The coordinate index, the lane's place and its lane half are worked out again from the thread
                // index (through an empty asm, so that the compiler cannot tell they are the values from the
                // top of the pass): kept alive across all layers they would be spilled to scratch memory.
                unsigned tid = threadIdx.x;
                asm volatile("" : "+v"(tid));
                const int lane = tid & 63, h = (tid >> 5) & 1;
                const int64_t ci = tile * PAIR_TILE + S.grp * 32 + (tid & 31);
                const bool valid = ci < A.n;
                const dhq_v4i *src = reinterpret_cast<const dhq_v4i *>(lds + 2 * PAIR_BUF + S.grp * 16384) + lane;
                const dhq_v4i *wA = reinterpret_cast<const dhq_v4i *>(buf);
                dhq_v16i acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
                for (int kb = 0; kb < PAIR_KB; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wA[kb * 64 + lane], src[kb * 64], acc, 0, 0, 0);
                const float *wB = reinterpret_cast<const float *>(lds + PAIR_BIAS + pair_bias_slot(L - 1) * 2048);
                const float c1 = A.c1[L - 1];
                if (valid) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                        if (row < A.m_out) A.out[ci * A.m_out + row] = __builtin_fmaf((float)acc[v], c1, wB[((v >> 2) * 2 + h) * 4 + (v & 3)]);
                    }
                }
            }
            cc += 1;
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// ---- two-sided rotation (Eq. 4 with both factors) at this width -------------------------------
// The layer's output comes out of the GEMM in the rotated basis and is multiplied by H_512 once more, exactly, in
// int32.  That product is linear in the weights: z = (q W'^T) H = q (H W')^T, so the kernel multiplies by U = H W'
// instead and has no un-rotation at all.  An entry of U takes up to 17 bits (a sum of 512 codes); it travels as two int8
// digits, u = 256 u1 + u0, where every |u| <= 32639 (the sum of 512 bell-shaped codes stays below about a tenth of that;
// weights with larger entries keep the layer-by-layer path): acc = q u1, acc <<= 8, acc += q u0 in the same
// accumulators, wrapping, the same int32 as before.  That is twice the MFMAs and weight bytes of the one-sided layer
// against nine integer butterfly stages and an exchange between the waves.
//
// The forward transform gives the bits of the layer-by-layer kernels: fp32 butterflies in their order of stages, feature
// bits 0, 1, 6, 7, 8, 2, 3, 4, 5.  Only the order of the stages decides the bits, not where a value lives, so the nine bits
// of the output feature are dealt to the hardware in that order (the rows of U are permuted offline):
//   accumulator v bits 0..3 <- feature bits 0, 1, 6, 7   the stages inside a tile, one butterfly per GEMM step
//   tile T bits 0..2        <- 8, 2, 3                   register stages after the GEMM
//   lane half               <- 4                         a lane swap, which trades places with v bit 0
//   role                    <- 5                         the exchange between the two waves of a pair, as above
// Role 1 has v bit 3 the other way round (feature bit 7 = v bit 3 xor role), so that both roles keep registers 0..7 and send
// 8..15; the stage over that bit is a multiply-add by +-1, which rounds like the addition.
//
// Six hidden layers of 512, 262 144 rows: 2 402 us layer by layer (per layer a GEMM and an un-rotation kernel, 5 KiB of
// traffic per row), 800 us here; 117 -> 85 us on 1 000 rows.
static inline int pair2_feature(int role, int T, int v, int h)
{
    return (v & 3) | ((T >> 1) & 1) << 2 | ((T >> 2) & 1) << 3 | h << 4 | role << 5 | ((v >> 2) & 1) << 6 | ((v >> 3) ^ role) << 7 | (T & 1) << 8;
}
// Rotated feature of byte jj of lane half u in k block kb of the codes a layer leaves: dwords 2 role, 2 role + 1 are the kept
// registers of tile kb % 8, whose bit 0 and the lane half have traded places; kb / 8 is the role bit after the exchange.
static inline int pair2_code_feature(int kb, int u, int jj)
{
    const int T = kb & 7, role = jj >> 3, i = jj & 7;
    return u | ((i >> 1) & 1) << 1 | ((T >> 1) & 1) << 2 | ((T >> 2) & 1) << 3 | (i & 1) << 4 | (kb >> 3) << 5 | (i >> 2) << 6 | role << 7 | (T & 1) << 8;
}

template <int ACTK>
struct pair2_ctx {
    pair_stream &S;
    dhq_v4i (&cd)[PAIR_KB];
    dhq_v16f (&y)[PAIR_NT];  // activations, then the transform inside the tiles
    const unsigned char *bufs[2];
    const float4 *bias;
    int cc, layer;
    float c1, c2, sgn;       // sgn: +1 for role 0, -1 for role 1
    dhq_v4i fr[PAIR_PF + 1];
    float4 bq[2];
    dhq_v16i acc[2];
    float ey;
    __device__ __forceinline__ pair2_ctx(pair_stream &S_, dhq_v4i (&cd_)[PAIR_KB], dhq_v16f (&y_)[PAIR_NT]) : S(S_), cd(cd_), y(y_) {}
};

// Butterfly B (stage B / 8) inside a tile.
template <int B>
__device__ __forceinline__ void pair2_butterfly(dhq_v16f &x, float sgn)
{
// the wavelet ends in a product, which must not melt into the first stage's additions
#pragma clang fp contract(off)
    constexpr int st = B / 8, j = B % 8;
    constexpr int v0 = ((j >> st) << (st + 1)) | (j & ((1 << st) - 1)), v1 = v0 | (1 << st);
    const float a = x[v0], b = x[v1];
    if constexpr (st < 3) {
        x[v0] = a + b;
        x[v1] = a - b;
    } else {
        x[v0] = __builtin_fmaf(a, sgn, b);   // role 0: a + b; role 1 holds them the other way round: b - a
        x[v1] = __builtin_fmaf(b, -sgn, a);  // role 0: a - b; role 1: a + b
    }
}

// One step of a hidden layer: the MFMA of step G (tile G / 32, digit plane (G / 16) % 2, high one first, k block G % 16), half
// of the epilogue of one value of the tile before, one butterfly of the tile before that.
template <int G, int ACTK>
__device__ __forceinline__ void pair2_step(pair2_ctx<ACTK> &C)
{
    constexpr int NM = PAIR_NT * 2 * PAIR_KB, PF = PAIR_PF;
    if constexpr (G >= 0 && G + PF < NM) {
        constexpr int pf = G + PF;
        if constexpr (pf % PAIR_KB == 0) pair_enter_chunk(C.S, C.cc + pf / PAIR_KB);
        C.fr[pf % (PF + 1)] = reinterpret_cast<const dhq_v4i *>(C.bufs[(pf / PAIR_KB) & 1])[(pf % PAIR_KB) * 64 + C.S.lane];
    }
    if constexpr (G + PF >= 0 && G + PF < NM) {
        constexpr int rel = (G + PF) % PAIR_KB;
        if constexpr (rel == 1) pair_copy_slot<0>(C.S);
        if constexpr (rel == 3) pair_copy_slot<1>(C.S);
        if constexpr (rel == 5) pair_copy_slot<2>(C.S);
        if constexpr (rel == 7) pair_copy_slot<3>(C.S);
    }
    if constexpr (G == 9) pair_copy_bias(C.S, C.layer + 1);
    if constexpr (G >= 0 && G < NM) {
        constexpr int t = G / 32, r = G % 32;
        if constexpr (r == 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) C.acc[t & 1][v] = 0;
        }
        if constexpr (r == 16) {
#pragma unroll
            for (int v = 0; v < 16; ++v) C.acc[t & 1][v] = (int)((unsigned)C.acc[t & 1][v] << 8);
        }
        C.acc[t & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(C.fr[G % (PF + 1)], C.cd[G % PAIR_KB], C.acc[t & 1], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr int E = G - 32, F = G - 64;
    if constexpr (F >= 0 && F < NM) pair2_butterfly<F % 32>(C.y[F / 32], C.sgn);
    if constexpr (E >= 0 && E < NM) {
        constexpr int td = E / 32, v = (E % 32) / 2;
        if constexpr ((E & 1) == 0) C.ey = __builtin_fmaf((float)C.acc[td & 1][v], C.c1, pair_comp(C.bq[(E / 8) & 1], v & 3));
        else C.y[td][v] = dhq_activate_rev_any(C.ey, dhq_act{DHQ_KIND(ACTK), C.c2});
    }
    if constexpr (E + 8 >= 0 && (E + 8) % 8 == 0 && E + 8 < NM) {
        constexpr int ge = (E + 8) / 8;  // biases of values 4 (ge % 4) .. + 3 of tile ge / 4; the slot's last value is done
        C.bq[ge & 1] = C.bias[ge * 2];
    }
    __builtin_amdgcn_sched_barrier(0);
}
template <int ACTK, int... Gs>
__device__ __forceinline__ void pair2_steps(pair2_ctx<ACTK> &C, std::integer_sequence<int, Gs...>)
{
    (pair2_step<Gs - PAIR_PF>(C), ...);
}

template <int ACTK>
__device__ __forceinline__ void pair2_hidden(pair_stream &S, int &cc, int layer, float c1, dhq_v4i (&cd)[PAIR_KB],
                                             dhq_v16f (&y)[PAIR_NT], int h)
{
    pair2_ctx<ACTK> C(S, cd, y);
    C.cc = cc;
    C.c1 = c1;
    C.c2 = S.A->c2;
    C.sgn = S.role ? -1.f : 1.f;
    C.ey = 0.f;
    C.layer = layer;
    C.bias = reinterpret_cast<const float4 *>(S.lds + PAIR_BIAS + pair_bias_slot(layer) * 2048) + S.role * 64 + h;
    pair_enter_chunk(S, cc);
    {
        const dhq_v4i *src = reinterpret_cast<const dhq_v4i *>(S.lds + 2 * PAIR_BUF + S.grp * 16384) + S.lane;
#pragma unroll
        for (int T = 0; T < PAIR_KB; ++T) cd[T] = src[T * 64];
    }
    C.bufs[0] = S.lds + (cc & 1) * PAIR_BUF + S.role * 16384;
    C.bufs[1] = S.lds + ((cc + 1) & 1) * PAIR_BUF + S.role * 16384;
#pragma unroll
    for (int m = 0; m < PAIR_PF; ++m) C.fr[m % (PAIR_PF + 1)] = reinterpret_cast<const dhq_v4i *>(C.bufs[0])[m * 64 + S.lane];
    pair2_steps<ACTK>(C, std::make_integer_sequence<int, PAIR_PF + PAIR_NT * 32 + 64>{});
    cc += 2 * PAIR_NT;
}

// The input layer (one k block: fan-in <= 4, or <= 32 with DHQ_CODES_IN): one chunk, per role [tile][digit plane] fragments.
template <int T, int ACTK>
__device__ __forceinline__ void pair2_input_tile(pair2_ctx<ACTK> &C)
{
    const dhq_v4i *fr = reinterpret_cast<const dhq_v4i *>(C.bufs[0]) + T * 128 + C.S.lane;
    const dhq_v4i f1 = fr[0], f0 = fr[64];
    float4 bq[4];
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) bq[gg] = C.bias[(T * 4 + gg) * 2];
    if constexpr (T == 0) pair_copy_slot<0>(C.S);
    if constexpr (T == 1) pair_copy_slot<1>(C.S);
    if constexpr (T == 2) pair_copy_slot<2>(C.S);
    if constexpr (T == 3) pair_copy_slot<3>(C.S);
    if constexpr (T == 4) pair_copy_bias(C.S, 1);
    dhq_v16i acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0;
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1, C.cd[0], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = (int)((unsigned)acc[v] << 8);
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(f0, C.cd[0], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v)
        C.y[T][v] = dhq_activate_rev_any(__builtin_fmaf((float)acc[v], C.c1, pair_comp(bq[v >> 2], v & 3)), dhq_act{DHQ_KIND(ACTK), C.c2});
}
template <int ACTK, int... Ts>
__device__ __forceinline__ void pair2_input_tiles(pair2_ctx<ACTK> &C, std::integer_sequence<int, Ts...>)
{
    (pair2_input_tile<Ts>(C), ...);
}
template <int T, int ACTK, int... Bs>
__device__ __forceinline__ void pair2_tile_butterflies(pair2_ctx<ACTK> &C, std::integer_sequence<int, Bs...>)
{
    (pair2_butterfly<Bs>(C.y[T], C.sgn), ...);
}
template <int ACTK, int... Ts>
__device__ __forceinline__ void pair2_input_butterflies(pair2_ctx<ACTK> &C, std::integer_sequence<int, Ts...>)
{
    (pair2_tile_butterflies<Ts>(C, std::make_integer_sequence<int, 32>{}), ...);
}

template <int ACTK>
__device__ __forceinline__ void pair2_input_layer(pair_stream &S, int &cc, float c1, dhq_v4i (&cd)[PAIR_KB], dhq_v16f (&y)[PAIR_NT], int h)
{
    pair2_ctx<ACTK> C(S, cd, y);
    C.cc = cc;
    C.c1 = c1;
    C.c2 = S.A->c2;
    C.sgn = S.role ? -1.f : 1.f;
    C.layer = 0;
    C.bias = reinterpret_cast<const float4 *>(S.lds + PAIR_BIAS + pair_bias_slot(0) * 2048) + S.role * 64 + h;
    pair_enter_chunk(S, cc);
    C.bufs[0] = C.bufs[1] = S.lds + (cc & 1) * PAIR_BUF + S.role * 16384;
    pair2_input_tiles<ACTK>(C, std::make_integer_sequence<int, PAIR_NT>{});
    pair2_input_butterflies<ACTK>(C, std::make_integer_sequence<int, PAIR_NT>{});
    cc += 1;
}

// Tiles T0 .. T0 + 3: outgoing registers to the exchange area, then the partner's.
template <int T0>
__device__ __forceinline__ void pair2_exchange(pair_stream &S, const dhq_v16f (&y)[PAIR_NT], float (&zl)[PAIR_NT][8], float (&zh)[PAIR_NT][8])
{
#pragma unroll
    for (int T = T0; T < T0 + 4; ++T) {
        float4 *d = pair_x_slot(S, S.wave, T);
        d[0] = make_float4(y[T][8], y[T][9], y[T][10], y[T][11]);
        d[64] = make_float4(y[T][12], y[T][13], y[T][14], y[T][15]);
    }
    pair_barrier();
    pair_recv<T0>(S, y, zl, zh);
    pair_recv<T0 + 1>(S, y, zl, zh);
    pair_recv<T0 + 2>(S, y, zl, zh);
    pair_recv<T0 + 3>(S, y, zl, zh);
    pair_barrier();  // everyone has read them: the slots are free again
}

// The stages over tile bits and lane half, the exchange, the quantizer; the codes go to the exchange area, which may be read
// after the next barrier.  (On entry nobody reads the exchange area any more: every wave took its codes before the barriers
// of this layer's later chunks, or before the input layer's chunk.)
__device__ __forceinline__ void pair2_transform_quant(pair_stream &S, dhq_v16f (&y)[PAIR_NT], float inv, int qlo, int qhi)
{
#pragma unroll
    for (int s = 1; s < PAIR_NT; s <<= 1) {
#pragma unroll
        for (int T = 0; T < PAIR_NT; ++T) {
            if ((T & s) == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float a = y[T][v], b = y[T | s][v];
                    y[T][v] = a + b;
                    y[T | s][v] = a - b;
                }
            }
        }
    }
#pragma unroll
    for (int T = 0; T < PAIR_NT; ++T) {
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            // the upper lanes of v for the lower lanes of v + 1: both halves of a pair then sit in one lane
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(y[T][v]), __float_as_uint(y[T][v + 1]), false, false);
            const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
            y[T][v] = a + b;
            y[T][v + 1] = a - b;
        }
    }
    float zl[PAIR_NT][8], zh[PAIR_NT][8];
    pair2_exchange<0>(S, y, zl, zh);
    pair2_exchange<4>(S, y, zl, zh);
    const float inv_hi = S.role ? -inv : inv;  // role 1's difference is minus the true one
    unsigned char *dst = S.lds + 2 * PAIR_BUF + S.grp * 16384 + S.lane * 16 + S.role * 8;
#pragma unroll
    for (int T = 0; T < PAIR_NT; ++T) {
        const unsigned a0 = fused_quant4(zl[T][0], zl[T][1], zl[T][2], zl[T][3], inv, qlo, qhi);
        const unsigned a1 = fused_quant4(zl[T][4], zl[T][5], zl[T][6], zl[T][7], inv, qlo, qhi);
        const unsigned b0 = fused_quant4(zh[T][0], zh[T][1], zh[T][2], zh[T][3], inv_hi, qlo, qhi);
        const unsigned b1 = fused_quant4(zh[T][4], zh[T][5], zh[T][6], zh[T][7], inv_hi, qlo, qhi);
        *reinterpret_cast<uint2 *>(dst + T * 1024) = make_uint2(a0, a1);
        *reinterpret_cast<uint2 *>(dst + (T + 8) * 1024) = make_uint2(b0, b1);
    }
}

template <int ACTK>
__global__ __launch_bounds__(PAIR_THREADS) void dhq_fused_pair2_kernel(const pair_args A)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = lane >> 5;
    const int L = A.n_layers;
    const int64_t n_tiles = (A.n + PAIR_TILE - 1) / PAIR_TILE;
    if ((int64_t)blockIdx.x >= n_tiles) return;
    const int my_tiles = (int)((n_tiles - 1 - blockIdx.x) / gridDim.x) + 1;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;

    pair_stream S;
    pair_stream_init(S, &A, lds, wave, lane);
    int cc = 0;
    pair_copy_now(S, 0, 0);
    pair_copy_bias(S, 0);

    for (int it = 0; it < my_tiles; ++it) {
        const int64_t tile = (int64_t)blockIdx.x + (int64_t)it * gridDim.x;
        dhq_v4i cd[PAIR_KB];
#pragma unroll
        for (int kb = 0; kb < PAIR_KB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
        {
            unsigned tid = threadIdx.x;  // (worked out afresh in every pass, see dhq_fused_pair_kernel)
            asm volatile("" : "+v"(tid));
            const int64_t ci = tile * PAIR_TILE + S.grp * 32 + (tid & 31);
            const int64_t cl = ci < A.n ? ci : A.n - 1;  // lanes past the end repeat the last coordinate and store nothing
            if constexpr ((ACTK & DHQ_CODES_IN) != 0) {
                dhq_v4i first[1] = {dhq_v4i{0, 0, 0, 0}};
                fused_load_codes(A.codes0, cl, A.k0p, (int)(tid >> 5) & 1, first);
                cd[0] = first[0];
            } else {
                cd[0][0] = fused_input_codes(A.coords, cl, A.k0, A.k0p, A.inv_in[0], A.qmax);
            }
        }
        dhq_v16f y[PAIR_NT];
        pair2_input_layer<ACTK>(S, cc, A.c1[0], cd, y, h);
        pair2_transform_quant(S, y, A.inv_in[1], qlo, qhi);
        for (int l = 1; l < L - 1; ++l) {
            pair2_hidden<ACTK>(S, cc, l, A.c1[l], cd, y, h);
            pair2_transform_quant(S, y, A.inv_in[l + 1], qlo, qhi);
        }
        // output layer: one zero-padded tile in two digit planes
        {
            pair_enter_chunk(S, cc);
            const unsigned char *buf = lds + (cc & 1) * PAIR_BUF;
            pair_copy_slot<0>(S); pair_copy_slot<1>(S); pair_copy_slot<2>(S); pair_copy_slot<3>(S);
            pair_copy_bias(S, 0);
            if (S.role == 0) {
                unsigned tid = threadIdx.x;
                asm volatile("" : "+v"(tid));
                const int lane = tid & 63, h = (tid >> 5) & 1;
                const int64_t ci = tile * PAIR_TILE + S.grp * 32 + (tid & 31);
                const bool valid = ci < A.n;
                const dhq_v4i *src = reinterpret_cast<const dhq_v4i *>(lds + 2 * PAIR_BUF + S.grp * 16384) + lane;
                const dhq_v4i *wA = reinterpret_cast<const dhq_v4i *>(buf);
                dhq_v16i acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
                for (int kb = 0; kb < PAIR_KB; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wA[kb * 64 + lane], src[kb * 64], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = (int)((unsigned)acc[v] << 8);
#pragma unroll
                for (int kb = 0; kb < PAIR_KB; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wA[1024 + kb * 64 + lane], src[kb * 64], acc, 0, 0, 0);
                const float *wB = reinterpret_cast<const float *>(lds + PAIR_BIAS + pair_bias_slot(L - 1) * 2048);
                const float c1 = A.c1[L - 1];
                if (valid) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                        if (row < A.m_out) A.out[ci * A.m_out + row] = __builtin_fmaf((float)acc[v], c1, wB[((v >> 2) * 2 + h) * 4 + (v & 3)]);
                    }
                }
            }
            cc += 1;
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// ---- one layer per launch: the dynamic quantization module (Sec. 3.3) at this width -----------
// With scales measured on line a layer's quantizer needs max |x^| over the whole batch before it
// can emit a code, so the whole-network kernel is cut at exactly that point, as
// dhq_fused_layer_kernel cuts the narrower one: a launch folds the per-workgroup maxima its
// predecessor left into this layer's constants (every workgroup for itself), quantizes its input
// with them, runs the layer with the code of the kernel above and writes the un-normalised
// transform x^ of its output (fp32) plus the workgroup's max |x^|.  x^ crosses device memory in the
// waves' register order: [128-coordinate tile][wave][q = 4 T + {zl 0..3, zl 4..7, zh 0..3, zh 4..7}][lane]
// x 16 B, every access of a wave 1 KiB contiguous; a wave reads back exactly what the wave in its
// place wrote (zh of role 1 with its sign flipped, which the negated multiplier undoes).
//   MODE 0  input layer: coordinates in, x^ out        MODE 1  hidden layer: x^ in, x^ out
//   MODE 2  output layer: x^ in, signal values out
struct pair_largs {
    pair_args w;               // n_chunks / chunk_base: this layer's chunks; c1 and inv_in are not used
    const float4 *xin;         // MODE 1, 2
    float4 *xout;              // MODE 0, 1
    const float *partial_in;   // max |x^| of this layer's input, one float per workgroup of the launch before
    int partial_count;
    int kp;                    // length of this layer's rotated input
    int layer;
    double c1_over_sa;         // epilogue multiplier divided by the activation scale
    float *dyn;                // this layer's {1 / (s_a sqrt(Kp)), epilogue multiplier, s_a}: written by workgroup 0
    float *partial;            // MODE 0, 1: max |x^| of the output per workgroup (not the buffer partial_in points to)
};

template <int MODE, int ACTK>
__global__ __launch_bounds__(PAIR_THREADS) void dhq_fused_pair_layer_kernel(const pair_largs D)
{
    const pair_args &A = D.w;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ float red_in[PAIR_WAVES], red[PAIR_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int64_t n_tiles = (A.n + PAIR_TILE - 1) / PAIR_TILE;  // the grid has at most that many workgroups
    const int my_tiles = (int)((n_tiles - 1 - blockIdx.x) / gridDim.x) + 1;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;

    pair_stream S;
    pair_stream_init(S, &A, lds, wave, lane);
    int cc = 0;
    pair_copy_now(S, A.chunk_base, 0);
    pair_copy_bias(S, D.layer);
    dhq_v4i hA[2];
    pair_h32_operand(c, h, S.role, hA);

    // this layer's constants from the maxima of its input
    float inv, c1, s_a;
    {
        float mi = 0.f;
        for (int i = threadIdx.x; i < D.partial_count; i += PAIR_THREADS) mi = fmaxf(mi, D.partial_in[i]);
#pragma unroll
        for (int m = 1; m < 64; m *= 2) mi = fmaxf(mi, __shfl_xor(mi, m, 64));
        if (lane == 0) red_in[wave] = mi;
        __syncthreads();
        mi = red_in[0];
#pragma unroll
        for (int w = 1; w < PAIR_WAVES; ++w) mi = fmaxf(mi, red_in[w]);
        dhq_dyn_constants(mi, D.kp, A.qmax, D.c1_over_sa, inv, c1, s_a);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            D.dyn[0] = inv; D.dyn[1] = c1; D.dyn[2] = s_a;
        }
    }
    float mx = 0.f;
    for (int it = 0; it < my_tiles; ++it) {
        const int64_t tile = (int64_t)blockIdx.x + (int64_t)it * gridDim.x;
        const size_t slot = ((size_t)tile * PAIR_WAVES + S.wave) * (4 * PAIR_NT) * 64 + lane;
        dhq_v4i cd[PAIR_KB];
#pragma unroll
        for (int kb = 0; kb < PAIR_KB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
        if constexpr (MODE == 0) {
            const int64_t ci = tile * PAIR_TILE + S.grp * 32 + c;
            const int64_t cl = ci < A.n ? ci : A.n - 1;  // lanes past the end repeat the last coordinate: no effect on the maximum
            cd[0][0] = fused_input_codes(A.coords, cl, A.k0, A.k0p, inv, A.qmax);
        } else {
            // the output layer's role-0 waves may still be reading the previous tile's codes
            if constexpr (MODE == 2) pair_barrier();
            // this wave's 128 values of the layer's input: quantized, its two dwords of every k block to the exchange
            // area, where pair_transform_quant puts them in the whole-network kernel
            const float inv_hi = S.role ? -inv : inv;
            unsigned char *dst = lds + 2 * PAIR_BUF + S.grp * 16384 + lane * 16 + S.role * 8;
#pragma unroll
            for (int T = 0; T < PAIR_NT; ++T) {
                const float4 l0 = D.xin[slot + (size_t)(4 * T) * 64], l1 = D.xin[slot + (size_t)(4 * T + 1) * 64];
                const float4 h0 = D.xin[slot + (size_t)(4 * T + 2) * 64], h1 = D.xin[slot + (size_t)(4 * T + 3) * 64];
                const unsigned a0 = fused_quant4(l0.x, l0.y, l0.z, l0.w, inv, qlo, qhi);
                const unsigned a1 = fused_quant4(l1.x, l1.y, l1.z, l1.w, inv, qlo, qhi);
                const unsigned b0 = fused_quant4(h0.x, h0.y, h0.z, h0.w, inv_hi, qlo, qhi);
                const unsigned b1 = fused_quant4(h1.x, h1.y, h1.z, h1.w, inv_hi, qlo, qhi);
                *reinterpret_cast<uint2 *>(dst + T * 1024) = make_uint2(a0, a1);
                *reinterpret_cast<uint2 *>(dst + (T + 8) * 1024) = make_uint2(b0, b1);
            }
        }
        if constexpr (MODE == 2) {
            // one zero-padded M tile, no activation: role 0 computes it while all waves copy the chunk in again
            pair_enter_chunk(S, cc);
            const unsigned char *buf = lds + (cc & 1) * PAIR_BUF;
            pair_copy_slot<0>(S); pair_copy_slot<1>(S); pair_copy_slot<2>(S); pair_copy_slot<3>(S);
            if (S.role == 0) {
                const int64_t ci = tile * PAIR_TILE + S.grp * 32 + c;
                const dhq_v4i *src = reinterpret_cast<const dhq_v4i *>(lds + 2 * PAIR_BUF + S.grp * 16384) + lane;
                const dhq_v4i *wA = reinterpret_cast<const dhq_v4i *>(buf);
                dhq_v16i acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0;
#pragma unroll
                for (int kb = 0; kb < PAIR_KB; ++kb) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wA[kb * 64 + lane], src[kb * 64], acc, 0, 0, 0);
                const float *wB = reinterpret_cast<const float *>(lds + PAIR_BIAS + pair_bias_slot(D.layer) * 2048);
                if (ci < A.n) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = 8 * (v >> 2) + 4 * h + (v & 3);
                        if (row < A.m_out) A.out[ci * A.m_out + row] = __builtin_fmaf((float)acc[v], c1, wB[((v >> 2) * 2 + h) * 4 + (v & 3)]);
                    }
                }
            }
            cc += 1;
        } else {
            dhq_v16f y[PAIR_NT];
            float zl[PAIR_NT][8], zh[PAIR_NT][8];
            if constexpr (MODE == 0) {
                pair_input_layer<ACTK>(S, cc, c1, cd, y, hA, h);
                pair_transform<true>(S, y, zl, zh);
            } else {
                pair_hidden<ACTK>(S, cc, D.layer, c1, cd, y, hA, h);
                pair_transform<false>(S, y, zl, zh);
            }
#pragma unroll
            for (int T = 0; T < PAIR_NT; ++T) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float(&z)[8] = (q < 2) ? zl[T] : zh[T];
                    const float4 x = make_float4(z[4 * (q & 1)], z[4 * (q & 1) + 1], z[4 * (q & 1) + 2], z[4 * (q & 1) + 3]);
                    mx = fmaxf(fmaxf(mx, fmaxf(fabsf(x.x), fabsf(x.y))), fmaxf(fabsf(x.z), fabsf(x.w)));
                    D.xout[slot + (size_t)(4 * T + q) * 64] = x;
                }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if constexpr (MODE != 2) {
#pragma unroll
        for (int m = 1; m < 64; m *= 2) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
        if (lane == 0) red[wave] = mx;
        __syncthreads();
        if (threadIdx.x == 0) {
            float r = red[0];
#pragma unroll
            for (int w = 1; w < PAIR_WAVES; ++w) r = fmaxf(r, red[w]);
            D.partial[blockIdx.x] = r;
        }
    }
}

// ---- test hook: one layer of the kernel above on caller-supplied codes ------------------------
struct pair_dargs {
    pair_args w;
    const int8_t *codes_in;
    float *xhat;        // rows rounded up to whole workgroup tiles
    int8_t *codes_out;  // the same
    int32_t *acc;       // n rows
    int layer, kp_in;
};

// The integer accumulators for the test hook: a plain MFMA loop over the layer's packed fragments,
// read from device memory.  One wave per 32 coordinates.
__global__ __launch_bounds__(64) void pair_debug_acc_kernel(const pair_dargs D)
{
    const pair_args &A = D.w;
    const int lane = threadIdx.x & 63;
    const int c = lane & 31, h = lane >> 5;
    const int l = D.layer;
    const int64_t ci = (int64_t)blockIdx.x * 32 + c;
    const bool valid = ci < A.n;
    const int64_t cl = valid ? ci : A.n - 1;
    const int KB = (l == 0) ? 1 : PAIR_KB;
    for (int T = 0; T < 16; ++T) {
        // input layer: chunk 0, fragments [tile]; hidden layer l: chunk 1 + 8 (l - 1) + T % 8, fragments [role = T / 8][k block]
        const dhq_v4i *fr = (l == 0) ? reinterpret_cast<const dhq_v4i *>(A.blob) + (size_t)T * 64
                                     : reinterpret_cast<const dhq_v4i *>(A.blob + (size_t)(1 + 8 * (l - 1) + (T & 7)) * PAIR_BUF + (T >> 3) * 16384);
        dhq_v16i acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0;
        for (int kb = 0; kb < KB; ++kb) {
            dhq_v4i b = dhq_v4i{0, 0, 0, 0};
            if (l == 0) {
                unsigned w = 0;
                for (int k = 0; k < D.kp_in; ++k) w |= (unsigned)(uint8_t)D.codes_in[cl * D.kp_in + k] << (8 * k);
                b[0] = (int)w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const int *>(D.codes_in + cl * D.kp_in + 32 * kb + 8 * j + 4 * h);
            }
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[kb * 64 + lane], b, acc, 0, 0, 0);
        }
        if (valid) {
#pragma unroll
            for (int v = 0; v < 16; ++v) D.acc[ci * 512 + 32 * T + 8 * (v >> 2) + 4 * h + (v & 3)] = acc[v];
        }
    }
}

template <int ACTK>
__global__ __launch_bounds__(PAIR_THREADS) void dhq_fused_pair_kernel_debug(const pair_dargs D)
{
    const pair_args &A = D.w;
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int l = D.layer;
    const int qlo = DHQ_MAGIC_I - A.qmax, qhi = DHQ_MAGIC_I + A.qmax;
    const int cc0 = (l == 0) ? 0 : 1 + 8 * (l - 1);  // the layer's first chunk

    pair_stream S;
    pair_stream_init(S, &A, lds, wave, lane);
    int cc = cc0;
    pair_copy_now(S, cc0, cc0 & 1);
    pair_copy_bias(S, l);
    dhq_v4i hA[2];
    pair_h32_operand(c, h, S.role, hA);
    const int64_t ci = (int64_t)blockIdx.x * PAIR_TILE + S.grp * 32 + c;
    const int64_t cl = ci < A.n ? ci : A.n - 1;
    dhq_v4i cd[PAIR_KB];
#pragma unroll
    for (int kb = 0; kb < PAIR_KB; ++kb) cd[kb] = dhq_v4i{0, 0, 0, 0};
    dhq_v16f y[PAIR_NT];
    if (l == 0) {
        unsigned w = 0;
        for (int k = 0; k < D.kp_in; ++k) w |= (unsigned)(uint8_t)D.codes_in[cl * D.kp_in + k] << (8 * k);
        cd[0][0] = (int)w;
        pair_input_layer<ACTK>(S, cc, A.c1[0], cd, y, hA, h);
    } else {
        // the hidden layer reads its codes from the exchange area: [group][k block][lane] x 16 B,
        // dword q of k block T = rotated features 32 T + 8 q + 4 h .. + 3; role r brings in dwords 2 r, 2 r + 1
        unsigned char *dst = lds + 2 * PAIR_BUF + S.grp * 16384 + lane * 16 + S.role * 8;
#pragma unroll
        for (int T = 0; T < PAIR_KB; ++T) {
            const int f = 32 * T + 16 * S.role + 4 * h;
            const unsigned a0 = *reinterpret_cast<const unsigned *>(D.codes_in + cl * D.kp_in + f);
            const unsigned a1 = *reinterpret_cast<const unsigned *>(D.codes_in + cl * D.kp_in + f + 8);
            *reinterpret_cast<uint2 *>(dst + T * 1024) = make_uint2(a0, a1);
        }
        pair_hidden<ACTK>(S, cc, l, A.c1[l], cd, y, hA, h);
    }
    // both outputs go to workspace buffers with room for whole workgroup tiles, so nothing here is conditional
    pair_transform_quant<true>(S, y, A.inv_in[l + 1], qlo, qhi, h, D.xhat + ci * 512, reinterpret_cast<int *>(D.codes_out + ci * 512));
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// ------------------------------------------------------------------------------- host code
// `padded`: hidden widths of 257 .. 511, or of both kinds.
static bool pair_shape_ok(const dhq_model *m, bool padded)
{
    const int L = m->n_layers;
    if (L < 2) return false;
    if (m->dims[0] > 4 || m->dims[L] > 32) return false;
    if (dhq_padded_width(m->dims, L) != 512 || dhq_all_hidden_are(m->dims, L, 512) == padded) return false;
    return !padded || dhq_pad_act_ok(m->act_kind, dhq_hidden_act(m).c2);
}

// Which M tile wave role r computes as its t-th.  Exact networks: role 0 tiles 0..7, role 1 tiles 8..15, as described above.
// In the padded ones the last tiles are padding, and role r has tiles 2 t + r, so that both have as much of it (RT = 5..8 tiles
// each that are not; the exchange is then in front of the stage over tile-index bit 0).  Complex width 181, twelve real tiles of
// sixteen, 3 layers, 65 536 rows: 70.5 -> 57.5 us; 4 x 300 features 81.5 -> 60.1, 4 x 400 (wavelet) 96.7 -> 88.2.
static int pair_place(bool padded, int T) { return padded ? (T & 1) * 8 + (T >> 1) : T; }  // 8 r + t
static int pair_tile(bool padded, int place) { return padded ? 2 * (place & 7) + (place >> 3) : place; }

// k position jj of lane half u in k block kb of a hidden layer's A fragment holds rotated input
// feature hm_index(16 kb' + jj, u), kb' = pair_tile(kb): the order in which the transform leaves the codes.
static void pair_pack_tile(const dhq_layer &Ly, bool padded, int T, int Kb, bool first, int8_t *frag)
{
    const int8_t *wq = Ly.wq_host.data();
    for (int kb = 0; kb < Kb; ++kb)
        for (int ln = 0; ln < 64; ++ln) {
            const int row = 32 * T + (ln & 31), u = ln >> 5;
            for (int jj = 0; jj < 16; ++jj) {
                int8_t val = 0;
                if (row < Ly.M) {
                    if (first) {
                        if (u == 0 && jj < Ly.Kp) val = wq[(size_t)row * Ly.Kp + jj];
                    } else {
                        val = wq[(size_t)row * Ly.Kp + hm_index(16 * pair_tile(padded, kb) + jj, u)];
                    }
                }
                frag[((size_t)kb * 64 + ln) * 16 + jj] = val;
            }
        }
}

int dhq_pair_create(const dhq_model *m, bool padded, dhq_pair_plan **plan_out)
{
    *plan_out = nullptr;
    if (!pair_shape_ok(m, padded)) return DHQ_OK;
    const int L = m->n_layers;
    dhq_pair_plan *P = new (std::nothrow) dhq_pair_plan();
    if (!P) return DHQ_ENOMEM;
    memset(&P->args, 0, sizeof(P->args));
    P->rt = PAIR_NT;
    if (padded) {
        int widest = 0;
        for (int l = 1; l < L; ++l) widest = m->dims[l] > widest ? m->dims[l] : widest;
        P->rt = (widest + 63) / 64;
    }
    const int n_chunks = 2 + P->rt * (L - 2);
    // chunks, one more chunk of padding (the in-kernel copy always moves 32 KiB), then the bias table
    const size_t bias_off = (size_t)(n_chunks + 1) * PAIR_BUF;
    std::vector<unsigned char> blob(bias_off + (size_t)L * 512 * sizeof(float), 0);
    auto slot = [&](int l, int f) { return bias_slot(l == L - 1 ? f : 32 * pair_place(padded, f >> 5) + (f & 31)); };
    for (int l = 0; l < L; ++l) {
        const dhq_layer &Ly = m->layer[l];
        if (l == 0) {
            for (int T = 0; T < 16; ++T)
                pair_pack_tile(Ly, padded, T, 1, true, reinterpret_cast<int8_t *>(blob.data()) + (size_t)pair_place(padded, T) * 1024);
        } else if (l == L - 1) {
            pair_pack_tile(Ly, padded, 0, PAIR_KB, false, reinterpret_cast<int8_t *>(blob.data()) + (size_t)(n_chunks - 1) * PAIR_BUF);
        } else {
            for (int r = 0; r < 2; ++r)
                for (int t = 0; t < P->rt; ++t)
                    pair_pack_tile(Ly, padded, pair_tile(padded, 8 * r + t), PAIR_KB, false,
                                   reinterpret_cast<int8_t *>(blob.data()) + (size_t)(1 + P->rt * (l - 1) + t) * PAIR_BUF + (size_t)r * 16384);
        }
        // biases: bias_slot order within a tile, in revolutions for the layers that end in an activation
        float *bias = reinterpret_cast<float *>(blob.data() + bias_off) + (size_t)l * 512;
        const std::vector<float> &src = (l == L - 1) ? Ly.bias_host : Ly.bias_rev_host;
        for (int f = 0; f < Ly.M; ++f) bias[slot(l, f)] = src[f];
        if (l < L - 1)
            for (int f = Ly.M; f < 512; ++f) bias[slot(l, f)] = dhq_pad_bias(m->act_kind, f);
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
    P->args.m_out = m->dims[L];
    P->args.qmax = m->qmax_a;
    P->args.n_chunks = n_chunks;
    P->args.bias_off = (uint32_t)bias_off;
    P->args.c2 = dhq_hidden_act(m).c2;
    P->args.scale = padded ? ldexpf(1.f, dhq_piece_scale_log2(m->act_kind, P->args.c2)) : 1.f;
    P->act_kind = m->act_kind;
    P->padded = padded;
    P->lds_bytes = (size_t)PAIR_BIAS + 3 * 2048;
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

void dhq_pair_destroy(dhq_pair_plan *P)
{
    if (!P) return;
    if (P->blob_dev) (void)hipFree(P->blob_dev);
    delete P;
}

int dhq_pair_update_scales(const dhq_model *m, dhq_pair_plan *P)
{
    if (!P) return DHQ_OK;
    for (int l = 0; l < m->n_layers; ++l) {
        const dhq_layer &Ly = m->layer[l];
        P->args.c1[l] = dhq_c1(m, l);
        P->args.inv_in[l] = (float)(1.0 / ((double)Ly.s_a * sqrt((double)Ly.Kp)));
        if (l > 0) P->args.inv_in[l] /= P->args.scale;  // a power of two
    }
    return DHQ_OK;
}

template <int ACTK>
static void (*pair_kernel_of(const dhq_pair_plan *P))(const pair_args)
{
    if (!P->padded) return dhq_fused_pair_kernel<ACTK, PAIR_NT>;
    switch (P->rt) {
        case 5: return dhq_fused_pair_kernel<ACTK | DHQ_SPLIT_RN, 5>;
        case 6: return dhq_fused_pair_kernel<ACTK | DHQ_SPLIT_RN, 6>;
        case 7: return dhq_fused_pair_kernel<ACTK | DHQ_SPLIT_RN, 7>;
        default: return dhq_fused_pair_kernel<ACTK | DHQ_SPLIT_RN, 8>;
    }
}

hipError_t dhq_pair_launch(const dhq_pair_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    if (!P) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    pair_args a = P->args;
    a.coords = coords;
    a.out = out;
    a.n = n;
    const int64_t tiles = (n + PAIR_TILE - 1) / PAIR_TILE;
    const unsigned grid = (unsigned)(tiles < P->n_cu ? tiles : P->n_cu);
    auto kern = (P->act_kind == DHQ_ACT_KIND_WAVELET)           ? pair_kernel_of<DHQ_ACT_KIND_WAVELET>(P)
                : (P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) ? pair_kernel_of<DHQ_ACT_KIND_WAVELET_COMPLEX>(P)
                                                                : pair_kernel_of<DHQ_ACT_KIND_SINE>(P);
    const hipError_t e = dhq_lds_limit_once(kern, P->lds_bytes, P->device);
    if (e != hipSuccess) return e;
    kern<<<grid, PAIR_THREADS, P->lds_bytes, st>>>(a);
    return hipGetLastError();
}

// ---- the two-sided kernel ----
// Fragment of one tile and digit plane: byte jj of lane (i, u) of k block kb is the digit of U[row(i)][feature(kb, u, jj)].
template <typename Weight, typename Row, typename Col>
static void pair2_pack(const std::vector<Weight> &U, int Kp, int n_rows, int Kb, int plane, Row row_of, Col col_of, int8_t *frag)
{
    for (int kb = 0; kb < Kb; ++kb)
        for (int ln = 0; ln < 64; ++ln) {
            const int row = row_of(ln & 31);
            if (row >= n_rows) continue;  // stays zero
            for (int jj = 0; jj < 16; ++jj) {
                const int k = col_of(kb, ln >> 5, jj);
                if (k < 0) continue;
                const int32_t u = U[(size_t)row * Kp + k], u0 = ((u + 128) & 255) - 128;
                frag[((size_t)kb * 64 + ln) * 16 + jj] = (int8_t)(plane ? (u - u0) / 256 : u0);
            }
        }
}

int dhq_pair2_create(const dhq_model *m, dhq_pair_plan **plan_out)
{
    *plan_out = nullptr;
    const int L = m->n_layers;
    if (L < 2 || m->dims[L] > 32) return DHQ_OK;
    // One-sided networks of 257 to 512 with a fan-in of 5 to 32 run here too, with U = W' and an upper digit of zero: the values are
    // then the layer-by-layer path's.
    const bool wide_input = m->dims[0] > 4;
    if (wide_input ? m->rot_out || m->layer[0].Kp > 32 || dhq_padded_width(m->dims, L) != 512 || !dhq_pad_act_ok(m->act_kind, dhq_hidden_act(m).c2)
                   : !m->rot_out || !dhq_all_hidden_are(m->dims, L, 512))
        return DHQ_OK;
    if (m->act_kind != DHQ_ACT_KIND_SINE && m->act_kind != DHQ_ACT_KIND_WAVELET) return DHQ_OK;
    for (int l = 0; l < L; ++l)
        for (int32_t u : m->layer[l].u_host)
            if (u > PAIR2_MAX_U || u < -PAIR2_MAX_U) return DHQ_OK;
    dhq_pair_plan *P = new (std::nothrow) dhq_pair_plan();
    if (!P) return DHQ_ENOMEM;
    memset(&P->args, 0, sizeof(P->args));
    const int n_chunks = 2 + 16 * (L - 2);
    const size_t bias_off = (size_t)(n_chunks + 1) * PAIR_BUF;
    std::vector<unsigned char> blob(bias_off + (size_t)L * 512 * sizeof(float), 0);
    int8_t *frags = reinterpret_cast<int8_t *>(blob.data());
    for (int l = 0; l < L; ++l) {
        const dhq_layer &Ly = m->layer[l];
        const bool first = (l == 0), last = (l == L - 1);
        const int Kp = Ly.Kp;
        auto col = [&](int kb, int u, int jj) { return first ? (16 * u + jj < Kp ? 16 * u + jj : -1) : pair2_code_feature(kb, u, jj); };
        auto pack = [&](int n_rows, int Kb, int plane, auto row, int8_t *frag) {
            if (wide_input) pair2_pack(Ly.wq_host, Kp, n_rows, Kb, plane, row, col, frag);
            else pair2_pack(Ly.u_host, Kp, n_rows, Kb, plane, row, col, frag);
        };
        float *bias = reinterpret_cast<float *>(blob.data() + bias_off) + (size_t)l * 512;
        if (last) {
            auto row = [](int i) { return i; };
            for (int p = 0; p < 2; ++p)
                pack(Ly.M, PAIR_KB, 1 - p, row, frags + (size_t)(n_chunks - 1) * PAIR_BUF + (size_t)p * 16384);
            for (int f = 0; f < Ly.M; ++f) bias[bias_slot(f)] = Ly.bias_host[f];
            continue;
        }
        for (int role = 0; role < 2; ++role)
            for (int T = 0; T < PAIR_NT; ++T) {
                // row 8 g + 4 h + e of an MFMA tile is accumulator 4 g + e of lane half h
                auto row = [&](int i) { return pair2_feature(role, T, 4 * (i >> 3) + (i & 3), (i >> 2) & 1); };
                for (int p = 0; p < 2; ++p) {
                    int8_t *dst = first ? frags + (size_t)role * 16384 + (size_t)(2 * T + p) * 1024
                                        : frags + (size_t)(1 + 16 * (l - 1) + 2 * T + p) * PAIR_BUF + (size_t)role * 16384;
                    pack(Ly.M, first ? 1 : PAIR_KB, 1 - p, row, dst);
                }
                for (int i = 0; i < 32; ++i)
                    bias[bias_slot(32 * (8 * role + T) + i)] = row(i) < Ly.M ? Ly.bias_rev_host[row(i)] : dhq_pad_bias(m->act_kind, row(i));
            }
    }
    P->blob_bytes = blob.size();
    if (hipMalloc((void **)&P->blob_dev, P->blob_bytes) != hipSuccess) {
        delete P;
        return DHQ_ENOMEM;
    }
    hipDeviceProp_t prop;
    if (hipMemcpy(P->blob_dev, blob.data(), P->blob_bytes, hipMemcpyHostToDevice) != hipSuccess ||
        hipGetDeviceProperties(&prop, m->device) != hipSuccess) {
        dhq_pair_destroy(P);
        return DHQ_EHIP;
    }
    P->args.blob = P->blob_dev;
    P->args.n_layers = L;
    P->args.k0 = m->dims[0];
    P->args.k0p = m->layer[0].Kp;
    P->args.m_out = m->dims[L];
    P->args.qmax = m->qmax_a;
    P->args.n_chunks = n_chunks;
    P->args.bias_off = (uint32_t)bias_off;
    P->args.c2 = dhq_hidden_act(m).c2;
    P->args.scale = 1.f;
    P->act_kind = m->act_kind;
    P->lds_bytes = (size_t)PAIR_BIAS + 3 * 2048;
    P->n_cu = prop.multiProcessorCount;
    P->device = m->device;
    *plan_out = P;
    return DHQ_OK;
}

template <int FLAGS>
static void (*pair2_kernel_of(const dhq_pair_plan *P))(const pair_args)
{
    return P->act_kind == DHQ_ACT_KIND_WAVELET ? dhq_fused_pair2_kernel<DHQ_ACT_KIND_WAVELET | FLAGS> : dhq_fused_pair2_kernel<DHQ_ACT_KIND_SINE | FLAGS>;
}

hipError_t dhq_pair2_launch(const dhq_model *m, const dhq_pair_plan *P, const float *coords, int64_t n, float *out, hipStream_t st)
{
    if (!P) return hipErrorInvalidValue;
    const bool wide_input = m->dims[0] > 4;
    auto kern = wide_input ? pair2_kernel_of<DHQ_CODES_IN>(P) : pair2_kernel_of<0>(P);
    hipError_t e = dhq_lds_limit_once(kern, P->lds_bytes, P->device);
    if (e != hipSuccess) return e;
    // a fan-in above 4: as in dhq_fused_launch
    const int64_t step = wide_input ? DHQ_CHUNK * (int64_t)m->max_kp / P->args.k0p : n;
    for (int64_t off = 0; off < n; off += step) {
        pair_args a = P->args;
        a.coords = coords + off * a.k0;
        a.out = out + off * a.m_out;
        a.n = n - off < step ? n - off : step;
        if (wide_input) {
            const dhq_layer &Ly = m->layer[0];
            e = dhq_launch_wht_quant(a.coords, a.n, Ly.K, Ly.Kp, a.inv_in[0], m->qmax_a, m->codes, nullptr, st);
            if (e != hipSuccess) return e;
            a.codes0 = m->codes;
        }
        const int64_t tiles = (a.n + PAIR_TILE - 1) / PAIR_TILE;
        const unsigned grid = (unsigned)(tiles < P->n_cu ? tiles : P->n_cu);
        kern<<<grid, PAIR_THREADS, P->lds_bytes, st>>>(a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The dynamic mode on the per-layer kernels above (same contract as dhq_fused_dynamic_launch): ws0 / ws1 hold
// dhq_pair_dynamic_rows(n) x 512 floats each.
size_t dhq_pair_dynamic_rows(int64_t n) { return (size_t)((n + PAIR_TILE - 1) / PAIR_TILE) * PAIR_TILE; }

template <int MODE, int ACTK>
static hipError_t pairl_launch_t(const dhq_pair_plan *P, const pair_largs &a, unsigned grid, hipStream_t st)
{
    auto kern = dhq_fused_pair_layer_kernel<MODE, ACTK>;
    hipError_t e = dhq_lds_limit_once(kern, P->lds_bytes, P->device);
    if (e != hipSuccess) return e;
    kern<<<grid, PAIR_THREADS, P->lds_bytes, st>>>(a);
    return hipGetLastError();
}

hipError_t dhq_pair_dynamic_launch(const dhq_model *m, const float *coords, int64_t n, float *out, float *ws0, float *ws1,
                                   float *partial, float *dyn, hipStream_t st)
{
    const dhq_pair_plan *P = m->pair;
    if (!P) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    const int L = m->n_layers;
    const bool wav = (P->act_kind == DHQ_ACT_KIND_WAVELET), cpx = (P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX);
    const int64_t tiles = (n + PAIR_TILE - 1) / PAIR_TILE;
    const unsigned grid = (unsigned)(tiles < P->n_cu ? tiles : P->n_cu);
    if (grid > DHQ_ABSMAX_PARTIALS) return hipErrorInvalidValue;
    // the input layer's scale: max over the rotated coordinates, left as per-workgroup maxima
    float *pbuf[2] = {partial, partial + DHQ_ABSMAX_PARTIALS};
    int count = 0;
    hipError_t e = dhq_launch_wht_absmax_partials(coords, n, m->layer[0].K, m->layer[0].Kp, pbuf[0], &count, st);
    if (e != hipSuccess) return e;
    float *bufs[2] = {ws0, ws1};
    for (int l = 0; l < L; ++l) {
        pair_largs a;
        memset(&a, 0, sizeof(a));
        a.w = P->args;
        a.w.coords = coords;
        a.w.out = out;
        a.w.n = n;
        // the chunks of this layer alone, in a cycle
        a.w.chunk_base = (l == 0) ? 0 : (l == L - 1 ? P->args.n_chunks - 1 : 1 + 8 * (l - 1));
        a.w.n_chunks = (l == 0 || l == L - 1) ? 1 : 8;
        a.xin = reinterpret_cast<const float4 *>(bufs[(l + 1) & 1]);
        a.xout = reinterpret_cast<float4 *>(bufs[l & 1]);
        a.partial_in = pbuf[l & 1];
        a.partial_count = count;
        a.kp = m->layer[l].Kp;
        a.layer = l;
        a.c1_over_sa = dhq_c1_over_sa(m, l);
        a.dyn = dyn + 3 * l;
        a.partial = pbuf[(l + 1) & 1];
        if (l == 0) e = wav ? pairl_launch_t<0, DHQ_ACT_KIND_WAVELET>(P, a, grid, st) : cpx ? pairl_launch_t<0, DHQ_ACT_KIND_WAVELET_COMPLEX>(P, a, grid, st)
                                                                                        : pairl_launch_t<0, DHQ_ACT_KIND_SINE>(P, a, grid, st);
        else if (l < L - 1) e = wav ? pairl_launch_t<1, DHQ_ACT_KIND_WAVELET>(P, a, grid, st) : cpx ? pairl_launch_t<1, DHQ_ACT_KIND_WAVELET_COMPLEX>(P, a, grid, st)
                                                                                                : pairl_launch_t<1, DHQ_ACT_KIND_SINE>(P, a, grid, st);
        else e = pairl_launch_t<2, DHQ_ACT_KIND_NONE>(P, a, grid, st);  // the output layer has no activation
        if (e != hipSuccess) return e;
        count = (int)grid;
    }
    return hipSuccess;
}

// Test hook behind dhq_forward_debug_fused for the two-wave kernel.
hipError_t dhq_pair_debug_launch(const dhq_model *m, int layer, const int8_t *codes_in, int64_t n, float *xhat, int8_t *codes_out,
                                 int32_t *acc, hipStream_t st)
{
    const dhq_pair_plan *P = m->pair;
    if (!P || layer < 0 || layer >= m->n_layers - 1) return hipErrorInvalidValue;
    if (n <= 0) return hipSuccess;
    if (n > DHQ_CHUNK) return hipErrorInvalidValue;  // the outputs pass through the model's workspace (whole tiles)
    pair_dargs d;
    memset(&d, 0, sizeof(d));
    d.w = P->args;
    d.w.n = n;
    d.codes_in = codes_in;
    d.xhat = m->act0;
    d.codes_out = m->codes;
    d.acc = acc;
    d.layer = layer;
    d.kp_in = m->layer[layer].Kp;
    const unsigned grid = (unsigned)((n + PAIR_TILE - 1) / PAIR_TILE);
    auto kern = (P->act_kind == DHQ_ACT_KIND_WAVELET) ? dhq_fused_pair_kernel_debug<DHQ_ACT_KIND_WAVELET>
                : (P->act_kind == DHQ_ACT_KIND_WAVELET_COMPLEX) ? dhq_fused_pair_kernel_debug<DHQ_ACT_KIND_WAVELET_COMPLEX>
                                                                : dhq_fused_pair_kernel_debug<DHQ_ACT_KIND_SINE>;
    hipError_t e = dhq_lds_limit_once(kern, P->lds_bytes, P->device);
    if (e != hipSuccess) return e;
    if (acc) {
        pair_debug_acc_kernel<<<(unsigned)((n + 31) / 32), 64, 0, st>>>(d);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (!xhat && !codes_out) return hipSuccess;
    kern<<<grid, PAIR_THREADS, P->lds_bytes, st>>>(d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (xhat && (e = hipMemcpyAsync(xhat, m->act0, sizeof(float) * (size_t)n * 512, hipMemcpyDeviceToDevice, st)) != hipSuccess) return e;
    if (codes_out && (e = hipMemcpyAsync(codes_out, m->codes, (size_t)n * 512, hipMemcpyDeviceToDevice, st)) != hipSuccess) return e;
    return hipSuccess;
}
