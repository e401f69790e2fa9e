// The training tile kernel: MLP forward, KL-gradient head (Sec. 4.2, eq.
// mcgradients), delta chain and weight gradients of a batch whose grid features
// were encoded level by level before (k_encode.hip); the tile's dG is stored
// for the scatter passes.
//
// What bounds it.  FP32 matrix instructions run on the vector unit's
// multipliers on this chip: a wave's FP32 products and any wave's vector
// instructions add up (matrix 250 us and vector 273 us of work take 511 us
// together), while BF16 products run beside vector work at 16 times the rate.
// So the FP32 form keeps FP32 instructions only where their exact sums decide
// something -- the forward pass, whose sign selects each ReLU -- and forms the
// products of the backward pass from operands split into three BF16 numbers
// (below): 24,576 of the 36,864 FP32 matrix cycles of a tile become 9,216 BF16
// ones that overlap the rest.
//
// Split operands: x = x0 + x1 + x2 exactly (8 + 8 + 8 significand bits, each
// remainder of a round-to-nearest BF16 conversion is exact in FP32), and the
// six products x0 y0, x0 y1, x1 y0, x1 y1, x0 y2, x2 y0 (Henry, Tang and
// Heinecke, 2019) leave out at most 2^-24 of the product (2^-26 or less in 97
// of 100), half an FP32 rounding step; adding x1 y2 and x2 y1 changed no
// gradient's error and cost 2.5 % of a step.  What does matter is how the
// products are summed: the matrix unit cuts an addend off at the last place of
// the largest of an instruction's 16 products and its sum, so the five small
// products, added to the sum of the large ones, lost their last bits each time.
// They are summed by themselves and added once by the vector unit: in the delta
// chain over the whole layer, in the weight gradients over a tile.  Weight
// gradients of the 16-level network, 30,001 vertices, error against 64 bits
// relative to the kernel with FP32 products: layers 0 to 3 1.20, 1.55, 1.19 and
// 0.96 with one sum, 1.02, 1.05, 1.01 and 0.97 with two, the whole gradient
// 1.15 and 1.00 (0.97 to 0.99 on other networks and sizes); a step of 2^20
// vertices takes 2 % longer for it.
//
// A wave is on its own from tile to tile: it keeps all weight-gradient blocks
// in accumulators (192 registers of the 512 a wave has at one per SIMD) and
// transposes its deltas and layer inputs itself, one 32-row block at a time,
// because the tile's vertices are the reduction dimension there.  No barrier
// stands between a block's waves; their weight gradients meet in LDS once at
// the end.
//
// Measured against the kernel that gathers (k_fused.hip), this one with its
// encode: 2^20 vertices on the 16-level hash grid FP32 1,075 -> 248 + 671 us,
// BF16 585 -> 198 + 250; NPM-product BF16, 300,001 vertices, 247 -> 83 + 118;
// 8-level dense grid FP32, 2^18 vertices, 179 -> 21 + 129.  What bounds it now,
// by counters at 2^20 vertices: FP32 form, 49k cycles a tile, the matrix unit
// busy for half of them (FP32 products 12.3k, BF16 12k) and vector instructions
// issuing for 42 %, which a single wave overlaps little; precision form, 18k
// cycles, vector instructions for 62 %.
#include <type_traits>

#include "fused_launch.h"

namespace npm {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <bool BF> constexpr int kPlanes = BF ? 1 : 3;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// R registers of a tile-layout vector as BF16 planes, two registers a word:
// one plane in the precision form, the three-way split in FP32.
template <int R, bool BF> struct Planes {
    uint32_t w[kPlanes<BF>][R / 2];

    __device__ __forceinline__ void set(const float *x)
    {
#pragma unroll
        for (int i = 0; i < R / 2; ++i) {
            float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
            for (int p = 0; p < kPlanes<BF>; ++p) {
                w[p][i] = pack_bf16(a, b);
                if (p + 1 < kPlanes<BF>) {
                    a -= lo_f32(w[p][i]);
                    b -= hi_f32(w[p][i]);
                }
            }
        }
    }
    // matrix operand of registers [8 s, 8 s + 8), plane p
    __device__ __forceinline__ bf16x8 op(int p, int s) const
    {
        const uint4 v = {w[p][4 * s], w[p][4 * s + 1], w[p][4 * s + 2], w[p][4 * s + 3]};
        return __builtin_bit_cast(bf16x8, v);
    }
};

// The planes' products from the smallest up: A[pa(i)] B[pb(i)], i = 0 .. N - 1.
template <bool BF> struct Products {
    static constexpr int N = BF ? 1 : 6;
    static constexpr int pa(int i) { return BF ? 0 : (int[]){2, 0, 1, 1, 0, 0}[i]; }
    static constexpr int pb(int i) { return BF ? 0 : (int[]){0, 2, 1, 0, 1, 0}[i]; }
};

__device__ __forceinline__ f32x16 zero16()
{
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.0f;
    return z;
}

// y (M wide) = W^T d for the planes d of a K-wide vector; img: plane p of the
// packed BF16 image of W^T at img + p * stride (device_math.h's layout).  The
// largest products and the others have sums of their own (see the top).
template <int K, int M, bool BF>
__device__ __forceinline__ void chain_layer(const __bf16 *img, int stride, const Planes<K / 2, BF> &d,
                                            float *y, int lane)
{
    constexpr int NB = M / 32, NS = K / 16, P = kPlanes<BF>;
    f32x16 acc[NB], low[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = low[b] = zero16();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        bf16x8 A[NB][P];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int p = 0; p < P; ++p)
                A[b][p] = *reinterpret_cast<const bf16x8 *>(img + p * stride + ((b * NS + s) * 64 + lane) * 8);
        // the blocks in turn: two products in a row never wait for one sum
#pragma unroll
        for (int i = 0; i < Products<BF>::N; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                f32x16 &q = i + 1 < Products<BF>::N ? low[b] : acc[b];
                q = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[b][Products<BF>::pa(i)],
                                                            d.op(Products<BF>::pb(i), s), q, 0, 0, 0);
            }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) y[16 * b + v] = BF ? acc[b][v] : acc[b][v] + low[b][v];
}

// A 32-row block with the tile's 32 vertices as the reduction dimension: lane
// i % 32 holds row i, and of the step s the half-wave h the vertices
// nf(h, 8 s + e).  The matrix unit transposes: with the block's planes as the
// left operand (rows = vertices) and the identity as the right one, the product
// has the block's rows as its columns, exactly (one term each), and its
// registers are the next operands.  Through LDS the same transposition took 16
// two-byte writes a block and plane and waited for its reads (8-level network,
// 2^18 vertices FP32, 160 -> 142 us; NPM-product in BF16, 300,001 vertices, 168
// -> 135 us).
struct Identity {
    bf16x8 k[2];
    __device__ __forceinline__ explicit Identity(int lane)
    {
        const int n = lane & 31, h = lane >> 5;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) k[s][e] = (__bf16)(n == nf(h, 8 * s + e) ? 1.0f : 0.0f);
    }
};
template <bool BF> struct Rows {
    bf16x8 k[2][kPlanes<BF>];

    // the registers [16 blk, 16 blk + 16) of v
    template <int R>
    __device__ __forceinline__ void load(const Identity &id, const Planes<R, BF> &v, int blk)
    {
        f32x16 t[kPlanes<BF>];
#pragma unroll
        for (int p = 0; p < kPlanes<BF>; ++p)
            t[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.op(p, 2 * blk), id.k[0], zero16(), 0, 0, 0);
#pragma unroll
        for (int p = 0; p < kPlanes<BF>; ++p)
            t[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.op(p, 2 * blk + 1), id.k[1], t[p], 0, 0, 0);
#pragma unroll
        for (int p = 0; p < kPlanes<BF>; ++p)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                uint32_t w[4];
                // the values are BF16 numbers: the upper halves of their FP32 forms
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    w[i] = __builtin_amdgcn_perm(__float_as_uint(t[p][8 * s + 2 * i + 1]),
                                                 __float_as_uint(t[p][8 * s + 2 * i]), 0x07060302u);
                k[s][p] = __builtin_bit_cast(bf16x8, uint4{w[0], w[1], w[2], w[3]});
            }
    }
};

// Weight-gradient blocks (32 x 32) of a network, layer by layer from the
// output layer down, each layer's blocks row block by row block.
template <int IN_P, int HID_P, int NH> struct DwBlocks {
    static constexpr int IN0 = IN_P < 32 ? 32 : IN_P;
    static constexpr int out_p(int L) { return L == NH ? 32 : HID_P; }
    static constexpr int in_p(int L) { return L == 0 ? IN0 : HID_P; }
    static constexpr int nbi(int L) { return in_p(L) / 32; }
    static constexpr int blocks(int L) { return (out_p(L) / 32) * nbi(L); }
    static constexpr int first(int L)
    {
        int g = 0;
        for (int l = NH; l > L; --l) g += blocks(l);
        return g;
    }
    static constexpr int total() { return first(-1); }
};

// A vertex with an infinite or NaN feature, or derivative of the head, takes no
// part in a tile's products: the split has no form for such a value, and the
// identity product would hand it to the other 31 rows of its block.  The tile
// loop takes it as zero, leaves kOddInput or kOddHead in the first row of its dG,
// and at the end of the block, the accumulators written, the wave evaluates such
// vertices one at a time (OddVertex), so that they mark the gradient entries they
// belong to -- those of the units that are on -- and no others.  The checks cost
// a finite batch 0.3 to 1 % of a step (2 % at 16,384 vertices).
constexpr uint32_t kOddInput = 0x7fc0dd01u, kOddHead = 0x7fc0dd02u;      // NaNs no sum makes
// the lanes with an infinite or NaN value among R
template <int R> __device__ __forceinline__ uint64_t odd_lanes(const float *x, float z = 0.0f)
{
    z *= 0.0f;
#pragma unroll
    for (int i = 0; i < R; ++i) z = fmaf(x[i], 0.0f, z);
    return __ballot(z != z);
}

// FP32 with three hidden layers or the selection sums: the first layer's
// activations wait in LDS (8 KB a wave), and the input features are read again
// for their weight gradient.
constexpr bool parks(bool bf, int hidden, bool sel) { return !bf && (hidden >= 3 || sel); }

// One vertex's layers by a wave, a unit per lane, weights read from memory as
// the form uses them (rounded to BF16 in the precision form).
template <bool BF> struct OddVertex {
    const float *w;                            // flat MLP weights
    float *g;                                  // their gradient
    int lane;

    __device__ __forceinline__ static float used(float x) { return BF ? (float)(__bf16)x : x; }
    // row `lane` of the layer at off times in
    __device__ __forceinline__ float forward(int64_t off, int rows, int cols, const float *in) const
    {
        float s = 0.0f;
        if (lane < rows)
            for (int i = 0; i < cols; ++i) s = fmaf(used(w[off + (int64_t)lane * cols + i]), used(in[i]), s);
        return s;
    }
    // the layer's weight gradient
    __device__ __forceinline__ void weights(int64_t off, int rows, int cols, const float *d, const float *in) const
    {
        for (int o = 0; o < rows; ++o)
            for (int i = lane; i < cols; i += 64)
                unsafeAtomicAdd(g + off + (int64_t)o * cols + i, used(d[o]) * used(in[i]));
    }
    // column `lane` of the layer times d
    __device__ __forceinline__ float back(int64_t off, int rows, int cols, const float *d) const
    {
        float s = 0.0f;
        if (lane < cols)
            for (int o = 0; o < rows; ++o) s = fmaf(used(w[off + (int64_t)o * cols + lane]), used(d[o]), s);
        return s;
    }
};

}  // namespace

// SEL: the network has the selection output (k_fused.hip); the row's gradient is
// kept per lane (its vertices' share of each feature) and summed at the end.
template <int IN_P, int HID_P, int NH, int F, bool BF, int PG, bool SEL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_train_tile(FusedArgs a, int mlp_weights,
                                                                                              int fwd_bytes, int t_elems)
{
    using DB = DwBlocks<IN_P, HID_P, NH>;
    constexpr int IN0 = DB::IN0, P = kPlanes<BF>, NDW = DB::total();
    constexpr int DGR = PG > 0 ? 32 : IN0;      // input-gradient rows (grid features only with PG)
    constexpr int ING = PG > 0 ? ProductShape<PG>::GF : IN_P;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double red[256];
    __shared__ __attribute__((aligned(16))) float s_wsel[SEL ? HID_P : 4];
    // LDS: the forward image, the planes of the backward (W^T) image
    const char *fwd = smem;
    __bf16 *bwd = reinterpret_cast<__bf16 *>(smem + fwd_bytes);
    for (int i = threadIdx.x; i < fwd_bytes / 16; i += 256)
        reinterpret_cast<f32x4 *>(smem)[i] = reinterpret_cast<const f32x4 *>(a.img)[i];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(p == 0 ? a.img_t : a.img_split + (size_t)(p - 1) * a.bwd_elems);
        for (int i = threadIdx.x; i < t_elems / 8; i += 256)
            reinterpret_cast<f32x4 *>(bwd + p * t_elems)[i] = src[i];
    }
    if constexpr (SEL)
        for (int i = threadIdx.x; i < HID_P; i += 256) s_wsel[i] = i < a.width ? a.wsel[i] : 0.0f;
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
    constexpr bool PARK = parks(BF, NH, SEL);
    f32x4 *park = reinterpret_cast<f32x4 *>(bwd + P * t_elems) + wave * (HID_P / 8 * 64) + lane;
    const Identity id(lane);
    const TrainIO io{a.n, a.pos, a.dir, a.rad, a.spdf, a.grad, a.invN, a.perm, a.rec, a.aux,
                     a.rec_stride, a.bsdf};
    const int gf = a.g.n_levels * F;
    f32x16 acc[NDW];
#pragma unroll
    for (int k = 0; k < NDW; ++k) acc[k] = zero16();
    float selacc[SEL ? HID_P / 2 : 1];
#pragma unroll
    for (int i = 0; i < (SEL ? HID_P / 2 : 1); ++i) selacc[i] = 0.0f;
    double lacc = 0.0, lsel = 0.0;
    bool any_odd = false;
    const int64_t n = a.n, ntiles = (n + 31) / 32;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    auto slot = [&](int64_t t) {
        const int64_t v = t * 32 + (lane & 31);
        return v < n ? v : n - 1;
    };
    int64_t t = blockIdx.x * (int64_t)4 + wave;
    FeatWords<ING, BF> fw;
    TrainInputs in_next;
    if (t < ntiles) {
        feat_load<ING, BF>(a.feat, gf, n, slot(t), h, fw);
        in_next = train_inputs(io, slot(t), slot(t));
    }
    for (; t < ntiles; t += nwaves) {
        bool valid = t * 32 + (lane & 31) < n;
        const TrainInputs in = in_next;
        float x[IN0 / 2];
        feat_take<IN_P, ING, BF>(fw, gf, h, x);
#pragma unroll
        for (int i = IN_P / 2; i < IN0 / 2; ++i) x[i] = 0.0f;
        if constexpr (PG > 0) {
            float a7[7];
            load_aux(io.rec, io.rec_stride, io.aux, n, slot(t), slot(t), a7);
            aux_fill<IN_P, ProductShape<PG>::GF, ProductShape<PG>::SHD>(h, a7, x);
        }
        const uint64_t odd_in = odd_lanes<IN_P / 2>(x);
        uint32_t odd = (uint32_t)odd_in | (uint32_t)(odd_in >> 32);
        const bool odd_x = (odd >> (lane & 31)) & 1u;
        valid = valid && !odd_x;
#pragma unroll
        for (int i = 0; i < IN_P / 2; ++i) x[i] = odd_x ? 0.0f : x[i];
        // the next tile's inputs, in flight during this one
        if (t + nwaves < ntiles) {
            feat_load<ING, BF>(a.feat, gf, n, slot(t + nwaves), h, fw);
            in_next = train_inputs(io, slot(t + nwaves), slot(t + nwaves));
        }
        // ---- forward
        float o[16], cp = 0.0f;
        float acts[BF ? 1 : NH][HID_P / 2];           // FP32 form
        Planes<HID_P / 2, true> ap[BF ? NH : 1];      // precision form: the activations as used
        Planes<IN0 / 2, BF> xp;
        if constexpr (BF) {
            xp.set(x);
            float y[HID_P / 2];
            mfma_layer_bf16<IN_P, HID_P>(reinterpret_cast<const __bf16 *>(fwd), x, y, lane);
#pragma unroll
            for (int li = 0; li < NH; ++li) {
#pragma unroll
                for (int i = 0; i < HID_P / 2; ++i) y[i] = fmaxf(y[i], 0.0f);
                if constexpr (SEL)
                    if (li == NH - 1) cp = select_logit<HID_P>(s_wsel, y, h);
                ap[li].set(y);
                const __bf16 *im = reinterpret_cast<const __bf16 *>(fwd) + HID_P * IN_P + li * HID_P * HID_P;
                if (li + 1 < NH) {
                    float z[HID_P / 2];
                    mfma_layer_bf16<HID_P, HID_P>(im, y, z, lane);
#pragma unroll
                    for (int i = 0; i < HID_P / 2; ++i) y[i] = z[i];
                } else {
                    mfma_layer_bf16<HID_P, 32>(im, y, o, lane);
                }
            }
        } else {
            const float *im = reinterpret_cast<const float *>(fwd);
            mfma_layer_f32<IN_P, HID_P>(im, x, acts[0], lane);
            im += HID_P * IN_P;
#pragma unroll
            for (int li = 0; li < NH; ++li) {
#pragma unroll
                for (int i = 0; i < HID_P / 2; ++i) acts[li][i] = fmaxf(acts[li][i], 0.0f);
                if (li + 1 < NH) mfma_layer_f32<HID_P, HID_P>(im, acts[li], acts[li + 1 < NH ? li + 1 : 0], lane);
                else mfma_layer_f32<HID_P, 32>(im, acts[li], o, lane);
                im += HID_P * HID_P;
                if (PARK && li == 0) {
#pragma unroll
                    for (int q = 0; q < HID_P / 8; ++q)
                        park[q * 64] = f32x4{acts[0][4 * q], acts[0][4 * q + 1], acts[0][4 * q + 2], acts[0][4 * q + 3]};
                }
            }
            if constexpr (SEL) cp = select_logit<HID_P>(s_wsel, acts[NH - 1], h);
        }
        // ---- head
        float d[16];
        const float lv = kl_head<!BF>(o, in, valid, io.invN, h, d, lacc);
        float ds = 0.0f;            // SEL: d loss / d c'
        if constexpr (SEL) {
            const float wgt = valid ? sample_weight(in.rad, in.spdf) : 0.0f;
            if (wgt != 0.0f && io.bsdf) {
                const float pb = io.bsdf[visit(io.perm, slot(t))];
                if (bsdf_valid(pb)) {
                    const float lpc = select_term(cp, pb, lv, -wgt * io.invN, ds);
                    if (h == 0) lsel -= (double)wgt * (double)lpc;
                }
            }
        }
        const uint64_t odd_out = odd_lanes<16>(d, ds);
        odd |= (uint32_t)odd_out | (uint32_t)(odd_out >> 32);
        const bool is_odd = (odd >> (lane & 31)) & 1u;
        any_odd |= odd != 0u;
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = is_odd ? 0.0f : d[i];
        if constexpr (SEL) ds = is_odd ? 0.0f : ds;
        // hidden unit i of layer li is on / the value its weight gradient takes
        auto on = [&](int li, int i) {
            if constexpr (BF) {
                const uint32_t w = ap[li].w[0][i >> 1];
                return ((i & 1) ? (w >> 16) : (w & 0xffffu)) != 0u;
            } else {
                return acts[li][i] > 0.0f;
            }
        };
        if constexpr (SEL) {
#pragma unroll
            for (int i = 0; i < HID_P / 2; ++i) {
                float v;
                if constexpr (BF) {
                    const uint32_t w = ap[NH - 1].w[0][i >> 1];
                    v = (i & 1) ? hi_f32(w) : lo_f32(w);
                } else {
                    v = acts[NH - 1][i];
                }
                selacc[i] = fmaf(ds, v, selacc[i]);
            }
        }
        // ---- per layer from the output layer down: the delta's planes, the
        // next delta, this layer's weight gradient
        float dh[HID_P / 2];
        const __bf16 *im = bwd;
        auto weight_gradient = [&](auto LC, const auto &dp, const auto &inp) {
            constexpr int L = decltype(LC)::value;
            constexpr int NBO = DB::out_p(L) / 32, NBI = DB::nbi(L);
            Rows<BF> rd[NBO];
#pragma unroll
            for (int b = 0; b < NBO; ++b) rd[b].load(id, dp, b);
#pragma unroll
            for (int c = 0; c < NBI; ++c) {
                Rows<BF> ri;
                ri.load(id, inp, c);
if constexpr (BF) {
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int b = 0; b < NBO; ++b) {
                            f32x16 &q = acc[DB::first(L) + b * NBI + c];
                            q = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd[b].k[s][0], ri.k[s][0], q, 0, 0, 0);
                        }
                } else {
#pragma unroll
                    for (int b = 0; b < NBO; ++b) {
                        f32x16 &q = acc[DB::first(L) + b * NBI + c];
                        f32x16 low = zero16();
#pragma unroll
                        for (int i = 0; i + 1 < Products<BF>::N; ++i)
#pragma unroll
                            for (int s = 0; s < 2; ++s)
                                low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    rd[b].k[s][Products<BF>::pa(i)], ri.k[s][Products<BF>::pb(i)], low, 0, 0, 0);
                        q += low;
#pragma unroll
                        for (int s = 0; s < 2; ++s)
                            q = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd[b].k[s][0], ri.k[s][0], q, 0, 0, 0);
                        // one block at a time: the small sums of two do not fit beside the rest
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        };
        {
            Planes<16, BF> dp;
            dp.set(d);
            chain_layer<32, HID_P, BF>(im, t_elems, dp, dh, lane);
            im += HID_P * 32;
            if constexpr (SEL) {
#pragma unroll
                for (int q = 0; q < HID_P / 8; ++q) {
                    const f32x4 w = *reinterpret_cast<const f32x4 *>(s_wsel + 8 * q + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dh[4 * q + e] = fmaf(ds, w[e], dh[4 * q + e]);
                }
            }
            if constexpr (BF) {
                weight_gradient(std::integral_constant<int, NH>{}, dp, ap[NH - 1]);
            } else {
                Planes<HID_P / 2, BF> ip;
                ip.set(acts[NH - 1]);
                weight_gradient(std::integral_constant<int, NH>{}, dp, ip);
            }
        }
        static_for_down<NH - 1, 1>([&](auto LC) {
            constexpr int li = decltype(LC)::value;
#pragma unroll
            for (int i = 0; i < HID_P / 2; ++i) dh[i] = on(li, i) ? dh[i] : 0.0f;
            if constexpr (PARK && li == 1) {
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < HID_P / 8; ++q) {
                    const f32x4 v = park[q * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acts[0][4 * q + e] = v[e];
                }
            }
            Planes<HID_P / 2, BF> dp;
            dp.set(dh);
            chain_layer<HID_P, HID_P, BF>(im, t_elems, dp, dh, lane);
            im += HID_P * HID_P;
            if constexpr (BF) {
                weight_gradient(LC, dp, ap[li - 1]);
            } else {
                Planes<HID_P / 2, BF> ip;
                ip.set(acts[li - 1]);
                weight_gradient(LC, dp, ip);
            }
        });
        {
#pragma unroll
            for (int i = 0; i < HID_P / 2; ++i) dh[i] = on(0, i) ? dh[i] : 0.0f;
            Planes<HID_P / 2, BF> dp;
            dp.set(dh);
            float dG[DGR / 2];
            chain_layer<HID_P, DGR, BF>(im, t_elems, dp, dG, lane);
            dG[0] = is_odd ? __uint_as_float(odd_x ? kOddInput : kOddHead) : dG[0];
            float *dst = a.dg_tiles + (size_t)t * IN0 * 32 + (lane & 31) + 4 * h * 32;
#pragma unroll
            for (int q = 0; q < DGR / 2; ++q) dst[nf(0, q) * 32] = dG[q];
            if constexpr (!BF) {
                if constexpr (PARK) {
                    FeatWords<ING, BF> again;
                    feat_load<ING, BF>(a.feat, gf, n, slot(t), h, again);
                    feat_take<IN_P, ING, BF>(again, gf, h, x);
#pragma unroll
                    for (int i = 0; i < IN_P / 2; ++i) x[i] = odd_x ? 0.0f : x[i];
                }
                xp.set(x);
            }
            weight_gradient(std::integral_constant<int, 0>{}, dp, xp);
        }
    }
    // ---- the waves' weight gradients meet in LDS (the images are no longer
    // read), one 32x32 block of 1,024 floats after the other, and go out in the
    // flat layout of the MLP weights (entries outside the real shapes dropped)
    float *sum = reinterpret_cast<float *>(smem);
    for (int w = 0; w < 4; ++w) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int g = 0; g < NDW; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float *q = sum + g * 1024 + r * 64 + lane;
                    *q = w == 0 ? acc[g][r] : *q + acc[g][r];
                }
        }
    }
    __syncthreads();
    float *out = a.dw_part + (int64_t)blockIdx.x * mlp_weights;
    static_for_down<NH, 0>([&](auto LC) {
        constexpr int L = decltype(LC)::value;
        const int out_r = L == NH ? 32 : a.width, in_r = L == 0 ? a.n_in : a.width;
        float *o = out + (L == 0 ? 0 : a.width * a.n_in + (L - 1) * a.width * a.width);
        for (int i = threadIdx.x; i < DB::blocks(L) * 1024; i += 256) {
            const int b = i >> 10, r = (i >> 6) & 15, ln = i & 63;
            const int row = 32 * (b / DB::nbi(L)) + nf(ln >> 5, r), col = 32 * (b % DB::nbi(L)) + (ln & 31);
            if (row < out_r && col < in_r) o[row * in_r + col] = sum[DB::first(L) * 1024 + i];
        }
    });
    if constexpr (SEL) {
        // the selection row (after the output layer's 32 rows): every vertex's
        // share of each feature, over the half-wave's lanes and the waves
        __syncthreads();
#pragma unroll
        for (int i = 0; i < HID_P / 2; ++i) {
            float v = selacc[i];
#pragma unroll
            for (int m = 1; m < 32; m <<= 1) v += __shfl_xor(v, m, 64);
            if ((lane & 31) == 0) sum[wave * HID_P + nf(h, i)] = v;
        }
        __syncthreads();
        if ((int)threadIdx.x < a.width) {
            float v = 0.0f;
            for (int w = 0; w < 4; ++w) v += sum[w * HID_P + threadIdx.x];
            const int64_t row = (int64_t)a.width * a.n_in + (int64_t)(NH - 1) * a.width * a.width + 32 * a.width;
            out[row + threadIdx.x] = v;
        }
    }
    // ---- the wave's vertices that are not finite
    __syncthreads();
    if (any_odd) {
        float *vin = reinterpret_cast<float *>(smem) + wave * 512, *vd = vin + 96, *va = vin + 160;
        const OddVertex<BF> ov{a.mlp, a.grad_mlp, lane};
        const int width = a.width, n_in = a.n_in;
        const int64_t out_off = (int64_t)width * n_in + (int64_t)(NH - 1) * width * width;
#pragma unroll 1
        for (int64_t tt = blockIdx.x * (int64_t)4 + wave; tt < ntiles; tt += nwaves) {
            float *col = a.dg_tiles + (size_t)tt * IN0 * 32;
            const uint32_t mark = __float_as_uint(col[lane & 31]);
            uint32_t todo = (uint32_t)__ballot(mark == kOddInput || mark == kOddHead);
            if (n - tt * 32 < 32) todo &= (1u << (n - tt * 32)) - 1u;
#pragma unroll 1
            for (; todo; todo &= todo - 1u) {
                const int j = __builtin_ctz(todo);
                const int64_t v = tt * 32 + j;
                const bool input = __shfl((int)mark, j, 64) == (int)kOddInput;
                // every lane loads the vertex; lane 0 and lane 32 hold its halves
                FeatWords<ING, BF> f;
                feat_load<ING, BF>(a.feat, gf, n, v, h, f);
                float x[IN_P / 2];
                feat_take<IN_P, ING, BF>(f, gf, h, x);
                if constexpr (PG > 0) {
                    float a7[7];
                    load_aux(io.rec, io.rec_stride, io.aux, n, v, v, a7);
                    aux_fill<IN_P, ProductShape<PG>::GF, ProductShape<PG>::SHD>(h, a7, x);
                }
                wave_lds_fence();
                if ((lane & 31) == 0)
#pragma unroll
                    for (int i = 0; i < IN_P / 2; ++i) vin[nf(h, i)] = x[i];
                wave_lds_fence();
                float y = fmaxf(ov.forward(0, width, n_in, vin), 0.0f);
                va[lane] = y;
                wave_lds_fence();
                for (int li = 1; li < NH; ++li) {
                    y = fmaxf(ov.forward((int64_t)width * n_in + (int64_t)(li - 1) * width * width, width, width, va + (li - 1) * 64), 0.0f);
                    va[li * 64 + lane] = y;
                    wave_lds_fence();
                }
                vd[lane] = ov.forward(out_off, 32, width, va + (NH - 1) * 64);
                wave_lds_fence();
                float o[16], d[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) o[i] = vd[nf(h, i)];
                const TrainInputs in = train_inputs(io, v, v);
                double l = 0.0;
                const float lv = kl_head<!BF>(o, in, true, io.invN, h, d, l);
                if (input && lane == 0) lacc += l;
                float ds = 0.0f;
                if constexpr (SEL) {
                    float cp = lane < width ? s_wsel[lane] * y : 0.0f;
#pragma unroll
                    for (int m = 1; m < 64; m <<= 1) cp += __shfl_xor(cp, m, 64);
                    const float wgt = sample_weight(in.rad, in.spdf);
                    if (wgt != 0.0f && io.bsdf) {
                        const float pb = io.bsdf[visit(io.perm, v)];
                        if (bsdf_valid(pb)) {
                            const float lpc = select_term(cp, pb, lv, -wgt * io.invN, ds);
                            if (input && lane == 0) lsel -= (double)wgt * (double)lpc;
                        }
                    }
                }
                wave_lds_fence();
                if ((lane & 31) == 0)
#pragma unroll
                    for (int i = 0; i < 16; ++i) vd[nf(h, i)] = d[i];
                wave_lds_fence();
                // from the output layer down: weights, then the delta through
                // the units that are on
                int64_t off = out_off;
                int rows = 32;
                for (int li = NH - 1; li >= 0; --li) {
                    const float *act = va + li * 64;
                    ov.weights(off, rows, width, vd, act);
                    float s = ov.back(off, rows, width, vd);
                    if constexpr (SEL)
                        if (li == NH - 1 && lane < width) {
                            unsafeAtomicAdd(a.grad_mlp + off + 32 * (int64_t)width + lane, ds * act[lane]);
                            s = fmaf(ds, s_wsel[lane], s);
                        }
                    const float dn = act[lane] > 0.0f ? s : 0.0f;
                    wave_lds_fence();
                    vd[lane] = dn;
                    wave_lds_fence();
                    rows = width;
                    off -= li > 0 ? (int64_t)width * width : (int64_t)width * n_in;
                }
                ov.weights(0, width, n_in, vd, vin);
                const float s = ov.back(0, width, n_in, vd);
                if (lane < DGR) col[lane * 32 + j] = lane < n_in ? s : 0.0f;
            }
        }
    }
    // ---- loss partials of the block (FP64)
    auto block_sum = [&](double v) {
        __syncthreads();
        red[threadIdx.x] = v;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        return red[0];
    };
    const double lsum = block_sum(lacc);
    if (threadIdx.x == 0) a.partials[blockIdx.x] = lsum;
    if constexpr (SEL) {
        const double ssum = block_sum(lsel);
        if (threadIdx.x == 0) a.partials_sel[blockIdx.x] = ssum;
    }
}

// ------------------------------------------------------------------ launch
template <int IN_P, int HID_P, int NH, int F, bool BF, int PG = 0, bool SEL = false>
static hipError_t run_train(npm_ctx *ctx, FusedArgs a, hipStream_t s)
{
    using DB = DwBlocks<IN_P, HID_P, NH>;
    if constexpr (!BF && (IN_P > 32 || (SEL && NH >= 3))) {
        return hipErrorNotSupported;      // train_tile_takes
    } else {
        // of W_0^T, the last segment, only the input-gradient rows are needed
        const int t_elems = a.bwd_elems - (DB::IN0 - (PG > 0 ? 32 : DB::IN0)) * HID_P;
        const int fwd_bytes = a.fwd_elems * (BF ? 2 : 4);
        const size_t lds = std::max<size_t>((size_t)fwd_bytes + (size_t)kPlanes<BF> * t_elems * 2 +
                                                (parks(BF, NH, SEL) ? 4 * HID_P / 2 * 64 * 4 : 0),
                                            (size_t)DB::total() * 4096);
        if (lds > kLdsBytes) return hipErrorInvalidValue;
        auto k = k_train_tile<IN_P, HID_P, NH, F, BF, PG, SEL>;
        const hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        const int count = (int)(ctx->net.lay.n_params - ctx->net.lay.grid_params);
        hipLaunchKernelGGL(k, dim3(train_blocks(a.n)), dim3(256), lds, s, a, count, fwd_bytes, t_elems);
        return hipGetLastError();
    }
}

hipError_t train_tile(npm_ctx *ctx, const FusedArgs &args, hipStream_t s)
{
    FusedArgs a = args;
    hipError_t e = hipSuccess;
    NPM_FUSED_RUN(run_train);
    return e;
}

}  // namespace npm
