// Fused queries of the NPM hot path (see k_fused.hip for the tile scheme).
#include <type_traits>

#include "fused_launch.h"

namespace npm {

// SEL: the network has the selection output (its logit is computed from the
// last hidden layer and the row staged in LDS; a.sel receives sigmoid of it).
template <int IN_P, int HID_P, int NH, int F, bool BF, int PG, bool SEL = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_query_fused(FusedArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ uint32_t s_off[NPM_MAX_LEVELS];
    __shared__ int s_res[NPM_MAX_LEVELS];
    __shared__ __attribute__((aligned(16))) float s_wsel[SEL ? HID_P : 4];
    {
        const int bytes = a.fwd_elems * (BF ? 2 : 4);
        for (int i = threadIdx.x; i < bytes / 16; i += blockDim.x)
            reinterpret_cast<f32x4 *>(smem)[i] = reinterpret_cast<const f32x4 *>(a.img)[i];
        stage_levels(a.g, s_off, s_res);
        if constexpr (SEL)
            for (int i = threadIdx.x; i < HID_P; i += blockDim.x)
                s_wsel[i] = i < a.width ? a.wsel[i] : 0.0f;
    }
    __syncthreads();
    const GridView gv = grid_view(a.g, s_off, s_res, a.grid32, a.grid16);
    const QueryIO io{a.n, a.pos, a.dir, a.lobes, a.pdf, a.sdir, a.spdf_out, a.seed, a.sid,
                     a.perm, a.qstage, a.rec, a.aux, a.rec_stride, a.sel, s_wsel};
    const int lane = threadIdx.x & 63;
    const int64_t ntiles = (a.n + 31) / 32;
    const int wpb = blockDim.x / 64, wave = threadIdx.x >> 6;
    if (gridDim.x % 8 == 0) {
        // Workgroups are dispatched to the eight XCDs in turn (block b on XCD
        // b mod 8), each XCD with its own L2: give each XCD a contiguous
        // eighth of the tiles, so that the tiles it runs at one time are
        // neighbours in the batch's order and share grid lines in its L2
        // (FP32 query 0.56 -> 0.53 ms at 2^20 vertices).  Any placement of
        // the blocks still covers every tile once.
        const int64_t xcd = blockIdx.x % 8, bl = blockIdx.x / 8;
        const int64_t wpx = (int64_t)(gridDim.x / 8) * wpb, span = (ntiles + 7) / 8;
        const int64_t t0 = xcd * span, t1 = t0 + span < ntiles ? t0 + span : ntiles;
        for (int64_t t = t0 + bl * wpb + wave; t < t1; t += wpx)
            query_tile<IN_P, HID_P, NH, F, BF, PG, SEL>(gv, smem, io, t, lane);
    } else {
        const int64_t nwaves = (int64_t)gridDim.x * wpb;
        for (int64_t t = blockIdx.x * (int64_t)wpb + wave; t < ntiles; t += nwaves)
            query_tile<IN_P, HID_P, NH, F, BF, PG, SEL>(gv, smem, io, t, lane);
    }
}

// Queries whose grid features were encoded level by level before
// (k_encode.hip): MLP, mappings, pdf and sample of the vertices in the
// caller's order, features and outputs streamed.  The next tile's features and
// directions are loaded while a tile is evaluated.
template <int IN_P, int HID_P, int NH, int F, bool BF, int PG, bool SEL = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_query_feat(FusedArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ __attribute__((aligned(16))) float s_wsel[SEL ? HID_P : 4];
    {
        const int bytes = a.fwd_elems * (BF ? 2 : 4);
        for (int i = threadIdx.x; i < bytes / 16; i += blockDim.x)
            reinterpret_cast<f32x4 *>(smem)[i] = reinterpret_cast<const f32x4 *>(a.img)[i];
        if constexpr (SEL)
            for (int i = threadIdx.x; i < HID_P; i += blockDim.x)
                s_wsel[i] = i < a.width ? a.wsel[i] : 0.0f;
    }
    __syncthreads();
    constexpr int ING = PG > 0 ? ProductShape<PG>::GF : IN_P;
    QueryIO io{a.n, a.pos, a.dir, a.lobes, a.pdf, a.sdir, a.spdf_out, a.seed, a.sid,
               nullptr, nullptr, nullptr, a.aux, a.rec_stride, a.sel, s_wsel};
    const int lane = threadIdx.x & 63, h = lane >> 5;
    int64_t n = a.n;
    const int64_t ntiles = (n + 31) / 32;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / 64);
    const int gf = a.g.n_levels * F;
    auto vertex = [&](int64_t t) {
        const int64_t v = t * 32 + (lane & 31);
        return v < n ? v : n - 1;
    };
    int64_t t = blockIdx.x * (int64_t)(blockDim.x / 64) + (threadIdx.x >> 6);
    if (t >= ntiles) return;
    FeatWords<ING, BF> fw;
    float w[3] = {0.0f, 0.0f, 0.0f};
    auto load = [&](int64_t tt) {
        const int64_t v = vertex(tt);
        feat_load<ING, BF>(a.feat, gf, n, v, h, fw);
        if (a.pdf) { w[0] = a.dir[v]; w[1] = a.dir[n + v]; w[2] = a.dir[2 * n + v]; }
    };
    load(t);
    for (; t < ntiles; t += nwaves) {
        // the array strides are products of n: formed anew for each tile by
        // the scalar unit rather than kept (they spilled to vector lanes)
        asm volatile("" : "+s"(n));
        io.n = n;
        const int64_t v = vertex(t);
        float x[IN_P / 2];
        feat_take<IN_P, ING, BF>(fw, gf, h, x);
        const float wx = w[0], wy = w[1], wz = w[2];
        if constexpr (PG > 0) {
            float a7[7];
            load_aux(nullptr, 8, a.aux, n, v, v, a7);
            aux_fill<IN_P, ProductShape<PG>::GF, ProductShape<PG>::SHD>(h, a7, x);
        }
        if (t + nwaves < ntiles) load(t + nwaves);
        float o[16], cp = 0.0f;
        mlp_forward<IN_P, HID_P, NH, BF, false, SEL>(smem, x, nullptr, o, lane, s_wsel, &cp);
        query_head<SEL>(io, v, t * 32 + (lane & 31) < n, nullptr, lane, o, cp, wx, wy, wz);
    }
}

// A layer's weights as matrix-instruction operands in registers: the packed
// image's groups of one lane (device_math.h), and the layer's product with
// the same instructions in the same order as mfma_layer_f32 / _bf16.
template <bool BF, int IN_P, int OUT_P> struct LayerRegs {
    static constexpr int NB = OUT_P / 32, NG = IN_P / (BF ? 16 : 8);
    using GT = typename std::conditional<BF, bf16x8, f32x4>::type;
    GT w[NB][NG];

    __device__ __forceinline__ void load(const void *img, int lane)
    {
        const GT *p = reinterpret_cast<const GT *>(img) + lane;
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int b = 0; b < NB; ++b) w[b][g] = p[(b * NG + g) * 64];
    }
    __device__ __forceinline__ void apply(const float *x, float *y) const
    {
        f32x16 acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if constexpr (BF) {
                bf16x8 xb;
#pragma unroll
                for (int e = 0; e < 8; ++e) xb[e] = (__bf16)x[8 * g + e];
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[b][g], xb, acc[b], 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[b][g][e], x[4 * g + e], acc[b],
                                                                      0, 0, 0);
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) y[16 * b + v] = acc[b][v];
    }
};

// Queries of at most a tile per SIMD, where a call's latency counts: one wave
// per block and tile, all weights loaded from the packed image straight into
// registers (a wave has 512) beside the tile's features, so that one memory
// latency covers both and no LDS staging, barrier or weight read stands
// between the layers.  GATHER: the features are gathered here, every corner
// of every level in flight at once; otherwise they were encoded level by level
// before (a.feat).
template <int IN_P, int HID_P, int NH, int F, bool BF, int PG, bool SEL, bool GATHER>
__global__ __launch_bounds__(64) void k_query_small(FusedArgs a)
{
    __shared__ __attribute__((aligned(16))) float s_wsel[SEL ? HID_P : 4];
    constexpr int ING = PG > 0 ? ProductShape<PG>::GF : IN_P;
    constexpr size_t ESZ = BF ? 2 : 4;
    // of a tile's two blocks one answers the lobes and the pdf, one the samples
    const int part = a.halves == 2 ? (int)(blockIdx.x & 1) : -1;
    const QueryIO io{a.n, a.pos, a.dir, part == 1 ? nullptr : a.lobes, part == 1 ? nullptr : a.pdf,
                     part == 0 ? nullptr : a.sdir, part == 0 ? nullptr : a.spdf_out, a.seed, a.sid,
                     nullptr, nullptr, nullptr, a.aux, a.rec_stride, part == 1 ? nullptr : a.sel,
                     s_wsel};
    const int lane = threadIdx.x & 63, h = lane >> 5, j = lane & 31;
    const int64_t n = a.n;
    const int64_t slot = (blockIdx.x / a.halves) * (int64_t)a.tile_v + min(j, a.tile_v - 1);
    const int64_t v = slot < n ? slot : n - 1;
    const bool valid = j < a.tile_v && slot < n;
    const int gf = a.g.n_levels * F;
    FeatWords<ING, BF> fw;
    TileGather<ING, F, BF> tg;
    GridView gv{};
    gv.n_levels = a.g.n_levels;
    gv.table_mask = a.g.table_mask;
    gv.g32 = a.grid32;
    gv.g16 = a.grid16;
    float px = 0.0f, py = 0.0f, pz = 0.0f;
    if constexpr (GATHER) {
        px = a.pos[v]; py = a.pos[n + v]; pz = a.pos[2 * n + v];
    } else {
        feat_load<ING, BF>(a.feat, gf, n, v, h, fw);
    }
    LayerRegs<BF, IN_P, HID_P> l0;
    LayerRegs<BF, HID_P, HID_P> lh[NH > 1 ? NH - 1 : 1];
    LayerRegs<BF, HID_P, 32> lo;
    const char *img = reinterpret_cast<const char *>(a.img);
    float wx = 0.0f, wy = 0.0f, wz = 0.0f;
    if (io.pdf) { wx = a.dir[v]; wy = a.dir[n + v]; wz = a.dir[2 * n + v]; }
    l0.load(img, lane);
#pragma unroll
    for (int i = 0; i < NH - 1; ++i) lh[i].load(img + (size_t)(IN_P + i * HID_P) * HID_P * ESZ, lane);
    lo.load(img + (size_t)(IN_P + (NH - 1) * HID_P) * HID_P * ESZ, lane);
    if constexpr (SEL) {
        for (int i = threadIdx.x; i < HID_P; i += 64) s_wsel[i] = i < a.width ? a.wsel[i] : 0.0f;
        __syncthreads();
    }
    // every load above is issued before anything waits for one
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (GATHER) {
        // the levels from the kernel's arguments: both half-waves' are known at
        // compile time, so that no staged table is read
        using TG = TileGather<ING, F, BF>;
        encode_issue<ING, F, BF>(gv, [&](int q) {
            const int l0_ = (8 * (q / TG::PER)) / F + q % TG::PER;
            const int l1_ = (8 * (q / TG::PER) + 4) / F + q % TG::PER;
            const int a0 = l0_ < a.g.n_levels ? l0_ : 0, a1 = l1_ < a.g.n_levels ? l1_ : 0;
            return LevelRef{h ? a.g.res[a1] : a.g.res[a0], h ? a.g.offset[a1] : a.g.offset[a0],
                            (bool)((a.g.hashed_mask >> (h ? a1 : a0)) & 1u)};
        }, px, py, pz, tg);
        __builtin_amdgcn_sched_barrier(0);
    }
    float x[IN_P / 2];
    if constexpr (GATHER) encode_finish<IN_P, ING, F, BF>(gv, h, tg, x);
    else feat_take<IN_P, ING, BF>(fw, gf, h, x);
    if constexpr (PG > 0) {
        float a7[7];
        load_aux(nullptr, 8, a.aux, n, v, v, a7);
        aux_fill<IN_P, ProductShape<PG>::GF, ProductShape<PG>::SHD>(h, a7, x);
    }
    float p[HID_P / 2], q[HID_P / 2], o[16], cp = 0.0f;
    l0.apply(x, p);
#pragma unroll
    for (int i = 0; i < HID_P / 2; ++i) p[i] = fmaxf(p[i], 0.0f);
#pragma unroll
    for (int li = 1; li < NH; ++li) {
        lh[li - 1].apply(p, q);
#pragma unroll
        for (int i = 0; i < HID_P / 2; ++i) p[i] = fmaxf(q[i], 0.0f);
    }
    if constexpr (SEL) cp = select_logit<HID_P>(s_wsel, p, h);
    lo.apply(p, o);
    query_head<SEL>(io, v, valid, nullptr, lane, o, cp, wx, wy, wz);
}

// Moves the staged outputs of a spatially ordered query to the caller's SoA
// buffers: vertex i (coalesced writes) reads its 160-byte slot inv[i].
__global__ __launch_bounds__(256) void k_query_unstage(int64_t n, const uint32_t *__restrict__ inv,
                                                       const float *__restrict__ stage,
                                                       float *__restrict__ lobes,
                                                       float *__restrict__ pdf,
                                                       float *__restrict__ sdir,
                                                       float *__restrict__ spdf,
                                                       float *__restrict__ sel)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(stage + (size_t)inv[i] * kStageFloats);
    f32x4 r[kStageFloats / 4];
#pragma unroll
    for (int q = 0; q < kStageFloats / 4; ++q) r[q] = src[q];
    const float *c = reinterpret_cast<const float *>(r);
    if (lobes)
#pragma unroll
        for (int k = 0; k < kLobes; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                lobes[(int64_t)(q * kLobes + k) * n + i] = c[20 * (k & 1) + 4 * (k >> 1) + q];
    if (pdf) pdf[i] = c[kStagePdf];
    if (sdir)
#pragma unroll
        for (int d = 0; d < 3; ++d) sdir[(int64_t)d * n + i] = c[kStageSdir + d];
    if (spdf) spdf[i] = c[kStageSpdf];
    if (sel) sel[i] = c[kStageSel];
}

// ------------------------------------------------------------------ launch
template <int IN_P, int HID_P, int NH, int F, bool BF, int PG = 0, bool SEL = false>
static hipError_t run_query(npm_ctx *ctx, FusedArgs a, hipStream_t s)
{
    const int64_t tiles = (a.n + 31) / 32;
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((tiles + 3) / 4, 2048));
    const size_t lds = (size_t)a.fwd_elems * (BF ? 2 : 4);
    auto k = k_query_fused<IN_P, HID_P, NH, F, BF, PG, SEL>;
    const hipError_t e = hipFuncSetAttribute((const void *)k,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(256), lds, s, a);
    return hipGetLastError();
}

template <int IN_P, int HID_P, int NH, int F, bool BF, int PG = 0, bool SEL = false>
static hipError_t run_query_feat(npm_ctx *ctx, FusedArgs a, hipStream_t s)
{
    const int64_t tiles = (a.n + 31) / 32;
    const size_t lds = (size_t)a.fwd_elems * (BF ? 2 : 4);
    // as many blocks as run at once (three waves per SIMD, or what the LDS holds)
    const int per_cu = std::min(3, (int)((160 * 1024) / (lds + 512)));
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((tiles + 3) / 4, 256 * per_cu));
    auto k = k_query_feat<IN_P, HID_P, NH, F, BF, PG, SEL>;
    const hipError_t e = hipFuncSetAttribute((const void *)k,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(blocks), dim3(256), lds, s, a);
    return hipGetLastError();
}

template <int IN_P, int HID_P, int NH, int F, bool BF, int PG = 0, bool SEL = false>
static hipError_t run_query_small(npm_ctx *ctx, FusedArgs a, hipStream_t s)
{
    // Up to a block per CU the tiles are split further: half-filled ones, whose
    // gathers are half as many requests of a CU, and the answers of a tile that
    // asks for both kinds shared by two blocks, which repeat the network.  16
    // levels, 2^19 entries, FP32: 1,000 vertices 18.9 -> 17.6 us, 2,048 19.2 ->
    // 19.0, but 4,096 20.1 -> 22.5.
    const bool tiny = a.n <= kQueryTiny, both = (a.lobes || a.pdf || a.sel) && (a.sdir || a.spdf_out);
    a.tile_v = tiny ? 16 : 32;
    a.halves = tiny && both ? 2 : 1;
    const dim3 grid((unsigned)((a.n + a.tile_v - 1) / a.tile_v * a.halves));
    if (a.feat)
        hipLaunchKernelGGL((k_query_small<IN_P, HID_P, NH, F, BF, PG, SEL, false>), grid, dim3(64), 0,
                           s, a);
    else
        hipLaunchKernelGGL((k_query_small<IN_P, HID_P, NH, F, BF, PG, SEL, true>), grid, dim3(64), 0,
                           s, a);
    return hipGetLastError();
}

hipError_t fused_query(npm_ctx *ctx, int64_t n, const float *pos, const float *aux,
                       const float *dir, uint64_t seed, uint32_t stream_id, float *lobes,
                       float *pdf, float *sdir, float *spdf, const uint32_t *perm,
                       const uint32_t *inv, const float *rec, float *stage, hipStream_t s,
                       float *sel, void *feat)
{
    FusedArgs a = fused_args(ctx, n, pos);
    a.aux = aux;
    const Weights w = query_weights(ctx);
    a.grid32 = w.grid32;
    a.grid16 = (const __half *)w.grid16;
    a.img = ctx->net.cfg.precision == NPM_PREC_BF16 ? w.img16 : (const void *)w.img;
    a.dir = dir;
    a.seed = seed;
    a.sid = stream_id;
    a.lobes = lobes;
    a.pdf = pdf;
    a.sdir = sdir;
    a.spdf_out = spdf;
    a.perm = perm;
    a.qstage = perm ? stage : nullptr;
    a.rec = perm ? rec : nullptr;
    a.wsel = selection_row(ctx, w.grid32);
    a.sel = sel;
    hipError_t e = hipSuccess;
    int tok;
    if (feat) {
        a.feat = feat;
        const bool b16 = ctx->net.cfg.precision == NPM_PREC_BF16;
        timed_begin(ctx, "query_encode", s, &tok);
        e = launch_grid_encode(ctx->net.grid, n, pos, nullptr, 0, w.grid32, w.grid16, b16, feat, s);
        timed_end(ctx, tok, s);
        if (e != hipSuccess) return e;
        timed_begin(ctx, "fused_query", s, &tok);
        if (n <= kQuerySmall) NPM_FUSED_RUN(run_query_small);
        else NPM_FUSED_RUN(run_query_feat);
        timed_end(ctx, tok, s);
        return e;
    }
    timed_begin(ctx, "fused_query", s, &tok);
    if (!perm && n <= kQuerySmall) NPM_FUSED_RUN(run_query_small);
    else NPM_FUSED_RUN(run_query);
    timed_end(ctx, tok, s);
    if (e != hipSuccess || !perm) return e;
    timed_begin(ctx, "query_unstage", s, &tok);
    hipLaunchKernelGGL(k_query_unstage, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, inv,
                       stage, lobes, pdf, sdir, spdf, sel);
    timed_end(ctx, tok, s);
    return hipGetLastError();
}

}  // namespace npm
