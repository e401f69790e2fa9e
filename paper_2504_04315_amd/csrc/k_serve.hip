// Persistent multi-session kernels of the serving form.  One launch covers
// every query (or every training batch) of a round, whatever the session:
// blocks pull chunks of tiles from a device counter, find the request a
// chunk belongs to, and restage that session's weight images and level table
// into LDS only when the session changes.  The per-tile work is exactly the
// fused path's (fused_tiles.h), so a request gives the same result alone or
// in a mix (queries bit for bit; training up to the order of atomic adds).
#include <cstring>

#include "fused_tiles.h"
#include "serve_internal.h"

namespace npm {

// Device descriptor of one request of a round.
struct DevReq {
    GridDesc g;
    const __half *grid16;
    const void *img;             // BF16 images of the session: forward then backward
    float *grad;                 // the session's gradient buffer (train)
    float *dgt;                  // per-tile dG of the request (train), or null: scattered here
    const float *pos, *dir, *rad, *spdf;
    float *lobes, *pdf, *sdir, *spdf_out;
    double *loss;                // loss slot of the round buffer (train)
    int64_t n;
    int64_t mlp_off;             // first MLP weight in the flat parameters
    uint64_t seed;
    uint32_t sid;
    int32_t skey;                // session identity (restaging test)
    int32_t chunk_begin;         // first chunk of the request in its launch
    int32_t fwd_elems, bwd_elems, n_in, width;
    float invN;
};

// A round launches one kernel per (network shape, request kind) group: at
// most two kinds for each of the kServeShapes shapes serve_supports admits.
constexpr int kServeShapes = 4;
constexpr int kMaxRoundGroups = 2 * kServeShapes;

struct RoundHdr {
    uint32_t counter[kMaxRoundGroups];   // chunk counters, one per launch (zero at upload)
    int32_t n_req;
    int32_t pad[3];
};
static_assert(sizeof(RoundHdr) <= 64, "the round header sits in the first 64 bytes");

constexpr int kQueryChunkTiles = 4;    // one tile per wave
// Training chunks hold kTrainWaves tiles for each round of the block's waves, up
// to four rounds (train_chunk_tiles).
constexpr int kTrainWaves = 4;
constexpr int kServeRows = 32;         // dG rows of a tile

// Bytes of a training block's LDS exchange buffer (BF16, after the images).
template <int IN_P, int HID_P, int NH>
constexpr size_t serve_xch_bytes()
{
    using Plan = BlockPlan<IN_P, HID_P, NH, 4>;
    return ((size_t)Plan::max_rows() * Plan::xs(true) * 2 + 15) / 16 * 16;
}

// Request of chunk c among [r0, r1): the last one whose chunk_begin <= c.
__device__ __forceinline__ int find_request(const int *s_begin, int r0, int r1, int c)
{
    int lo = r0, hi = r1 - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_begin[mid] <= c) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ void stage_bytes(char *dst, const void *src, int bytes)
{
    for (int i = threadIdx.x; i < bytes / 16; i += blockDim.x)
        reinterpret_cast<f32x4 *>(dst)[i] = reinterpret_cast<const f32x4 *>(src)[i];
}

// Queries of requests [r0, r1) of the round; `which` selects the counter.
template <int IN_P, int HID_P, int NH, int F>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_serve_query(RoundHdr *hdr, const DevReq *__restrict__ reqs,
                                                     int r0, int r1, int n_chunks, int which)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ uint32_t s_off[NPM_MAX_LEVELS];
    __shared__ int s_res[NPM_MAX_LEVELS];
    __shared__ int s_begin[kMaxRoundRequests];
    __shared__ int s_chunk;
    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) s_begin[i] = reqs[i].chunk_begin;
    int staged = -1;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_chunk = (int)atomicAdd(&hdr->counter[which], 1u);
        __syncthreads();
        const int chunk = s_chunk;
        if (chunk >= n_chunks) break;
        const int r = find_request(s_begin, r0, r1, chunk);
        const DevReq &q = reqs[r];
        if (q.skey != staged) {
            stage_bytes(smem, q.img, q.fwd_elems * 2);
            stage_levels(q.g, s_off, s_res);
            staged = q.skey;
            __syncthreads();
        }
        const int64_t t = (int64_t)(chunk - q.chunk_begin) * kQueryChunkTiles + wave;
        if (t * 32 < q.n) {
            const GridView gv = grid_view(q.g, s_off, s_res, nullptr, q.grid16);
            const QueryIO io{q.n, q.pos, q.dir, q.lobes, q.pdf, q.sdir, q.spdf_out, q.seed, q.sid};
            query_tile<IN_P, HID_P, NH, F, true>(gv, smem, io, t, lane);
        }
    }
}

// Training batches of requests [r0, r1), the fused path's block-cooperative
// scheme (fused_tiles.h): a chunk is chunk_tiles tiles of one request, run as
// rounds of one tile per wave; per layer the waves exchange deltas and inputs
// in LDS and each wave accumulates its share of the weight-gradient blocks over
// the round's 128 vertices.  The shares stay in registers while the block's
// chunks belong to one request (its chunks are handed out in order, so a block
// usually takes several in a row) and are added into that session's gradient
// with FP32 atomics when the request changes and at the end: per block and
// request, one add per weight.
//
// Each tile's dG goes to the request's buffer, for the chunked and binned
// scatters of the per-session path, which sum in LDS (integer fixed point).
// Scattered from here, 16 levels of 36,868 unordered vertices took 2.4 M line
// requests of memory-side atomics from 73 blocks: 263 us, now 74 with two
// rounds of tiles a chunk, so that every CU has a block, and 100 for the
// scatters.  A request whose dG found no room in the server's scratch is scattered
// tile by tile from the wave's LDS buffer, its coarse levels through a 32-bit
// fixed-point window, the rest by FP32 atomics.
template <int IN_P, int HID_P, int NH, int F>
__global__ __launch_bounds__(256) void k_serve_train(RoundHdr *hdr, const DevReq *__restrict__ reqs,
                                                     int r0, int r1, int n_chunks, int which,
                                                     int chunk_tiles, int img_bytes_max)
{
    constexpr int WV = kTrainWaves;
    using Plan = BlockPlan<IN_P, HID_P, NH, WV>;
    constexpr int IN0 = Plan::IN0;
    constexpr int XS = Plan::xs(true);
    constexpr int NS = Plan::slots();
    constexpr int WIN_PTS = (HID_P - IN0) * kStride / (2 * F);
    static_assert(Plan::scratch_fits(true), "split blocks' sums fit in the exchange buffer");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ uint32_t s_off[NPM_MAX_LEVELS];
    __shared__ int s_res[NPM_MAX_LEVELS];
    __shared__ int s_begin[kMaxRoundRequests];
    __shared__ int s_chunk;
    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) s_begin[i] = reqs[i].chunk_begin;
    int staged = -1, cur = -1;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
    const size_t img_al = ((size_t)img_bytes_max + 15) / 16 * 16;
    __bf16 *xb = reinterpret_cast<__bf16 *>(smem + img_al);
    float *tbuf = reinterpret_cast<float *>(smem + img_al + serve_xch_bytes<IN_P, HID_P, NH>()) +
                  wave * HID_P * kStride;
    f32x16 acc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[k][v] = 0.0f;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_chunk = (int)atomicAdd(&hdr->counter[which], 1u);
        __syncthreads();
        const int chunk = s_chunk;
        const int r = chunk < n_chunks ? find_request(s_begin, r0, r1, chunk) : -1;
        if (r != cur) {
            if (cur >= 0) {
                const DevReq &c = reqs[cur];
                dw_write<Plan, NH, WV, true>(c.grad + c.mlp_off, c.n_in, c.width, wave, acc, lane,
                                             reinterpret_cast<float *>(xb));
#pragma unroll
                for (int k = 0; k < NS; ++k)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[k][v] = 0.0f;
            }
            cur = r;
        }
        if (chunk >= n_chunks) break;
        const DevReq &q = reqs[r];
        if (q.skey != staged) {
            stage_bytes(smem, q.img, (q.fwd_elems + q.bwd_elems) * 2);
            stage_levels(q.g, s_off, s_res);
            staged = q.skey;
            __syncthreads();
        }
        const GridView gv = grid_view(q.g, s_off, s_res, nullptr, q.grid16);
        const TrainIO io{q.n, q.pos, q.dir, q.rad, q.spdf, q.grad, q.invN, nullptr};
        const char *fwd = smem;
        const char *bwd = smem + (size_t)q.fwd_elems * 2;
        const int64_t ntiles = (q.n + 31) / 32;
        const int64_t c0 = (int64_t)(chunk - q.chunk_begin) * chunk_tiles;
        double lacc = 0.0;
        for (int rr = 0; rr < chunk_tiles / WV; ++rr) {
            // every wave runs every round of the chunk (the phases
            // synchronise); a wave past the batch takes a tile with no valid
            // vertex
            const int64_t t0 = c0 + (int64_t)rr * WV;
            if (t0 >= ntiles) break;                    // uniform over the block
            const int64_t t = t0 + wave;
            const int64_t v = t * 32 + (lane & 31);
            const bool valid = v < q.n;
            const int64_t vs = valid ? v : q.n - 1;
            const TrainInputs in = train_inputs(io, vs, vs);
            float x[IN0 / 2];
            tile_input<IN_P, F, true, 0>(gv, io, in, vs, vs, h, x);
            float acts[NH][HID_P / 2], o[16], d[16];
            mlp_forward<IN_P, HID_P, NH, true, true>(fwd, x, acts, o, lane);
            kl_head<false>(o, in, valid, io.invN, h, d, lacc);
            // ---- output layer's dW, then the delta chain
            float dh[HID_P / 2];
            dw_phase<Plan, NH, WV, XS>(xb, d, acts[NH - 1], wave, acc, lane);
            layer<true, 32, HID_P>(bwd, d, dh, lane);
            __syncthreads();
            const char *im = bwd + (size_t)HID_P * 32 * 2;
            static_for_down<NH - 1, 1>([&](auto LC) {
                constexpr int li = decltype(LC)::value;
#pragma unroll
                for (int i = 0; i < HID_P / 2; ++i) dh[i] = acts[li][i] > 0.0f ? dh[i] : 0.0f;
                dw_phase<Plan, li, WV, XS>(xb, dh, acts[li - 1], wave, acc, lane);
                float nd[HID_P / 2];
                layer<true, HID_P, HID_P>(im, dh, nd, lane);
                im += (size_t)HID_P * HID_P * 2;
#pragma unroll
                for (int i = 0; i < HID_P / 2; ++i) dh[i] = nd[i];
                __syncthreads();
            });
#pragma unroll
            for (int i = 0; i < HID_P / 2; ++i) dh[i] = acts[0][i] > 0.0f ? dh[i] : 0.0f;
            dw_phase<Plan, 0, WV, XS>(xb, dh, x, wave, acc, lane);
            float dG[IN0 / 2];
            layer<true, HID_P, IN0>(im, dh, dG, lane);
            __syncthreads();
            if (t < ntiles && q.dgt) {
                float *dst = q.dgt + (size_t)t * kServeRows * 32 + (lane & 31);
#pragma unroll
                for (int i = 0; i < IN0 / 2; ++i) dst[nf(h, i) * 32] = dG[i];
            } else if (t < ntiles) {
                // the tile's grid scatter from the wave's own buffer
                float lo[3], hi[3];
                if constexpr (WIN_PTS > 0) tile_bbox(in.px, in.py, in.pz, lo, hi);
                wave_lds_fence();
                t32_to_lds<IN0 / 2>(tbuf, dG, lane);
                wave_lds_fence();
                scatter_tile<F, WIN_PTS>(gv, tbuf, io.pos, nullptr, q.n, t, lane, io.grad, lo,
                                              hi, reinterpret_cast<int *>(tbuf + IN0 * kStride));
            }
        }
        // FP64 loss of the wave (half 0 holds it), one atomic per wave
        double l = lacc;
        for (int off = 16; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
        if (lane == 0 && l != 0.0) atomicAdd(q.loss, l);
    }
}

// stats[0] = loss / n for each training request of the round.
__global__ void k_serve_finish(const DevReq *__restrict__ reqs, const double *const *stats_out,
                               int r0, int r1)
{
    const int i = r0 + blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= r1) return;
    double *st = const_cast<double *>(stats_out[i]);
    if (st) st[0] = *reqs[i].loss * (1.0 / (double)reqs[i].n);
}

// ------------------------------------------------------------------ host side
struct RoundLayout {
    size_t hdr = 0, reqs = 0, loss = 0, stats = 0, total = 0;
};

static RoundLayout round_layout(int requests)
{
    RoundLayout L;
    L.hdr = 0;
    L.reqs = 64;
    L.loss = L.reqs + sizeof(DevReq) * requests;
    L.stats = L.loss + sizeof(double) * requests;
    L.total = (L.stats + sizeof(double *) * requests + 15) / 16 * 16;
    return L;
}

// The round's descriptors from pinned host memory.  A copy through the runtime
// went to a copy engine, whose queues it opened in the middle of the first loads:
// 6.3 ms each, twice, with 2^20 vertices of requests waiting.
__global__ void k_round_upload(uint4 *__restrict__ dst, const uint4 *__restrict__ src, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t round_buffers_init(RoundBuffers *b)
{
    const RoundLayout L = round_layout(kMaxRoundRequests);
    b->bytes = L.total;
    hipError_t e = hipHostMalloc(&b->host, L.total, hipHostMallocDefault);
    if (e == hipSuccess) e = hipMalloc(&b->dev, L.total);
    return e;
}

void round_buffers_free(RoundBuffers *b)
{
    if (b->host) (void)hipHostFree(b->host);
    if (b->dev) (void)hipFree(b->dev);
    b->host = b->dev = nullptr;
}

hipError_t serve_lanes_init(ServeLanes *l)
{
    hipError_t e = hipStreamCreateWithFlags(&l->side, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&l->fork, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&l->join, hipEventDisableTiming);
    return e;
}

void serve_lanes_free(ServeLanes *l)
{
    if (l->side) (void)hipStreamDestroy(l->side);
    if (l->fork) (void)hipEventDestroy(l->fork);
    if (l->join) (void)hipEventDestroy(l->join);
    for (ServeBuf *b : {&l->dgt, &l->cnt, &l->items})
        if (b->p) (void)hipFree(b->p);
    *l = ServeLanes{};
}

// The binned levels of a training batch of n vertices (in its own order) of the
// network, or false.
static bool request_bins(const Net &net, int64_t n, BinDesc *b)
{
    const int mode = net.cfg.scatter_mode;
    return mode != NPM_SCATTER_ATOMIC && (mode == NPM_SCATTER_BINNED || n >= kBinMinBatch) &&
           bin_plan(net, n, false, b) && (mode == NPM_SCATTER_BINNED || b->nbins >= kBinMinBins);
}

static size_t dgt_words(int64_t n) { return (size_t)((n + 31) / 32) * kServeRows * 32; }

void serve_lanes_size(ServeLanes *l, int64_t vertices, int64_t bytes,
                      const std::vector<Net> &nets, hipStream_t s)
{
    ServeBuf *const bufs[3] = {&l->dgt, &l->cnt, &l->items};
    bool drained = false;
    if (nets.empty()) vertices = bytes = 0;       // nothing to scatter: given back
    bytes = std::max<int64_t>(bytes, 0);
    for (;; vertices /= 2) {
        size_t want[3] = {0, 0, 0};
        if (vertices >= kMinLaneVertices) {
            // every request of a round may end in a part of a tile
            want[0] = dgt_words(vertices + 32 * kMaxRoundRequests);
            for (const Net &net : nets) {
                BinDesc b;
                if (!request_bins(net, vertices, &b)) continue;
                want[1] = std::max(want[1], bin_count_words(b));
                want[2] = std::max(want[2], bin_item_words(b, net.grid.feat));
            }
        }
        if ((int64_t)(want[0] + want[1] + want[2]) * 4 > bytes) continue;
        // what is there stays unless it is too small, or more than `bytes`
        bool fits = true, over = (int64_t)(l->dgt.words + l->cnt.words + l->items.words) * 4 > bytes;
        for (int i = 0; i < 3; ++i) fits = fits && bufs[i]->words >= want[i];
        if (fits && !over) return;
        if (!drained && hipStreamSynchronize(s) != hipSuccess) return;
        drained = true;
        bool ok = true;
        for (int i = 0; i < 3; ++i) {
            if (bufs[i]->p) (void)hipFree(bufs[i]->p);
            *bufs[i] = ServeBuf{};
        }
        for (int i = 0; i < 3 && ok; ++i) {
            if (want[i] == 0) continue;
            ok = hipMalloc((void **)&bufs[i]->p, want[i] * 4) == hipSuccess;
            if (ok) {
                bufs[i]->words = want[i];
            } else {
                bufs[i]->p = nullptr;
                (void)hipGetLastError();
            }
        }
        if (ok || vertices == 0) return;
    }
}

static int shape_key(const Net &net)
{
    const MlpDesc &m = net.mlp;
    return net.grid.feat * 1000 + (m.in_p == 32) * 100 + (m.hid_p == 64) * 10 + m.n_hidden;
}

bool serve_supports(const npm_config *cfg)
{
    Net net;
    std::string err;
    if (describe(cfg, &net, &err) != NPM_OK) return false;
    if (cfg->sh_degree != 0) return false;
    const int k = shape_key(net);
    static_assert(kServeShapes == 4, "the shapes listed here and in launch_shape");
    return k == 2113 || k == 4012 || k == 2002 || k == 2112;
}

template <int IN_P, int HID_P, int NH, int F>
static hipError_t launch_group(RoundHdr *hdr, const DevReq *reqs, int r0, int r1, int chunks,
                               int which, bool train, int chunk_tiles, bool tile_scatter,
                               int img_bytes_max, hipStream_t s)
{
    if (chunks <= 0) return hipSuccess;
    const int blocks = std::max(1, std::min(chunks, 1024));
    if (!train) {
        auto k = k_serve_query<IN_P, HID_P, NH, F>;
        const int lds = img_bytes_max;
        const hipError_t e = hipFuncSetAttribute((const void *)k,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3(blocks), dim3(256), lds, s, hdr, reqs, r0, r1, chunks, which);
    } else {
        auto k = k_serve_train<IN_P, HID_P, NH, F>;
        // images, the exchange buffer, and where a request is scattered tile by
        // tile the four waves' buffers for that
        const int lds = (img_bytes_max + 15) / 16 * 16 + (int)serve_xch_bytes<IN_P, HID_P, NH>() +
                        (tile_scatter ? 4 * HID_P * kStride * (int)sizeof(float) : 0);
        const hipError_t e = hipFuncSetAttribute((const void *)k,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3(std::min(blocks, 256)), dim3(256), lds, s, hdr, reqs, r0, r1,
                           chunks, which, chunk_tiles, img_bytes_max);
    }
    return hipGetLastError();
}

static hipError_t launch_shape(int key, RoundHdr *hdr, const DevReq *reqs, int r0, int r1,
                               int chunks, int which, bool train, int chunk_tiles,
                               bool tile_scatter, int img_bytes_max, hipStream_t s)
{
    switch (key) {
    case 2113: return launch_group<32, 64, 3, 2>(hdr, reqs, r0, r1, chunks, which, train, chunk_tiles, tile_scatter, img_bytes_max, s);
    case 2112: return launch_group<32, 64, 2, 2>(hdr, reqs, r0, r1, chunks, which, train, chunk_tiles, tile_scatter, img_bytes_max, s);
    case 4012: return launch_group<16, 64, 2, 4>(hdr, reqs, r0, r1, chunks, which, train, chunk_tiles, tile_scatter, img_bytes_max, s);
    case 2002: return launch_group<16, 32, 2, 2>(hdr, reqs, r0, r1, chunks, which, train, chunk_tiles, tile_scatter, img_bytes_max, s);
    default: return hipErrorNotSupported;
    }
}

// Tiles of a training chunk: up to four rounds of a tile per wave, as many as
// leave every CU a block.
static int train_chunk_tiles(int64_t tiles)
{
    const int64_t rounds = (tiles + 256 * kTrainWaves - 1) / (256 * kTrainWaves);
    return kTrainWaves * (int)std::max<int64_t>(1, std::min<int64_t>(4, rounds));
}

// The grid scatter of one request's dG (in the request's order: its bins hold
// every hashed level).
static hipError_t scatter_request(const ServeRequest &q, ServeLanes *l, const float *dgt,
                                  hipStream_t s)
{
    const GridDesc &g = q.ctx->net.grid;
    BinDesc b;
    const bool binned = request_bins(q.ctx->net, q.n, &b) && l->cnt.words >= bin_count_words(b) &&
                        l->items.words >= bin_item_words(b, g.feat);
    uint32_t left = g.n_levels >= 32 ? ~0u : (1u << g.n_levels) - 1u;
    if (binned)
        for (int j = 0; j < b.nb; ++j) left &= ~(1u << b.lv[j]);
    hipError_t e = chunk_scatter(q.ctx->net, q.n, q.pos, nullptr, nullptr, 8, dgt, kServeRows,
                                 q.ctx->grads, left, s);
    if (e == hipSuccess && binned)
        e = binned_scatter(q.ctx, b, q.n, q.pos, nullptr, nullptr, 8, dgt, kServeRows,
                           q.ctx->grads, l->cnt.p, l->items.p, false, s);
    return e;
}

// Round buffer: [header][DevReq x n][loss x n][stats pointer x n].  Requests
// are ordered by (shape, kind) so that each launch covers a contiguous range.
// With both kinds in a round the queries run on the side stream beside the
// training kernels (both only read the weights); the Adam steps follow both.
// Eight queries of 2^10 .. 2^17 vertices and two training batches, one stream /
// two: 587 / 545 us a round, submission and completion included.
hipError_t serve_launch_round(RoundBuffers *b, ServeLanes *lanes,
                              const std::vector<ServeRequest> &in, hipStream_t s)
{
    const int nreq = (int)in.size();
    if (nreq == 0) return hipSuccess;
    if (nreq > kMaxRoundRequests) return hipErrorInvalidValue;
    const RoundLayout L = round_layout(nreq);
    std::vector<int> order(nreq);
    for (int i = 0; i < nreq; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int c) {
        const int ka = shape_key(in[a].ctx->net) * 2 + in[a].kind;
        const int kc = shape_key(in[c].ctx->net) * 2 + in[c].kind;
        return ka < kc;
    });
    char *host = (char *)b->host;
    char *dev = (char *)b->dev;
    std::memset(host, 0, L.reqs);
    RoundHdr *hh = (RoundHdr *)host;
    hh->n_req = nreq;
    DevReq *hr = (DevReq *)(host + L.reqs);
    double *hloss = (double *)(host + L.loss);
    double **hstats = (double **)(host + L.stats);
    DevReq *dr = (DevReq *)(dev + L.reqs);
    double *dloss = (double *)(dev + L.loss);
    struct Group { int key, kind, r0, r1, chunks, img, tiles; bool tile_scatter; };
    std::vector<Group> groups;
    int64_t train_tiles = 0;
    for (const ServeRequest &q : in)
        if (q.kind == 1) train_tiles += (q.n + 31) / 32;
    const int per_train = train_chunk_tiles(train_tiles);
    // dG of the round's training batches, one after the other, as far as they
    // fit; the bins hold one batch at a time
    size_t dgt_at = 0;
    for (int j = 0; j < nreq; ++j) {
        const ServeRequest &q = in[order[j]];
        npm_ctx *ctx = q.ctx;
        const Net &net = ctx->net;
        const int key = shape_key(net);
        if (groups.empty() || groups.back().key != key || groups.back().kind != q.kind)
            groups.push_back({key, q.kind, j, j, 0, 0, q.kind == 0 ? kQueryChunkTiles : per_train, false});
        Group &g = groups.back();
        DevReq &d = hr[j];
        std::memset(&d, 0, sizeof(d));
        d.g = net.grid;
        const Weights w = q.kind == 0 ? query_weights(ctx) : trained_weights(ctx);
        d.grid16 = (const __half *)w.grid16;
        d.img = w.img16;
        d.grad = ctx->grads;
        d.pos = q.pos; d.dir = q.dir; d.rad = q.rad; d.spdf = q.spdf;
        d.lobes = q.lobes; d.pdf = q.pdf; d.sdir = q.sdir; d.spdf_out = q.spdf_out;
        d.loss = dloss + j;
        d.n = q.n;
        d.mlp_off = net.lay.grid_params;
        d.seed = q.seed;
        d.sid = q.stream_id;
        d.skey = q.session;
        d.fwd_elems = (int)net.mlp.fwd_elems;
        d.bwd_elems = (int)net.mlp.bwd_elems;
        d.n_in = net.mlp.n_in;
        d.width = net.mlp.width;
        d.invN = q.n > 0 ? 1.0f / (float)q.n : 0.0f;
        const int64_t tiles = (q.n + 31) / 32;
        if (q.kind == 1 && q.n > 0) {
            if (dgt_at + dgt_words(q.n) <= lanes->dgt.words) {
                d.dgt = (float *)lanes->dgt.p + dgt_at;
                dgt_at += dgt_words(q.n);
            } else {
                g.tile_scatter = true;
            }
        }
        d.chunk_begin = g.chunks;
        g.chunks += (int)((tiles + g.tiles - 1) / g.tiles);
        g.r1 = j + 1;
        const int img = (int)((q.kind == 0 ? net.mlp.fwd_elems : net.mlp.fwd_elems + net.mlp.bwd_elems) * 2);
        g.img = std::max(g.img, img);
        hloss[j] = 0.0;
        hstats[j] = q.stats;
    }
    // one counter per launch; serve_supports admits kServeShapes shapes
    if ((int)groups.size() > kMaxRoundGroups) return hipErrorNotSupported;
    const int pieces = (int)(L.total / 16);
    hipLaunchKernelGGL(k_round_upload, dim3((pieces + 255) / 256), dim3(256), 0, s, (uint4 *)dev,
                       (const uint4 *)host, pieces);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    RoundHdr *dh = (RoundHdr *)dev;
    bool trains = false, both = false;
    for (const Group &g : groups) trains |= g.kind == 1;
    for (const Group &g : groups) both |= trains && g.kind == 0;
    hipStream_t sq = s;                      // the queries' stream
    if (both) {
        sq = lanes->side;
        e = hipEventRecord(lanes->fork, s);
        if (e == hipSuccess) e = hipStreamWaitEvent(sq, lanes->fork, 0);
        if (e != hipSuccess) return e;
    }
    // the training kernels first: a block of theirs needs a CU's registers
    for (int kind = 1; kind >= 0; --kind)
        for (int gi = 0; gi < (int)groups.size() && e == hipSuccess; ++gi) {
            const Group &g = groups[gi];
            if (g.kind != kind) continue;
            e = launch_shape(g.key, dh, dr, g.r0, g.r1, g.chunks, gi, kind == 1, g.tiles,
                             g.tile_scatter, g.img, kind == 0 ? sq : s);
        }
    for (int gi = 0; gi < (int)groups.size() && e == hipSuccess; ++gi) {
        const Group &g = groups[gi];
        if (g.kind != 1) continue;
        hipLaunchKernelGGL(k_serve_finish, dim3((g.r1 - g.r0 + 63) / 64), dim3(64), 0, s, dr,
                           (const double *const *)(dev + L.stats), g.r0, g.r1);
        e = hipGetLastError();
        for (int j = g.r0; j < g.r1 && e == hipSuccess; ++j)
            if (hr[j].dgt) e = scatter_request(in[order[j]], lanes, hr[j].dgt, s);
    }
    // joined whatever failed: what follows on s, and the round's end, come
    // after the queries too
    if (both) {
        hipError_t ej = hipEventRecord(lanes->join, sq);
        if (ej == hipSuccess) ej = hipStreamWaitEvent(s, lanes->join, 0);
        if (ej != hipSuccess) (void)hipStreamSynchronize(sq);
        if (e == hipSuccess) e = ej;
    }
    for (int gi = 0; gi < (int)groups.size() && e == hipSuccess; ++gi) {
        const Group &g = groups[gi];
        for (int j = g.r0; g.kind == 1 && j < g.r1 && e == hipSuccess; ++j) {
            const ServeRequest &q = in[order[j]];
            q.ctx->step += 1;
            e = launch_adam(q.ctx, q.ctx->grads, q.stats ? q.stats + 1 : nullptr, s);
        }
    }
    return e;
}

}  // namespace npm
