// Kernels shared by every execution mode: parameter initialisation, packing of
// the MLP weights into MFMA-ready LDS images (and their BF16 copies), the FP16
// grid copy, fused Adam (Sec. 5.3, Kingma and Ba), and FP64 reductions.
#include "device_math.h"

namespace npm {

// ---------------------------------------------------------------- timing
void timed_begin(npm_ctx *ctx, const char *name, hipStream_t s, int *token)
{
    *token = -1;
    Timing &t = ctx->timing;
    if (!t.enabled) return;
    int id = -1;
    for (size_t i = 0; i < t.names.size(); ++i)
        if (t.names[i] == name) { id = (int)i; break; }
    if (id < 0) {
        id = (int)t.names.size();
        t.names.emplace_back(name);
        t.launches.push_back(0);
        t.total_ms.push_back(0.0);
    }
    hipEvent_t a, b;
    for (hipEvent_t *e : {&a, &b}) {
        if (!t.free_events.empty()) { *e = t.free_events.back(); t.free_events.pop_back(); }
        else if (hipEventCreate(e) != hipSuccess) return;
    }
    (void)hipEventRecord(a, s);      // a failed record only loses the timing
    t.pending.push_back({id, a, b});
    *token = (int)t.pending.size() - 1;
}

void timed_end(npm_ctx *ctx, int token, hipStream_t s)
{
    if (token < 0) return;
    (void)hipEventRecord(ctx->timing.pending[token].b, s);
}

// ---------------------------------------------------------------- init
// Parameters from Philox4x32-10 keyed by the seed, one counter per parameter:
// grid N(0, scale^2) or U(-scale, scale); MLP layer i Xavier-uniform.
struct InitDesc {
    int64_t grid_params;
    int64_t layer_off[NPM_MAX_LAYERS + 1];
    float layer_bound[NPM_MAX_LAYERS];
    int n_layers;
    int grid_init;
    float grid_scale;
    uint64_t seed;
};

__global__ void k_init(InitDesc d, float *__restrict__ p, int64_t np)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < np;
         i += (int64_t)gridDim.x * blockDim.x) {
        float u[3];
        philox_uniforms((uint64_t)i, d.seed, 0x1417u, 0u, u);
        float v;
        if (i < d.grid_params) {
            if (d.grid_init == NPM_INIT_NORMAL) {
                const float r = sqrtf(-2.0f * logf(1.0f - u[0]));    // 1 - u0 in (0, 1]
                v = d.grid_scale * r * cospif(2.0f * u[1]);
            } else {
                v = d.grid_scale * (2.0f * u[0] - 1.0f);
            }
        } else {
            int li = 0;
            while (li + 1 < d.n_layers && i >= d.layer_off[li + 1]) ++li;
            v = d.layer_bound[li] * (2.0f * u[0] - 1.0f);
        }
        p[i] = v;
    }
}

hipError_t launch_init_params(npm_ctx *ctx, hipStream_t s)
{
    const Net &net = ctx->net;
    InitDesc d{};
    d.grid_params = net.lay.grid_params;
    d.n_layers = net.lay.n_layers;
    for (int i = 0; i < d.n_layers; ++i) {
        d.layer_off[i] = net.lay.layer_offset[i];
        d.layer_bound[i] = sqrtf(6.0f / (float)(net.lay.layer_in[i] + net.lay.layer_out[i]));
    }
    d.layer_off[d.n_layers] = net.lay.n_params;
    d.grid_init = net.cfg.grid_init;
    d.grid_scale = net.cfg.grid_init_scale;
    d.seed = net.cfg.seed;
    const int64_t np = net.lay.n_params;
    const int blocks = (int)std::min<int64_t>((np + 255) / 256, 8192);
    hipLaunchKernelGGL(k_init, dim3(blocks), dim3(256), 0, s, d, ctx->params, np);
    return hipGetLastError();
}

// ---------------------------------------------------------------- packing
// One segment per (layer, direction) of the packed images.  Element idx of a
// segment maps to (block b, step, lane, e) and reads W[row][col] of the layer
// (forward) or of its transpose (backward), zero outside the real shape.
struct PackSeg {
    int64_t dst;        // first element in the image
    int64_t src;        // first weight of the layer in the flat parameters
    int32_t out_p, in_p; // padded shape of the image matrix
    int32_t out_r, in_r; // real shape of the image matrix
    int32_t ld;          // row length of the stored (untransposed) matrix
    int32_t transpose;
};

struct PackDesc {
    PackSeg seg[2 * NPM_MAX_LAYERS];
    int n_seg;
    int64_t total;
};

// The weight that element idx of the packed image (FP32 or BF16 order) holds.
template <bool BF16>
__device__ __forceinline__ float pack_value(const PackDesc &d, int64_t i, const float *__restrict__ params)
{
    int si = 0;
    while (si + 1 < d.n_seg && i >= d.seg[si + 1].dst) ++si;
    const PackSeg &g = d.seg[si];
    const int64_t k = i - g.dst;
    int lane, b, step;
    if (!BF16) {
        const int e = (int)(k & 3);
        lane = (int)((k >> 2) & 63);
        const int64_t rest = k >> 8;
        const int ns4 = g.in_p / 8;
        b = (int)(rest / ns4);
        step = (int)(rest % ns4) * 4 + e;
    } else {
        const int e = (int)(k & 7);
        lane = (int)((k >> 3) & 63);
        const int64_t rest = k >> 9;
        const int ns = g.in_p / 16;
        b = (int)(rest / ns);
        step = (int)(rest % ns) * 8 + e;
    }
    const int row = 32 * b + (lane & 31);
    const int col = nf(lane >> 5, step);
    if (row >= g.out_r || col >= g.in_r) return 0.0f;
    return g.transpose ? params[g.src + (int64_t)col * g.ld + row]
                       : params[g.src + (int64_t)row * g.ld + col];
}

static PackDesc pack_desc(const Net &net)
{
    const MlpDesc &m = net.mlp;
    const npm_layout &L = net.lay;
    PackDesc d{};
    int n = 0;
    for (int i = 0; i < L.n_layers; ++i) {
        PackSeg &g = d.seg[n++];
        g.dst = m.fwd_off[i];
        g.src = L.layer_offset[i];
        g.in_p = (i == 0) ? m.in_p : m.hid_p;
        g.out_p = (i == L.n_layers - 1) ? 32 : m.hid_p;
        g.out_r = L.layer_out[i];
        g.in_r = L.layer_in[i];
        g.ld = L.layer_in[i];
        g.transpose = 0;
    }
    // backward images are stored from the last layer to the first; segments
    // must be in increasing dst order for the lookup in k_pack
    for (int i = L.n_layers - 1; i >= 0; --i) {
        PackSeg &g = d.seg[n++];
        g.dst = m.fwd_elems + m.bwd_off[i];
        g.src = L.layer_offset[i];
        const int fin = (i == 0) ? m.in_p : m.hid_p;
        const int fout = (i == L.n_layers - 1) ? 32 : m.hid_p;
        g.in_p = fout;
        g.out_p = fin < 32 ? 32 : fin;
        g.out_r = L.layer_in[i];
        g.in_r = L.layer_out[i];
        g.ld = L.layer_in[i];
        g.transpose = 1;
    }
    d.n_seg = n;
    d.total = m.fwd_elems + m.bwd_elems;
    return d;
}

// The row-major image of the gathering training kernel (MlpDesc::rm_off):
// layer L as its padded rows x cols matrix, rows cols + 1 floats apart, zero
// outside the real weights.
struct RmDesc {
    int64_t off[NPM_MAX_LAYERS + 1];
    int64_t src[NPM_MAX_LAYERS];
    int32_t cols[NPM_MAX_LAYERS], out_r[NPM_MAX_LAYERS], in_r[NPM_MAX_LAYERS];
    int32_t n_layers;
};

__device__ __forceinline__ float rm_value(const RmDesc &d, int64_t i, const float *__restrict__ params)
{
    int L = 0;
    while (L + 1 < d.n_layers && i >= d.off[L + 1]) ++L;
    const int64_t k = i - d.off[L];
    const int S = d.cols[L] + 1;
    const int o = (int)(k / S), c = (int)(k % S);
    return (o < d.out_r[L] && c < d.in_r[L]) ? params[d.src[L] + (int64_t)o * d.in_r[L] + c] : 0.0f;
}

// Every image of a network's weights, and of their average (ema non-null), in
// one launch: an element each of the FP32 image, the BF16 image (its backward
// part with the two further planes of the three-way split, x = x0 + x1 + x2,
// where `split` is set) and the row-major image, one after the other in the
// index.  The grid's last block sums `nparts` FP64 partials into *sum (where
// set).  One launch for what took up to six of 4 us each (a 16,384-vertex
// training step of the 4-level network 101 -> 83 us, with the loss sum folded
// into the weight-gradient sum).
struct PackJob {
    PackDesc d;
    RmDesc r;
    int64_t fwd, n_rm;             // elements of the forward image, of the row-major image (or 0)
    const float *params, *ema;
    float *img, *rm, *ema_img;
    __bf16 *img16, *split, *ema_img16;
    const double *part;
    int nparts;
    double *sum;
};

__global__ __launch_bounds__(256) void k_pack(PackJob j)
{
    if (j.sum && blockIdx.x == gridDim.x - 1) {
        const double s = sum_partials(j.part, j.nparts);
        if (threadIdx.x == 0) *j.sum = s;
        return;
    }
    const int64_t T = j.d.total;
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (i < T) {
        j.img[i] = pack_value<false>(j.d, i, j.params);
        if (j.ema) j.ema_img[i] = pack_value<false>(j.d, i, j.ema);
    } else if (i < 2 * T) {
        const int64_t k = i - T;
        const float v = pack_value<true>(j.d, k, j.params);
        const __bf16 v0 = (__bf16)v;
        j.img16[k] = v0;
        if (j.split && k >= j.fwd) {
            const float r1 = v - (float)v0;
            const __bf16 v1 = (__bf16)r1;
            j.split[k - j.fwd] = v1;
            j.split[T - j.fwd + k - j.fwd] = (__bf16)(r1 - (float)v1);
        }
        if (j.ema) j.ema_img16[k] = (__bf16)pack_value<true>(j.d, k, j.ema);
    } else if (i < 2 * T + j.n_rm) {
        j.rm[i - 2 * T] = rm_value(j.r, i - 2 * T, j.params);
    }
}

// nparts > 0: also sums ctx->partials into *sum.
static hipError_t pack_images(npm_ctx *ctx, int nparts, double *sum, hipStream_t s)
{
    const Net &net = ctx->net;
    const MlpDesc &m = net.mlp;
    PackJob j{};
    j.d = pack_desc(net);
    j.fwd = m.fwd_elems;
    j.params = ctx->params;
    j.ema = ctx->ema;
    j.img = ctx->mlp_img;
    j.ema_img = ctx->ema_img;
    j.img16 = (__bf16 *)ctx->mlp_img16;
    j.split = (__bf16 *)ctx->mlp_split;
    j.ema_img16 = (__bf16 *)ctx->ema_img16;
    if (net.cfg.precision == NPM_PREC_FP32) {      // read by the FP32 training kernel only
        j.n_rm = m.rm_elems;
        j.rm = ctx->mlp_img + m.fwd_elems + m.bwd_elems;
        j.r.n_layers = net.lay.n_layers;
        for (int i = 0; i < j.r.n_layers; ++i) {
            j.r.off[i] = m.rm_off[i];
            j.r.src[i] = net.lay.layer_offset[i];
            j.r.cols[i] = i == 0 ? std::max(m.in_p, 32) : m.hid_p;
            j.r.out_r[i] = net.lay.layer_out[i];
            j.r.in_r[i] = net.lay.layer_in[i];
        }
        j.r.off[j.r.n_layers] = m.rm_elems;
    }
    j.part = ctx->partials;
    j.nparts = nparts;
    j.sum = nparts > 0 ? sum : nullptr;
    const int64_t elems = 2 * j.d.total + j.n_rm;
    const int blocks = (int)((elems + 255) / 256) + (j.sum ? 1 : 0);
    hipLaunchKernelGGL(k_pack, dim3(blocks), dim3(256), 0, s, j);
    return hipGetLastError();
}

__global__ void k_grid_to_half(const float *__restrict__ p, __half *__restrict__ h, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        h[i] = __float2half_rn(p[i]);
}

hipError_t launch_refresh_lowp(npm_ctx *ctx, hipStream_t s)
{
    const hipError_t e = pack_images(ctx, 0, nullptr, s);
    if (e != hipSuccess) return e;
    const int64_t n = ctx->net.lay.grid_params;
    if (ctx->grid16)
        hipLaunchKernelGGL(k_grid_to_half, dim3(2048), dim3(256), 0, s, ctx->params,
                           (__half *)ctx->grid16, n);
    if (ctx->ema_grid16)
        hipLaunchKernelGGL(k_grid_to_half, dim3(2048), dim3(256), 0, s, ctx->ema,
                           (__half *)ctx->ema_grid16, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------- Adam
// m <- b1 m + (1-b1) g; v <- b2 v + (1-b2) g^2; p <- p - lr m^/(sqrt(v^) + eps)
// with m^ = m / (1 - b1^t), v^ = v / (1 - b2^t); g is zeroed; the FP16 copy of
// the grid is written in the same pass; sum g^2 is reduced in FP64.  With a
// moving average kept (ema non-null), ema <- d ema + (1 - d) p after the step,
// and its FP16 grid copy too.
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ p, float *__restrict__ g,
                                              float *__restrict__ m, float *__restrict__ v,
                                              int64_t np, float lr, float b1, float b2, float eps,
                                              float c1inv, float c2inv, __half *__restrict__ grid16,
                                              int64_t grid_params, double *__restrict__ partials,
                                              float *__restrict__ ema, __half *__restrict__ ema16,
                                              float decay)
{
    double acc = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < np;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * (gi * gi);
        const float pi = p[i] - lr * (mi * c1inv) / (sqrtf(vi * c2inv) + eps);
        m[i] = mi;
        v[i] = vi;
        p[i] = pi;
        g[i] = 0.0f;
        if (grid16 && i < grid_params) grid16[i] = __float2half_rn(pi);
        if (ema) {
            const float ei = decay * ema[i] + (1.0f - decay) * pi;
            ema[i] = ei;
            if (ema16 && i < grid_params) ema16[i] = __float2half_rn(ei);
        }
        acc += (double)gi * (double)gi;
    }
    __shared__ double red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = red[0];
}

hipError_t launch_adam(npm_ctx *ctx, float *grad, double *gradnorm_out, hipStream_t s)
{
    const npm_config &c = ctx->net.cfg;
    const double t = (double)ctx->step;
    const float c1inv = (float)(1.0 / (1.0 - pow((double)c.beta1, t)));
    const float c2inv = (float)(1.0 / (1.0 - pow((double)c.beta2, t)));
    const int64_t np = ctx->net.lay.n_params;
    const int blocks = (int)std::min<int64_t>((np + 255) / 256, 2048);
    int tok;
    timed_begin(ctx, "adam", s, &tok);
    hipLaunchKernelGGL(k_adam, dim3(blocks), dim3(256), 0, s, ctx->params, grad, ctx->adam_m,
                       ctx->adam_v, np, c.lr, c.beta1, c.beta2, c.eps, c1inv, c2inv,
                       (__half *)ctx->grid16, ctx->net.lay.grid_params, ctx->partials, ctx->ema,
                       (__half *)ctx->ema_grid16, c.ema_decay);
    timed_end(ctx, tok, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the packed MLP images follow the new weights; with them the gradient norm
    return pack_images(ctx, gradnorm_out ? blocks : 0, gradnorm_out, s);
}

// ---------------------------------------------------------------- reductions
// Sums nparts FP64 partials in a fixed order into *out (times scale).
__global__ __launch_bounds__(256) void k_reduce(const double *__restrict__ part, int nparts,
                                                double scale, double *__restrict__ out)
{
    const double s = sum_partials(part, nparts);
    if (threadIdx.x == 0) *out = s * scale;
}

hipError_t launch_reduce_scaled(const double *part, int nparts, double scale, double *out,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(256), 0, s, part, nparts, scale, out);
    return hipGetLastError();
}

__global__ void k_fill(float *__restrict__ p, int64_t n, float v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s)
{
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

}  // namespace npm
