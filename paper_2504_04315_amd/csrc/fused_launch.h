// What the fused launchers share (k_query.hip, k_fused.hip): the kernels'
// argument block and the dispatch over the network shapes they are built for.
#pragma once

#include "fused_tiles.h"

namespace npm {

struct FusedArgs {
    GridDesc g;
    int64_t n;
    const float *pos, *dir, *rad, *spdf;
    const float *grid32;     // FP32 grid (plain form)
    const __half *grid16;    // FP16 grid (precision form)
    const void *img;         // packed MLP images: forward then backward
    int fwd_elems, bwd_elems;
    int n_in, width;
    uint64_t seed;
    uint32_t sid;
    float *lobes, *pdf, *sdir, *spdf_out;
    float *grad;             // accumulated gradient (backward)
    float *dw_part;          // per-wave weight-gradient partials (backward)
    double *partials;        // per-block FP64 loss partials
    float invN;
    const uint32_t *perm;    // visiting order of the vertices (backward), or null
    float *dg_tiles;         // per-tile dG for the aggregated scatter (backward)
    float *qstage;           // staged query outputs in visiting order (with perm)
    const float *rec;        // inputs in visiting order (with perm), rec_stride floats each
    const float *aux;        // NPM-product inputs [7][n]
    int rec_stride;
    // learned selection probability (networks with the selection output)
    const float *wsel;       // the selection row of the last layer (FP32 weights)
    const float *bsdf;       // BSDF densities [n] of the selection term (backward), or null
    double *partials_sel;    // per-block FP64 partials of the selection loss
    float *sel;              // selection probability [n] (query), or null
    int tile_v, halves;      // vertices per block and blocks per tile (k_query_small)
    const void *feat;        // level-major grid features of the batch (k_encode.hip)
    const __bf16 *img_t;     // packed BF16 image of W^T (the backward image), and the two
    const __bf16 *img_split; // further planes of its three-way split (FP32 training)
    const float *mlp;        // the flat FP32 MLP weights (backward)
    float *grad_mlp;         // and their gradient
};

inline FusedArgs fused_args(npm_ctx *ctx, int64_t n, const float *pos)
{
    FusedArgs a{};
    const Net &net = ctx->net;
    a.g = net.grid;
    a.n = n;
    a.pos = pos;
    a.grid32 = ctx->params;
    a.grid16 = (const __half *)ctx->grid16;
    const bool bf = net.cfg.precision == NPM_PREC_BF16;
    a.img = bf ? ctx->mlp_img16 : (const void *)ctx->mlp_img;
    a.fwd_elems = (int)net.mlp.fwd_elems;
    a.bwd_elems = (int)net.mlp.bwd_elems;
    a.n_in = net.mlp.n_in;
    a.width = net.mlp.width;
    a.rec_stride = net.cfg.sh_degree ? 16 : 8;
    return a;
}

#define NPM_FUSED_DISPATCH(RUN, BFV)                                                              \
    do {                                                                                          \
        const MlpDesc &m_ = ctx->net.mlp;                                                         \
        const int F_ = ctx->net.grid.feat;                                                        \
        const int key_ = F_ * 1000 + (m_.in_p == 32) * 100 + (m_.hid_p == 64) * 10 + m_.n_hidden; \
        switch (key_) {                                                                           \
        case 1002: e = RUN<16, 32, 2, 1, BFV>(ctx, a, s); break;                                  \
        case 1112: e = RUN<32, 64, 2, 1, BFV>(ctx, a, s); break;                                  \
        case 1113: e = RUN<32, 64, 3, 1, BFV>(ctx, a, s); break;                                  \
        case 2002: e = RUN<16, 32, 2, 2, BFV>(ctx, a, s); break;                                  \
        case 2012: e = RUN<16, 64, 2, 2, BFV>(ctx, a, s); break;                                  \
        case 2112: e = RUN<32, 64, 2, 2, BFV>(ctx, a, s); break;                                  \
        case 2113: e = RUN<32, 64, 3, 2, BFV>(ctx, a, s); break;                                  \
        case 4012: e = RUN<16, 64, 2, 4, BFV>(ctx, a, s); break;                                  \
        case 4013: e = RUN<16, 64, 3, 4, BFV>(ctx, a, s); break;                                  \
        case 4112: e = RUN<32, 64, 2, 4, BFV>(ctx, a, s); break;                                  \
        case 4113: e = RUN<32, 64, 3, 4, BFV>(ctx, a, s); break;                                  \
        default: return hipErrorNotSupported;                                                     \
        }                                                                                         \
    } while (0)

// NPM-product shapes (sh_degree 4 on 32 grid features, 65 inputs in a 96-wide
// first layer; sh_degree 2 on 4 grid features, 13 inputs).
#define NPM_FUSED_PRODUCT_DISPATCH(RUN, BFV)                                                      \
    do {                                                                                          \
        const MlpDesc &m_ = ctx->net.mlp;                                                         \
        const int F_ = ctx->net.grid.feat;                                                        \
        const int key_ = m_.sh_degree * 100000 + F_ * 10000 + m_.in_p * 100 +                    \
                         (m_.hid_p == 64) * 10 + m_.n_hidden;                                     \
        switch (key_) {                                                                           \
        case 429612: e = RUN<96, 64, 2, 2, BFV, 1>(ctx, a, s); break;                             \
        case 429613: e = RUN<96, 64, 3, 2, BFV, 1>(ctx, a, s); break;                             \
        case 449612: e = RUN<96, 64, 2, 4, BFV, 1>(ctx, a, s); break;                             \
        case 449613: e = RUN<96, 64, 3, 4, BFV, 1>(ctx, a, s); break;                             \
        case 221602: e = RUN<16, 32, 2, 2, BFV, 2>(ctx, a, s); break;                             \
        default: return hipErrorNotSupported;                                                     \
        }                                                                                         \
    } while (0)

// Networks with the selection output: the tiny (4 inputs, width 8), cfg1
// (16 inputs, 64 x 2), the paper's (32 inputs, 64 x 2) and the production
// (32 inputs, 64 x 3) shapes.
#define NPM_FUSED_SEL_DISPATCH(RUN, BFV)                                                          \
    do {                                                                                          \
        const MlpDesc &m_ = ctx->net.mlp;                                                         \
        const int F_ = ctx->net.grid.feat;                                                        \
        const int key_ = F_ * 1000 + (m_.in_p == 32) * 100 + (m_.hid_p == 64) * 10 + m_.n_hidden; \
        switch (key_) {                                                                           \
        case 2002: e = RUN<16, 32, 2, 2, BFV, 0, true>(ctx, a, s); break;                         \
        case 4012: e = RUN<16, 64, 2, 4, BFV, 0, true>(ctx, a, s); break;                         \
        case 4112: e = RUN<32, 64, 2, 4, BFV, 0, true>(ctx, a, s); break;                         \
        case 2113: e = RUN<32, 64, 3, 2, BFV, 0, true>(ctx, a, s); break;                         \
        default: return hipErrorNotSupported;                                                     \
        }                                                                                         \
    } while (0)

#define NPM_FUSED_RUN(RUN)                                                                        \
    do {                                                                                          \
        const bool bf_ = ctx->net.cfg.precision == NPM_PREC_BF16;                                 \
        if (ctx->net.cfg.learn_selection) {                                                       \
            if (bf_) NPM_FUSED_SEL_DISPATCH(RUN, true);                                           \
            else NPM_FUSED_SEL_DISPATCH(RUN, false);                                              \
        } else if (ctx->net.mlp.sh_degree > 0) {                                                  \
            if (bf_) NPM_FUSED_PRODUCT_DISPATCH(RUN, true);                                       \
            else NPM_FUSED_PRODUCT_DISPATCH(RUN, false);                                          \
        } else {                                                                                  \
            if (bf_) NPM_FUSED_DISPATCH(RUN, true);                                               \
            else NPM_FUSED_DISPATCH(RUN, false);                                                  \
        }                                                                                         \
    } while (0)

// Blocks of the training kernels: one per compute unit at most (the weight
// images take most of its LDS), four waves each.
constexpr int kTrainWaves = 4;
constexpr int kTrainMaxBlocks = 256;
inline int train_blocks(int64_t n)
{
    const int64_t tiles = (n + 31) / 32;
    return (int)std::max<int64_t>(1, std::min<int64_t>((tiles + kTrainWaves - 1) / kTrainWaves,
                                                       kTrainMaxBlocks));
}

// Dynamic LDS a training block may take: gfx950's 160 KB per workgroup less
// room for the kernel's static arrays (level table, FP64 loss partials).
constexpr size_t kLdsBytes = 160 * 1024 - 4096;

// The training tile kernel of a batch with encoded features (k_train.hip);
// args as for the gathering kernel, feat set.
hipError_t train_tile(npm_ctx *ctx, const FusedArgs &args, hipStream_t s);

}  // namespace npm
