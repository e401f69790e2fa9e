// Internal host-side declarations of libnpm: the context, the derived network
// description, and the launchers each kernel file provides.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "npm.h"

namespace npm {

constexpr int kLobes = 8;             // K (Sec. 5.3)
constexpr int kOut = 4 * kLobes;      // lobe raw outputs per vertex (a selection
                                      // network has one more, the logit, at kOut)
constexpr int kWave = 64;             // CDNA wavefront
constexpr int kTile = 32;             // vertices per wave tile (32x32 MFMA)

// Grid description passed to kernels by value.
struct GridDesc {
    uint32_t offset[NPM_MAX_LEVELS];  // first entry of each level
    int32_t res[NPM_MAX_LEVELS];      // D_l
    uint32_t hashed_mask;             // bit l set: level l is hashed
    uint32_t table_mask;              // 2^log2T - 1
    int32_t n_levels;
    int32_t feat;
};

// MLP shape as the kernels see it: widths padded to MFMA tiles.
struct MlpDesc {
    int n_in, width, n_hidden;        // real sizes
    int in_p, hid_p;                  // padded: in_p in {16, 32, 64, 96}, hid_p in {32, 64}
    int gf;                           // grid features (n_levels * feat), the first inputs
    int sh_degree;                    // NPM-product: SH bands of omega_o and the normal
    int64_t fwd_off[NPM_MAX_LAYERS];  // offset of each layer's image in the packed
    int64_t bwd_off[NPM_MAX_LAYERS];  //   forward / backward weight images (elements)
    int64_t fwd_elems, bwd_elems;
    // Row-major FP32 image of the training kernel: layer L as its padded
    // out_p x c_L matrix (c_0 = max(in_p, 32), c_L = hid_p otherwise) with
    // rows c_L + 1 floats apart, read as W (forward) and as W^T (backward)
    int64_t rm_off[NPM_MAX_LAYERS];
    int64_t rm_elems;
};

struct Net {
    npm_config cfg;
    npm_layout lay;
    GridDesc grid;
    MlpDesc mlp;
};

// Fills *net from *cfg; returns NPM_OK or NPM_ERR_INVALID_ARG with a message.
npm_status describe(const npm_config *cfg, Net *net, std::string *err);

// Sets the calling thread's npm_last_error() message.
void set_error(const char *msg);

// Per-kernel event timing.
struct Timing {
    bool enabled = false;
    std::vector<std::string> names;
    std::vector<int64_t> launches;
    std::vector<double> total_ms;
    struct Pending { int id; hipEvent_t a, b; };
    std::vector<Pending> pending;
    std::vector<hipEvent_t> free_events;
};

}  // namespace npm

struct npm_ctx {
    npm::Net net;
    int device = 0;
    int64_t step = 0;
    // FP32 master state, n_params each
    float *params = nullptr, *grads = nullptr, *adam_m = nullptr, *adam_v = nullptr;
    // Low-precision copies (NPM_PREC_BF16): FP16 grid, BF16 packed MLP images
    void *grid16 = nullptr;
    // Packed MLP weight images (forward and backward), FP32 and BF16
    float *mlp_img = nullptr;          // [fwd_elems + bwd_elems + rm_elems] FP32
    void *mlp_img16 = nullptr;         // [fwd_elems + bwd_elems] BF16
    void *mlp_split = nullptr;         // [2][bwd_elems] BF16: the backward image's two further
                                       // planes (FP32 form: weight = sum of three BF16 numbers)
    // Exponential moving average of the parameters (ema_decay > 0): FP32
    // master, its packed images and (NPM_PREC_BF16) its FP16 grid
    float *ema = nullptr, *ema_img = nullptr;
    void *ema_img16 = nullptr, *ema_grid16 = nullptr;
    // FP64 reduction scratch
    double *partials = nullptr;        // kPartials doubles
    double *stats = nullptr;           // 4 doubles: loss, gradnorm, spare
    // Staged-path scratch, grown on demand
    int64_t scratch_n = 0;
    float *s_G = nullptr, *s_raw = nullptr, *s_acts = nullptr, *s_delta = nullptr,
          *s_draw = nullptr, *s_dG = nullptr;
    float *s_dw_part = nullptr;        // dW partials
    int64_t dw_part_elems = 0;
    // spatial order of a training batch (fused path)
    uint32_t *s_perm = nullptr;        // [sort_n] visiting slot -> vertex
    uint32_t *s_inv = nullptr;         // [sort_n] vertex -> visiting slot
    float *s_rec = nullptr;            // [sort_n][8] inputs in visiting order
    float *s_qstage = nullptr;         // [qstage_n][40] staged query outputs
    int64_t qstage_n = 0;
    // grid features of a batch encoded level by level: 32-bit words
    uint32_t *s_feat = nullptr;
    size_t feat_cap = 0;
    uint32_t *s_cells = nullptr;       // 2^18 cell counts / offsets, 256 block totals
    int64_t sort_n = 0;
    // per-tile dG of a fused training batch, for the aggregated scatter
    // ([tiles][max(in_p, 32)][32]), and behind it the batch's grid features
    // where the tile kernel reads them and there was room (dgt_short: there
    // was not)
    float *s_dgt = nullptr;
    size_t dgt_words = 0;
    bool dgt_short = false;
    // binned scatter of the hashed levels: per-chunk bin counts / offsets
    // (and the scan's block totals), and the binned items
    uint32_t *s_bin_cnt = nullptr, *s_bin_items = nullptr;
    size_t bin_cnt_words = 0, bin_item_words = 0;
    // a second stream (default priority) on which the chunked scatter and
    // the weight-gradient sum run beside the binned scatter, forked from and
    // joined back to the caller's stream by the two events
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    npm::Timing timing;
};

namespace npm {

constexpr int kPartials = 4096;        // FP64 partial slots per reduction

// The weights a kernel reads: the trained ones, or, for the network npm_query
// evaluates, their moving average when it is kept.
struct Weights {
    const float *grid32;      // FP32 grid (the head of the flat parameters)
    const void *grid16;       // FP16 grid (precision form) or null
    const float *img;         // packed FP32 images
    const void *img16;        // packed BF16 images
};
inline Weights trained_weights(const npm_ctx *c)
{
    return Weights{c->params, c->grid16, c->mlp_img, c->mlp_img16};
}
inline Weights query_weights(const npm_ctx *c)
{
    return c->ema ? Weights{c->ema, c->ema_grid16, c->ema_img, c->ema_img16} : trained_weights(c);
}

// The selection row of the last layer within the flat parameters `flat`
// (width FP32 weights after the output layer's 4K rows), or null when the
// network has no selection output.
inline const float *selection_row(const npm_ctx *c, const float *flat)
{
    const npm_layout &L = c->net.lay;
    if (!c->net.cfg.learn_selection) return nullptr;
    return flat + L.layer_offset[L.n_layers - 1] + (int64_t)kOut * c->net.mlp.width;
}

// ---------------------------------------------------------------- launchers
// All return hipSuccess or the first launch error.  `s` is the stream.
struct Launch {
    npm_ctx *ctx;
    hipStream_t s;
};

// Timing bracket (no-op unless enabled).
void timed_begin(npm_ctx *ctx, const char *name, hipStream_t s, int *token);
void timed_end(npm_ctx *ctx, int token, hipStream_t s);

// npm_create; reserve: with the feature scratch of the queries that are too small
// to be sorted, so that they never allocate
npm_status create_context(const npm_config *cfg, bool reserve, npm_ctx **out);

// common kernels (k_common.hip)
hipError_t launch_init_params(npm_ctx *ctx, hipStream_t s);
// repacks the images and rewrites the FP16 grids from the FP32 masters
hipError_t launch_refresh_lowp(npm_ctx *ctx, hipStream_t s);
hipError_t launch_adam(npm_ctx *ctx, float *grad, double *gradnorm_out, hipStream_t s);
hipError_t launch_reduce_scaled(const double *part, int nparts, double scale, double *out,
                                hipStream_t s);
hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s);

// level-major grid encoding (k_encode.hip): the features of n vertices,
// positions from pos [3][n] or (rec set) the first three floats of rec's
// records, rec_stride floats each.  b16: from the FP16 table, rounded to BF16
// and stored in feature pairs [ceil(features / 2)][n]; otherwise FP32
// [features][n].
hipError_t launch_grid_encode(const GridDesc &g, int64_t n, const float *pos, const float *rec,
                              int rec_stride, const float *grid32, const void *grid16, bool b16,
                              void *out, hipStream_t s);
// 32-bit words of its output
inline size_t feat_words(const Net &net, int64_t n)
{
    const int gf = net.mlp.gf;
    return (size_t)(net.cfg.precision == NPM_PREC_BF16 ? (gf + 1) / 2 : gf) * (size_t)n;
}

// staged path (k_staged.hip)
hipError_t staged_corner_index(npm_ctx *ctx, int64_t n, const float *pos, uint32_t *idx,
                               hipStream_t s);
// w: the weights to evaluate (the trained ones by default)
// aux: the NPM-product inputs [7][n] (required when the network takes them)
hipError_t staged_encode(npm_ctx *ctx, int64_t n, const float *pos, float *G, hipStream_t s,
                         const Weights *w = nullptr, const float *aux = nullptr);
hipError_t staged_mlp_fwd(npm_ctx *ctx, int64_t n, const float *G, float *acts, float *raw,
                          hipStream_t s, const Weights *w = nullptr);
// sel (or null): the selection probability of each vertex (selection networks)
hipError_t staged_head(npm_ctx *ctx, int64_t n, const float *raw, const float *dir,
                       uint64_t seed, uint32_t stream_id, float *lobes, float *pdf,
                       float *sdir, float *spdf, hipStream_t s, float *sel = nullptr);
// bsdf (or null): the BSDF density of each sample, for the selection term of a
// network with the selection output; its loss then goes to loss_out[1]
hipError_t staged_loss_grad(npm_ctx *ctx, int64_t n, const float *raw, const float *dir,
                            const float *rad, const float *spdf, float *draw, double *loss_out,
                            hipStream_t s, const float *bsdf = nullptr);
hipError_t staged_mlp_bwd(npm_ctx *ctx, int64_t n, const float *draw, const float *acts,
                          float *delta, float *dG, hipStream_t s);
hipError_t staged_mlp_dw(npm_ctx *ctx, int64_t n, const float *G, const float *acts,
                         const float *delta, const float *draw, float *grad, hipStream_t s);
hipError_t staged_scatter(npm_ctx *ctx, int64_t n, const float *pos, const float *dG,
                          float *grad, hipStream_t s);

// spatial order of a batch (k_sort.hip): perm lists the vertices by cell,
// inv (required, n entries) receives its inverse; clear: further words to zero
// on the way (the bins' totals), or null
hipError_t spatial_order(npm_ctx *ctx, int64_t n, const float *pos, const float *aux,
                         const float *dir, const float *rad, const float *spdf, uint32_t *perm,
                         uint32_t *inv, float *rec, uint32_t *cells, hipStream_t s,
                         uint32_t *clear = nullptr, int clear_words = 0);
// Smallest batch NPM_ORDER_AUTO sorts.  On the 16-level hash grid at 2^20
// vertices the sort (0.12 ms) lets the scatter sum shared corners and lines in
// LDS and speeds the encode's gathers (475 -> 262 us with a thread per vertex);
// a batch of 2^15 vertices is still dense enough to share the coarse levels'.
constexpr int64_t kSortMinBatch = 1 << 15;
// 32-bit words of the sort's cell scratch: 2^18 cell counters, then 256
// block totals of its scan.
constexpr size_t kSortCellWords = ((size_t)1 << 18) + 256;

// Binned scatter of the hashed levels (k_bin.hip).  The corner contributions
// of a training batch are binned by (level, table slice) in chunks of
// kBinChunk visiting slots, as pairs of x-neighbour corners (which the hash
// keeps in one slice), and each bin (a slice of kBinSliceFloats table floats)
// is summed by one block in LDS, replacing one memory-side FP32 atomic per
// corner.
constexpr int kBinChunk = 1024;           // 512 with one item per corner (its LDS then capped it)
constexpr int kBinSliceFloats = 16384;      // table floats per bin (8,192 entries at F = 2)
constexpr int kBinReduceThreads = 1024;
constexpr int kBinReduceBatch = 4;         // items in flight per thread
constexpr int kBinMaxBins = 2048;
constexpr int kBinMaxSlices = 1024;
// Smallest batch NPM_SCATTER_AUTO bins (the count, place and reduce launches,
// and the reduce's pass over every slice, whatever the batch).  Training step,
// chunked scatter alone / binned: 2^17 entries, 6,001 vertices 100 / 117 us,
// 20,001 148 / 131, 30,001 186 / 138; 2^19 entries, 8,001 190 / 216, 16,001 209
// / 214, 30,001 272 / 254.
constexpr int64_t kBinMinBatch = 20000;
// ... and only grids whose binned levels split into this many slices (small
// tables leave the reduce too few blocks).  2^17 entries, 160 slices, chunked
// scatter alone / binned: 40,001 vertices 204 / 159 us, 120,001 495 / 304,
// 400,001 937 / 536, 1,000,001 2207 / 1753.
constexpr int kBinMinBins = 128;
// In a spatially ordered batch the hashed levels with D_l below this share
// enough lines to stay with the chunked scatter.  One line for every batch size
// lies where the sparser batches, which share fewer lines, want it: training
// step of the 16-level production grid with the line at 100 / 140 / 180 / 250,
// 100,003 vertices 470 / 473 / 484 / 499 us, 300,001 545 / 564 / 580 / 622; at
// 2^20 140 would be the better one by 3 to 4 % (FP32 1.68 / 1.61 / 1.63 / 1.66
// ms, precision form 1.18 / 1.15 / 1.18 / 1.19).
constexpr int kBinMinResOrdered = 100;
struct BinDesc {
    int32_t nb;                        // binned levels
    int32_t lv[NPM_MAX_LEVELS];        // their indices
    int32_t log2s;                     // log2 of the table entries per slice
    int32_t ns;                        // slices per level
    int32_t nbins;                     // nb * ns
    int64_t n_chunks;                  // ceil(n / kBinChunk)
    int64_t cap;                       // item (corner pair) capacity: n * 4 * nb
};
// false when the batch has no level to bin or exceeds the pass's limits
bool bin_plan(const Net &net, int64_t n, bool ordered, BinDesc *out);
size_t bin_count_words(const BinDesc &b);
int bin_clear_words(const BinDesc &b);     // the first words of the counters
size_t bin_item_words(const BinDesc &b, int feat);
// dgt/rows: the per-tile dG of the batch in visiting order (perm / rec as
// for the fused backward); cnt and items: bin_count_words and
// bin_item_words 32-bit words; cleared: the first bin_clear_words of cnt are
// already zero
hipError_t binned_scatter(npm_ctx *ctx, const BinDesc &b, int64_t n, const float *pos,
                          const uint32_t *perm, const float *rec, int rec_stride,
                          const float *dgt, int rows, float *grad, uint32_t *cnt,
                          uint32_t *items, bool cleared, hipStream_t s);

// Grid scatter of the levels of level_mask (k_scatter.hip): chunks of the
// visiting order summed line by line in LDS, then one FP32 atomic per touched
// float.  dgt/rows: as above.
hipError_t chunk_scatter(const Net &net, int64_t n, const float *pos, const uint32_t *perm,
                         const float *rec, int rec_stride, const float *dgt, int rows,
                         float *grad, uint32_t level_mask, hipStream_t s);

// Whether the training tile kernel on encoded features (k_train.hip) takes the
// network; the gathering kernel (k_fused.hip) takes the others.  In FP32 the
// weight images and planes of the wide NPM-product input exceed the LDS, and
// the sums of the selection row beside three hidden layers the registers: 133
// would be spilled, and around spilled registers this compiler's rewriting of
// the matrix instructions' sums has given wrong weight gradients, so that no
// shape that spills is built (200,001 vertices on the 16-level hash grid with
// the selection output, spilling 490 us, gathering 506; 30,001 vertices 167 and
// 154).
inline bool train_tile_takes(const Net &net)
{
    return net.cfg.precision == NPM_PREC_BF16 ||
           (net.mlp.in_p <= 32 && !(net.cfg.learn_selection && net.mlp.n_hidden >= 3));
}

// fused path (k_query.hip, k_fused.hip)
// whether the fused kernels are instantiated for the network's shape (the
// dispatch tables of k_fused.hip)
bool fused_shape_supported(const Net &net);
// Queries of at most this many vertices (a 32-vertex tile for each of the 1,024
// SIMDs) run one wave per block with the weights in registers
// (k_query_small); a larger batch gives a SIMD several tiles, which then share
// one weight image in LDS.  On the 8-level dense grid, FP32, 4,096 vertices
// 20.3 -> 16.3 us, 32,768 23.0 -> 20.9 us, and 65,536 would be 41 against 34 us.
constexpr int64_t kQuerySmall = 1 << 15;
// Of those, the ones of at most this many are split over more blocks (k_query.hip).
constexpr int64_t kQueryTiny = 2048;
// Queries of more vertices than this on a grid with hashed levels encode the
// batch level by level first (k_encode.hip): the second launch costs 3 us,
// and up to here gathering every corner of a tile at once is no slower.  16
// levels, 2^19 entries, gathered / encoded first: FP32 20,011 vertices 33.0 /
// 38.5 us, 28,001 39.3 / 42.4, 32,767 40.8 / 43.9 (2^17 entries, 32,767: 33.2 /
// 37.6), 50,001 78 / 52; with the wide NPM-product input, whose first layer the
// gathers wait for, 20,001 35.4 / -, 25,001 - / 37.0, 32,767 43.9 / 39.1; BF16
// 16,384 22.1 / 22.3, 20,011 24.5 / 23.3, 30,001 - / 25.9, 32,767 29.0 / -.  2^20 vertices against the
// spatially ordered gather kernel with its sort and un-permute: FP32 711 -> 666
// us, BF16 588 -> 420.  A dense grid's levels stay in the caches, and its corners
// are gathered in the query kernel at every size (8 levels, 921,600 vertices,
// FP32 296 us against 355 encoded first).
constexpr int64_t kFeatQuery32 = kQuerySmall - 1, kFeatQuery32Wide = 24576, kFeatQuery16 = 16384;

// perm/inv (optional): visiting order and its inverse; the outputs then go
// through `stage` (n slots of 40 floats) and an un-permuting pass.  feat
// (optional, without perm): a buffer of feat_words(net, n) words for the
// batch's grid features, encoded level by level in a pass of its own
hipError_t fused_query(npm_ctx *ctx, int64_t n, const float *pos, const float *aux,
                       const float *dir, uint64_t seed, uint32_t stream_id, float *lobes,
                       float *pdf, float *sdir, float *spdf, const uint32_t *perm,
                       const uint32_t *inv, const float *rec, float *stage, hipStream_t s,
                       float *sel = nullptr, void *feat = nullptr);
// perm (optional): the order in which to visit the vertices; dg_tiles: the
// per-tile dG buffer (required when grad is set); bins (optional): the levels
// to scatter through the binned pass, with the context's bin buffers; feat
// (optional, with grad): feat_words(net, n) words for the grid features, then
// encoded level by level for the tile kernel that reads them (k_train.hip)
hipError_t fused_backward(npm_ctx *ctx, int64_t n, const float *pos, const float *aux,
                          const float *dir, const float *rad, const float *spdf, float *grad,
                          double *loss_out, const uint32_t *perm, const float *rec,
                          float *dg_tiles, const BinDesc *bins, hipStream_t s,
                          const float *bsdf = nullptr, void *feat = nullptr);

}  // namespace npm
