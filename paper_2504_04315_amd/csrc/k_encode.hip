// Level-major grid encoding (Sec. 5.1): the trilinear features of a whole
// batch, one grid level after the other, written feature-major.
//
// What bounds it: the rate at which the L1s take in 128-byte lines from L2,
// about 160 G lines/s for the chip whether the level's table is resident or
// not -- on a fine hashed level a vertex's eight corners lie on four lines
// (28 us a level; by counters, all 16 levels of 2^20 vertices in the caller's
// order make 74 M L2 requests, 86 % hits, in 350 us).
// Level-major order keeps one table (4 MB FP32, 2 MB FP16 at 2^19 entries)
// live at a time, which each XCD's 4 MB L2 holds, so that the gathers are L2
// hits; a kernel that takes all levels of a tile at once misses L2 instead.
//
// A pair of adjacent lanes takes one vertex: lane x of the pair loads the
// four corners with x offset x, so that the two lanes of an instruction meet
// on one line (x-neighbours are adjacent in a dense level, and in a hashed
// one 15 times out of 16 within a 128-byte line), and the pair then swaps
// halves by DPP: each lane sums half of the level's features over all eight
// corners, in the same order as a lane that holds them all.  2^20 vertices on
// the 16-level grid (2^19 entries, F = 2), caller's order: 475 us with a lane
// per vertex -> 341 us FP32, 372 -> 277 us FP16; spatially sorted 262 -> 206
// and 193 -> 165 us.
#include "device_math.h"

namespace npm {

namespace {

// Value of the neighbouring lane (lane ^ 1).
__device__ __forceinline__ float pair_swap(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));
}

// The F features of table entry e as loaded (words), and as floats.
template <int F, bool HALF> struct EncWord;
template <> struct EncWord<1, false> { using T = float; };
template <> struct EncWord<2, false> { using T = float2; };
template <> struct EncWord<4, false> { using T = float4; };
template <> struct EncWord<1, true> { using T = __half; };
template <> struct EncWord<2, true> { using T = __half2; };
template <> struct EncWord<4, true> { using T = uint2; };

template <int F, bool HALF>
__device__ __forceinline__ void enc_floats(const typename EncWord<F, HALF>::T &r, float *v)
{
    if constexpr (HALF) {
        if constexpr (F == 1) {
            v[0] = __half2float(r);
        } else if constexpr (F == 2) {
            v[0] = __low2float(r); v[1] = __high2float(r);
        } else {
            const __half2 lo = *reinterpret_cast<const __half2 *>(&r.x);
            const __half2 hi = *reinterpret_cast<const __half2 *>(&r.y);
            v[0] = __low2float(lo); v[1] = __high2float(lo);
            v[2] = __low2float(hi); v[3] = __high2float(hi);
        }
    } else {
        if constexpr (F == 1) {
            v[0] = r;
        } else if constexpr (F == 2) {
            v[0] = r.x; v[1] = r.y;
        } else {
            v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
        }
    }
}

}  // namespace

constexpr int kEncPairs = 2;             // vertices per lane pair (their loads in flight together)
constexpr int kEncBlock = 128 * kEncPairs;   // vertices per block of 256 threads

// The work is the list of (level, block of vertices) in level-major order.
// Workgroups go to the eight XCDs in turn (block b on XCD b mod 8), each with
// its own L2, and take their part of the list in one of two ways:
//   spans (nb > 0)  XCD i takes the list items [begin[i], begin[i + 1]), so
//                   that a table is fetched by one or two XCDs only;
//   levels in turn  (nb = 0; blockIdx.y = level) XCD i takes a contiguous
//                   eighth of the vertices on every level: the tables are
//                   fetched by all eight, but the load is even (and a sorted
//                   batch's XCD touches its own part of a coarse table).
struct EncSpans {
    int nb;
    int begin[9];
};

// HALF: the table is the FP16 copy.  B16: the features are rounded to BF16
// and stored in pairs, out[(feature / 2) n + v] holding features 2i, 2i + 1;
// otherwise FP32, out[feature n + v].
template <int F, bool HALF, bool B16>
__global__ __launch_bounds__(256) void k_grid_encode(GridDesc g, EncSpans sp, int64_t n,
                                                     const float *__restrict__ pos,
                                                     const float *__restrict__ rec, int rec_stride,
                                                     const void *__restrict__ table,
                                                     void *__restrict__ out)
{
    using WT = typename EncWord<F, HALF>::T;
    constexpr int U = kEncPairs;
    constexpr int FO = F > 1 ? F / 2 : 1;       // features a lane finishes
    const int x = threadIdx.x & 1, xcd = blockIdx.x & 7;
    int l;
    int64_t blk;
    if (sp.nb > 0) {
        const int item = sp.begin[xcd] + (int)(blockIdx.x >> 3);
        if (item >= sp.begin[xcd + 1]) return;
        l = item / sp.nb;
        blk = item - l * sp.nb;
    } else {
        l = blockIdx.y;
        blk = (int64_t)xcd * (gridDim.x >> 3) + (blockIdx.x >> 3);
        if (blk * kEncBlock >= n) return;
    }
    const int64_t v0 = blk * kEncBlock + (threadIdx.x >> 1);
    const int D = g.res[l];
    const uint32_t d1 = (uint32_t)D + 1u, off = g.offset[l];
    const bool hashed = (g.hashed_mask >> l) & 1u;
    const WT *tab = reinterpret_cast<const WT *>(table);
    WT raw[U][4];
    float fr[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t vu = v0 + 128 * u, v = vu < n ? vu : n - 1;
        float p[3];
        if (rec) {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(rec + (size_t)v * rec_stride);
            p[0] = a[0]; p[1] = a[1]; p[2] = a[2];
        } else {
            p[0] = pos[v]; p[1] = pos[n + v]; p[2] = pos[2 * n + v];
        }
        int c[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) lattice_cell(p[a], D, c[a], fr[u][a]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t X = c[0] + x, Y = c[1] + (q & 1), Z = c[2] + (q >> 1);
            const uint32_t e = off + (hashed ? ((X ^ (Y * 2654435761u) ^ (Z * 805459861u)) & g.table_mask)
                                             : X + d1 * (Y + d1 * Z));
            raw[u][q] = tab[e];
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float wx[2] = {1.0f - fr[u][0], fr[u][0]}, wy[2] = {1.0f - fr[u][1], fr[u][1]},
                    wz[2] = {1.0f - fr[u][2], fr[u][2]};
        float acc[FO];
#pragma unroll
        for (int f = 0; f < FO; ++f) acc[f] = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float own[F];
            enc_floats<F, HALF>(raw[u][q], own);
            const float w0 = wx[0] * wy[q & 1] * wz[q >> 1], w1 = wx[1] * wy[q & 1] * wz[q >> 1];
#pragma unroll
            for (int f = 0; f < FO; ++f) {
                // keep the features this lane finishes, hand over the other half
                float keep = own[f], send = own[f];
                if constexpr (F > 1) {
                    keep = x ? own[FO + f] : own[f];
                    send = x ? own[f] : own[FO + f];
                }
                const float got = pair_swap(send);
                const float c0 = x ? got : keep, c1 = x ? keep : got;
                acc[f] += w0 * c0;
                acc[f] += w1 * c1;
            }
        }
        const int64_t v = v0 + 128 * u;
        if (v >= n) continue;
#pragma unroll
        for (int f = 0; f < FO; ++f) {
            const int fo = l * F + x * (F > 1 ? FO : 0) + f;     // the feature
            if constexpr (B16) {
                // one 2-byte half of the pair's word (F = 4: both halves are this lane's)
                if (F == 1 && x) continue;
                reinterpret_cast<__bf16 *>(out)[((int64_t)(fo >> 1) * n + v) * 2 + (fo & 1)] = (__bf16)acc[f];
            } else {
                if (F == 1 && x) continue;
                reinterpret_cast<float *>(out)[(int64_t)fo * n + v] = acc[f];
            }
        }
    }
}

// Relative cost of a level's gathers, in hundredths of a table beyond L2: in
// the caller's order by the table's size (a small one sits in the L1s), in a
// sorted batch by the resolution (neighbouring vertices share lines).
static int level_cost(const GridDesc &g, int l, int64_t entries, bool sorted)
{
    if (sorted) {
        const int D = g.res[l];
        return D < 60 ? 22 : D < 100 ? 33 : D < 200 ? 45 : D < 400 ? 65 : 95;
    }
    const int64_t bytes = entries * g.feat * 4;
    return bytes < 100000 ? 35 : bytes < 500000 ? 55 : bytes < 3000000 ? 70 : 100;
}

// The spans of equal cost.
static EncSpans enc_spans(const GridDesc &g, int64_t n, bool sorted)
{
    EncSpans sp{};
    sp.nb = (int)((n + kEncBlock - 1) / kEncBlock);
    int64_t cost[NPM_MAX_LEVELS], total = 0;
    for (int l = 0; l < g.n_levels; ++l) {
        const int64_t pts = (int64_t)(g.res[l] + 1) * (g.res[l] + 1) * (g.res[l] + 1);
        cost[l] = level_cost(g, l, ((g.hashed_mask >> l) & 1u) ? (int64_t)g.table_mask + 1 : pts, sorted);
        total += cost[l];
    }
    for (int i = 1; i < 8; ++i) {
        const int64_t want = total * i;              // in eighths
        int64_t acc = 0;
        int l = 0;
        while (l < g.n_levels && (acc + cost[l]) * 8 <= want) acc += cost[l++];
        sp.begin[i] = l * sp.nb + (l < g.n_levels ? (int)((want - acc * 8) * sp.nb / (cost[l] * 8)) : 0);
    }
    sp.begin[8] = g.n_levels * sp.nb;
    return sp;
}

// Table bytes per vertex above which the spans are taken: below, every XCD's
// gathers outweigh its share of fetching the tables and the even load wins.
// Measured on the 16-level grid (49 MB FP32, 24 MB FP16), spans / in turn:
// caller's order FP32 4,096 vertices 6.7 / 7.1 us, 32,768 18.6 / 29.6,
// 100,003 40 / 61, 2^18 101 / 105, 2^19 201 / 185; FP16 100,003 34 / 39,
// 2^18 89 / 81; sorted FP32 100,003 34 / 46, 2^18 66 / 73, 2^19 125 / 121;
// FP16 100,003 28 / 30, 2^18 64 / 57.
constexpr int64_t kEncSpanBytes = 180;

hipError_t launch_grid_encode(const GridDesc &g, int64_t n, const float *pos, const float *rec,
                              int rec_stride, const float *grid32, const void *grid16, bool b16,
                              void *out, hipStream_t s)
{
    const int64_t nb = ((n + kEncBlock - 1) / kEncBlock + 7) / 8 * 8;
    EncSpans sp{};
    dim3 grid((unsigned)nb, (unsigned)g.n_levels);
    int64_t entries = 0;
    for (int l = 0; l < g.n_levels; ++l) {
        const int64_t pts = (int64_t)(g.res[l] + 1) * (g.res[l] + 1) * (g.res[l] + 1);
        entries += ((g.hashed_mask >> l) & 1u) ? (int64_t)g.table_mask + 1 : pts;
    }
    if (n * kEncSpanBytes < entries * g.feat * (b16 ? 2 : 4)) {
        sp = enc_spans(g, n, rec != nullptr);
        int most = 0;
        for (int i = 0; i < 8; ++i) most = std::max(most, sp.begin[i + 1] - sp.begin[i]);
        grid = dim3((unsigned)(8 * most), 1);
    }
    const dim3 block(256);
    const void *table = b16 ? grid16 : (const void *)grid32;
#define NPM_ENC(FV)                                                                                \
    if (b16)                                                                                       \
        hipLaunchKernelGGL((k_grid_encode<FV, true, true>), grid, block, 0, s, g, sp, n, pos, rec, \
                           rec_stride, table, out);                                                \
    else                                                                                           \
        hipLaunchKernelGGL((k_grid_encode<FV, false, false>), grid, block, 0, s, g, sp, n, pos,    \
                           rec, rec_stride, table, out)
    switch (g.feat) {
    case 1: NPM_ENC(1); break;
    case 2: NPM_ENC(2); break;
    case 4: NPM_ENC(4); break;
    default: return hipErrorInvalidValue;
    }
#undef NPM_ENC
    return hipGetLastError();
}

}  // namespace npm
