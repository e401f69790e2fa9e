// Binned grid scatter (the gradient of Sec. 4.2 pushed through the
// trilinear interpolation of Sec. 5.1 into the hashed levels).
//
// On a hashed level neighbouring vertices land on unrelated table entries, so
// no spatial order or line table brings their corners together, and every
// corner becomes one FP32 atomic request executed at the memory side -- the
// rate that bounds the plain scatter.  Here the corner contributions of those
// levels are instead binned by table slice (kBinSliceFloats floats) and each
// slice is summed by one block.  An item is a pair of x-neighbour corners:
// the hash takes x unmultiplied, so slot(x + 1) = slot(x) ^ (x ^ (x + 1)),
// which stays in the slice of slot(x) while the resolution is below the
// slice's entry count (the plan checks it).  An item holds the key (the
// lower corner's entry within the slice, and above bit 16 the xor to the
// upper one), the x fraction f and the F values wy wz dG; the reduce adds
// (1 - f) times them to the lower entry and f times them to the upper one.
//
//   count   per chunk of kBinChunk visiting slots, the number of items of
//           every (level, slice) bin; the chunk's run of each bin follows the
//           runs counted before it (one add to the bin's total)
//   place   the chunk's items, ordered by bin in LDS and written out as
//           contiguous runs of (key, fraction, F values) records, the bins one
//           after the other in the item buffer
//   reduce  one block per bin: LDS accumulation of its items -- FP64, or in
//           the precision form 64-bit fixed point (no FP64) -- then one
//           coalesced read-add-write of the slice into the gradient
//
// Items are recomputed identically by count and place (same inputs, same
// arithmetic), so place fills each chunk's run exactly; every LDS and global
// index is still checked against its buffer.  The values are the atomic
// scatter's corner weights applied to dG in another grouping (wx (wy wz dG)
// instead of (wx wy wz) dG) and summed in another order.
#include <type_traits>

#include "device_math.h"

namespace npm {

namespace {

__device__ __forceinline__ void slot_position(const float *__restrict__ pos, const uint32_t *perm,
                                              const float *__restrict__ rec, int rec_stride,
                                              int64_t n, int64_t s, float p[3])
{
    if (rec) {
        const f32x4 a = *reinterpret_cast<const f32x4 *>(rec + (size_t)s * rec_stride);
        p[0] = a[0]; p[1] = a[1]; p[2] = a[2];
    } else {
        const int64_t v = perm ? (int64_t)perm[s] : s;
        p[0] = pos[v]; p[1] = pos[n + v]; p[2] = pos[2 * n + v];
    }
}

// dG of slot s, level l, read from the per-tile rows (row l F + f, 32 slots).
// The loads are only issued here: the passes read the next level's values
// while they bin the current level's, and test them when that level comes.
template <int F>
__device__ __forceinline__ void slot_dg(const float *__restrict__ dgt, int rows, int64_t s, int l,
                                        float d[F])
{
    const float *src = dgt + (size_t)(s >> 5) * rows * 32 + (s & 31);
#pragma unroll
    for (int f = 0; f < F; ++f) d[f] = src[(l * F + f) * 32];
}

// Takes the prefetched values into d; true if any is non-zero (a slot whose
// dG is zero at a level adds nothing there and is not binned).
template <int F>
__device__ __forceinline__ bool take_dg(const float dn[F], float d[F])
{
    bool any = false;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        d[f] = dn[f];
        any |= dn[f] != 0.0f;
    }
    return any;
}

// Hashed table slot of the lower corner of pair p (y offset p & 1, z offset
// p >> 1) of the cell, the xor m to its x-neighbour's slot, and the pair's
// weight wy wz (the same hash as the atomic scatter).
__device__ __forceinline__ uint32_t pair_slot(const int c[3], const float fr[3], int p,
                                              uint32_t mask, uint32_t &m, float &wyz)
{
    const int by = p & 1, bz = (p >> 1) & 1;
    const uint32_t X = c[0], Y = c[1] + by, Z = c[2] + bz;
    m = (X ^ (X + 1u)) & mask;
    wyz = (by ? fr[1] : 1.0f - fr[1]) * (bz ? fr[2] : 1.0f - fr[2]);
    return (X ^ (Y * 2654435761u) ^ (Z * 805459861u)) & mask;
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x, int lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(x, o, 64);
        if (lane >= o) x += t;
    }
    return x;
}

}  // namespace

// The binned levels j0 .. j1 - 1 of a block's share (blockIdx.y of gridDim.y).
__device__ __forceinline__ void level_share(int nb, int &j0, int &j1)
{
    j0 = nb * (int)blockIdx.y / (int)gridDim.y;
    j1 = nb * ((int)blockIdx.y + 1) / (int)gridDim.y;
}

// Exclusive prefix sum of the m <= 2 kBinChunk words of v into out (LDS), by a
// block of kBinChunk threads; wsum: 16 words of LDS.
__device__ __forceinline__ void block_exclusive_scan(const uint32_t *__restrict__ v, int m,
                                                     uint32_t *out, uint32_t *wsum)
{
    static_assert(kBinMaxBins <= 2 * kBinChunk && kBinChunk == 1024, "two bins a thread, 16 waves");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t x0 = 2 * t < m ? v[2 * t] : 0u, x1 = 2 * t + 1 < m ? v[2 * t + 1] : 0u;
    const uint32_t inc = wave_inclusive_scan(x0 + x1, lane);
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    if (wave == 0) {
        const uint32_t ws = lane < 16 ? wsum[lane] : 0u;
        const uint32_t wi = wave_inclusive_scan(ws, lane);
        if (lane < 16) wsum[lane] = wi - ws;
    }
    __syncthreads();
    const uint32_t e = wsum[wave] + inc - x0 - x1;
    if (2 * t < m) out[2 * t] = e;
    if (2 * t + 1 < m) out[2 * t + 1] = e + x0;
}

// Clears the bins' totals and the two words of the batch after them.
__global__ void k_bin_zero(uint32_t *__restrict__ tot, int words)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < words) tot[i] = 0u;
}

// Bound by the LDS counts and the reads of position and dG.  The offsets come
// from one add per chunk and bin to the bin's total (0.65 M at 2^20 vertices, a
// few microseconds), which replaced three passes over chunk-major counters
// (16 us together, 25 more where another stream's blocks held the CUs); a
// chunk's runs lie together, one line request for 16 of them.
//
// Per chunk: {offset within the bin, items} of every bin into run[chunk][bin],
// the largest finite |dG| into tot[nbins], which scales the fixed-point reduce,
// and into tot[nbins + 1] whether a binned dG is infinite or NaN.
template <int F>
__global__ __launch_bounds__(kBinChunk) void k_bin_count(GridDesc g, BinDesc bd, int64_t n,
                                                         const float *__restrict__ pos,
                                                         const uint32_t *perm,
                                                         const float *__restrict__ rec,
                                                         int rec_stride,
                                                         const float *__restrict__ dgt, int rows,
                                                         uint2 *__restrict__ run,
                                                         uint32_t *__restrict__ tot)
{
    // NC copies of the histogram, lane t counting in copy t mod NC: fewer lanes of
    // one instruction on one counter (the copies sit HS words apart, off each
    // other's banks); the chunk's count is their sum (precision-form step
    // 2.06 -> 2.04 ms, FP32 within noise)
    constexpr int NC = 4, HS = kBinMaxBins + 1;
    __shared__ uint32_t hist[NC * HS];
    __shared__ int s_lv[NPM_MAX_LEVELS], s_res[NPM_MAX_LEVELS];
    __shared__ uint32_t s_max, s_odd;
    int j0, j1;
    level_share(bd.nb, j0, j1);
    const int k0 = j0 * bd.ns, nk = (j1 - j0) * bd.ns;
    for (int k = threadIdx.x; k < nk; k += kBinChunk)
#pragma unroll
        for (int r = 0; r < NC; ++r) hist[r * HS + k] = 0u;
    if (threadIdx.x == 0) s_max = s_odd = 0u;
    if (threadIdx.x < NPM_MAX_LEVELS) {
        s_lv[threadIdx.x] = bd.lv[threadIdx.x];
        s_res[threadIdx.x] = g.res[threadIdx.x];
    }
    __syncthreads();
    const int64_t s = blockIdx.x * (int64_t)kBinChunk + threadIdx.x;
    uint32_t *hc = hist + (threadIdx.x & (NC - 1)) * HS;
    uint32_t dmax = 0u;     // largest finite |dG| the chunk bins (bounds every finite item): its bits
    bool odd = false;       // an infinite or NaN one among them
    if (s < n) {
        float p[3];
        slot_position(pos, perm, rec, rec_stride, n, s, p);
        float dn[F];
        slot_dg<F>(dgt, rows, s, s_lv[j0], dn);
        for (int j = j0; j < j1; ++j) {
            const int l = s_lv[j];
            float d[F];
            const bool any = take_dg<F>(dn, d);
            if (j + 1 < j1) slot_dg<F>(dgt, rows, s, s_lv[j + 1], dn);
            if (!any) continue;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                // non-negative floats order as their bit patterns
                const uint32_t u = __float_as_uint(d[f]) & 0x7fffffffu;
                const bool finite = u < 0x7f800000u;
                dmax = max(dmax, finite ? u : 0u);
                odd |= !finite;
            }
            int c[3];
            float fr[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) lattice_cell(p[a], s_res[l], c[a], fr[a]);
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                uint32_t m;
                float wyz;
                const uint32_t slot = pair_slot(c, fr, pr, g.table_mask, m, wyz);
                atomicAdd(&hc[(j - j0) * bd.ns + (int)(slot >> bd.log2s)], 1u);
            }
        }
    }
    atomicMax(&s_max, dmax);
    if (odd) s_odd = 1u;
    __syncthreads();
    for (int k = threadIdx.x; k < nk; k += kBinChunk) {
        uint32_t c = 0u;
#pragma unroll
        for (int r = 0; r < NC; ++r) c += hist[r * HS + k];
        const uint32_t o = c ? atomicAdd(&tot[k0 + k], c) : 0u;
        run[(size_t)blockIdx.x * bd.nbins + k0 + k] = make_uint2(o, c);
    }
    if (threadIdx.x == 0 && s_max) atomicMax(&tot[bd.nbins], s_max);
    if (threadIdx.x == 0 && s_odd) atomicMax(&tot[bd.nbins + 1], 1u);
}

template <int F>
__global__ __launch_bounds__(kBinChunk) void k_bin_place(GridDesc g, BinDesc bd, int64_t n,
                                                         const float *__restrict__ pos,
                                                         const uint32_t *perm,
                                                         const float *__restrict__ rec,
                                                         int rec_stride,
                                                         const float *__restrict__ dgt, int rows,
                                                         const uint2 *__restrict__ run,
                                                         const uint32_t *__restrict__ tot,
                                                         uint32_t *__restrict__ base,
                                                         uint32_t *__restrict__ items)
{
    constexpr int W = 2 + F;                 // words per item: key, fraction, F values
    constexpr int CAP = kBinChunk * 4;       // items (corner pairs) of one chunk and level
    __shared__ __attribute__((aligned(16))) uint32_t st[CAP * W];
    __shared__ uint16_t sb[CAP];
    __shared__ int s_lv[NPM_MAX_LEVELS], s_res[NPM_MAX_LEVELS];
    __shared__ uint32_t wsum[16];
    // sized by the launch: each bin's run start and length, then the level's
    // local bases and ranks (bin_place_lds_bytes)
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    uint32_t *gd = dyn, *cn = dyn + bd.nbins, *lb = cn + bd.nbins, *rk = lb + bd.ns + 1;
    const int t = threadIdx.x, lane = t & 63;
    if (t < NPM_MAX_LEVELS) {
        s_lv[t] = bd.lv[t];
        s_res[t] = g.res[t];
    }
    const int64_t chunk = blockIdx.x;
    int j0, j1;
    level_share(bd.nb, j0, j1);
    // this chunk's run of every bin of its levels (start, length)
    block_exclusive_scan(tot, bd.nbins, gd, wsum);
    __syncthreads();
    if (blockIdx.x == 0 && blockIdx.y == 0) {          // for the reduce
        for (int kk = t; kk < bd.nbins; kk += kBinChunk) base[kk] = gd[kk];
        __syncthreads();
    }
    for (int kk = j0 * bd.ns + t; kk < j1 * bd.ns; kk += kBinChunk) {
        const uint2 r = run[(size_t)chunk * bd.nbins + kk];
        gd[kk] += r.x;
        cn[kk] = r.y;
    }
    const int64_t s = chunk * kBinChunk + t;
    const bool live = s < n;
    float p[3] = {0.0f, 0.0f, 0.0f};
    if (live) slot_position(pos, perm, rec, rec_stride, n, s, p);
    const uint32_t smask = (1u << bd.log2s) - 1u;
    __syncthreads();
    float dn[F];
#pragma unroll
    for (int f = 0; f < F; ++f) dn[f] = 0.0f;
    if (live) slot_dg<F>(dgt, rows, s, s_lv[j0], dn);
    for (int j = j0; j < j1; ++j) {
        // local base of the chunk's run of each bin of the level
        if (t < 64) {
            uint32_t c0 = 0u;
            for (int k0 = 0; k0 < bd.ns; k0 += 64) {
                const int k = k0 + lane;
                uint32_t c = 0u;
                if (k < bd.ns) {
                    c = cn[j * bd.ns + k];
                    rk[k] = 0u;
                }
                const uint32_t inc = wave_inclusive_scan(c, lane);
                if (k < bd.ns) lb[k] = c0 + inc - c;
                c0 += __shfl(inc, 63, 64);
            }
            if (lane == 0) lb[bd.ns] = c0;
        }
        __syncthreads();
        const int l = s_lv[j];
        float d[F];
        const bool any = take_dg<F>(dn, d);
        if (live && j + 1 < j1) slot_dg<F>(dgt, rows, s, s_lv[j + 1], dn);
        if (live && any) {
            int c[3];
            float fr[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) lattice_cell(p[a], s_res[l], c[a], fr[a]);
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                uint32_t m;
                float wyz;
                const uint32_t slot = pair_slot(c, fr, pr, g.table_mask, m, wyz);
                const int k = (int)(slot >> bd.log2s);
                const uint32_t q = lb[k] + atomicAdd(&rk[k], 1u);
                if (q < lb[k + 1] && q < (uint32_t)CAP) {
                    if constexpr (W == 4) {
                        uint4 r;
                        r.x = (slot & smask) | (m << 16);
                        r.y = __float_as_uint(fr[0]);
                        r.z = __float_as_uint(wyz * d[0]);
                        r.w = __float_as_uint(wyz * d[1]);
                        *reinterpret_cast<uint4 *>(st + q * W) = r;
                    } else {
                        st[q * W] = (slot & smask) | (m << 16);
                        st[q * W + 1] = __float_as_uint(fr[0]);
#pragma unroll
                        for (int f = 0; f < F; ++f) st[q * W + 2 + f] = __float_as_uint(wyz * d[f]);
                    }
                    sb[q] = (uint16_t)k;
                }
            }
        }
        __syncthreads();
        const uint32_t tot = min(lb[bd.ns], (uint32_t)CAP);
        for (uint32_t q = t; q < tot; q += kBinChunk) {
            const int k = sb[q];
            if (k >= bd.ns) continue;
            const uint32_t dst = gd[j * bd.ns + k] + (q - lb[k]);
            if (dst < bd.cap) {
                uint32_t *it = items + (size_t)dst * W;
                if constexpr (W == 4) {
                    // nontemporal: the records are read once, by the reduce, after
                    // every chunk has written its own (FP32 step 2.75 -> 2.73 ms,
                    // precision form 2.11 -> 2.07 ms with the reduce's loads below)
                    __builtin_nontemporal_store(*reinterpret_cast<const f32x4 *>(st + q * W),
                                                reinterpret_cast<f32x4 *>(it));
                } else {
#pragma unroll
                    for (int w = 0; w < W; ++w) it[w] = st[q * W + w];
                }
            }
        }
        __syncthreads();
    }
}

// One block per bin: the slice's sums in LDS, then one coalesced
// read-add-write of the slice into the gradient.  The sums are FP64 (LDS
// FP64 atomic adds run several times faster than FP32 ones on this chip, and
// the wider sum rounds once, when it is added to the FP32 gradient), or, in
// the precision form (FIXED), 64-bit fixed point: with every finite corner value
// below the batch's largest finite |dG|, M < 2^e, and 2c corner values in the bin of
// c items (2c <= 2^b), the scale 2^(62 - e - b) keeps every entry's sum below
// 2^62; each value is rounded to a multiple of 2^(e + b - 62) (below 1e-12 of
// M for any bin of at most 2^22 items) and the sum is exact in any order.  An
// infinite or NaN value goes to the gradient itself, as a float.
//
// Bound by the items' 16 bytes and the LDS adds, which a batch of loads
// followed by its adds paid one after the other: the next batch is in flight
// while one is added, and a feature's sums lie together, so that one add's
// lanes spread over all the banks and not every F-th (FP64, 10 levels of 2^20
// vertices: 277 -> 247 us; fixed point 199 -> 195, its 671 MB at 3.4 TB/s, the
// 640 blocks making two and a half rounds of the chip).
template <int F, bool FIXED>
__global__ __launch_bounds__(kBinReduceThreads) void k_bin_reduce(GridDesc g, BinDesc bd,
                                                                  const uint32_t *__restrict__ tot,
                                                                  const uint32_t *__restrict__ base,
                                                                  const uint32_t *__restrict__ items,
                                                                  float *__restrict__ grad)
{
    constexpr int NT = kBinReduceThreads, U = kBinReduceBatch;
    using AccT = typename std::conditional<FIXED, unsigned long long, double>::type;
    __shared__ AccT acc[kBinSliceFloats];
    constexpr int W = 2 + F;                 // words per item: key, fraction, F values
    const int k = blockIdx.x, j = k / bd.ns, slice = k - j * bd.ns;
    const uint32_t S = 1u << bd.log2s;
    const int nf = (int)S * F;
    const uint64_t beg = base[k];
    const uint64_t end = min(beg + tot[k], (uint64_t)bd.cap);
    float *dst = grad + ((size_t)g.offset[bd.lv[j]] + (size_t)slice * S) * F;
    int kx = 0;                                  // fixed point: the scale is 2^kx
    bool odd = false;                            // the batch has infinite or NaN values (uniform)
    if constexpr (FIXED) {
        const float M = __uint_as_float(tot[bd.nbins]);
        odd = tot[bd.nbins + 1] != 0u;
        if (!(M > 0.0f || odd) || end <= beg) return;   // nothing to add (block-uniform)
        int e;
        frexpf(M, &e);                           // M < 2^e
        const uint64_t c = 2 * (end - beg);                            // corner values
        const int b = c > 1 ? 64 - __clzll((long long)(c - 1)) : 0;   // c <= 2^b
        kx = 62 - e - b;
    }
    for (int i = threadIdx.x; i < nf; i += NT) acc[i] = AccT(0);
    __syncthreads();
    auto add1 = [&](uint32_t e, float v) {
        if constexpr (FIXED)
            __hip_atomic_fetch_add(&acc[e], (unsigned long long)__float2ll_rn(ldexpf(v, kx)),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_fetch_add(&acc[e], (double)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // item: (1 - fx) v to the lower corner's entry, fx v to the upper one's
    auto add = [&](uint32_t key, float fx, const float *v) {
        const uint32_t e0 = key & 0xffffu, e1 = e0 ^ (key >> 16);
        if (e0 < S && e1 < S) {
            const float w0 = 1.0f - fx;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                if (FIXED && odd && !isfinite(v[f])) {
                    unsafeAtomicAdd(dst + (size_t)e0 * F + f, w0 * v[f]);
                    unsafeAtomicAdd(dst + (size_t)e1 * F + f, fx * v[f]);
                    continue;
                }
                add1(f * S + e0, w0 * v[f]);
                add1(f * S + e1, fx * v[f]);
            }
        }
    };
    uint64_t i = beg + threadIdx.x;
    // U items in flight per thread besides the U being added
    // one item: its W words (one 16-byte nontemporal load at F = 2: each record
    // is read once)
    auto load = [&](uint64_t ii, uint32_t &e, float &fx, float *v) {
        const uint32_t *it = items + ii * W;
        if constexpr (W == 4) {
            const f32x4 r = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(it));
            e = __float_as_uint(r[0]);
            fx = r[1];
            v[0] = r[2];
            v[1] = r[3];
        } else {
            e = it[0];
            fx = __uint_as_float(it[1]);
#pragma unroll
            for (int f = 0; f < F; ++f) v[f] = __uint_as_float(it[2 + f]);
        }
    };
    const uint64_t step = (uint64_t)U * NT;
    uint32_t e[U];
    float fx[U], v[U][F];
    bool more = i + (uint64_t)(U - 1) * NT < end;
    if (more)
#pragma unroll
        for (int u = 0; u < U; ++u) load(i + (uint64_t)u * NT, e[u], fx[u], v[u]);
    while (more) {
        i += step;
        more = i + (uint64_t)(U - 1) * NT < end;
        uint32_t en[U];
        float fn[U], vn[U][F];
        if (more)
#pragma unroll
            for (int u = 0; u < U; ++u) load(i + (uint64_t)u * NT, en[u], fn[u], vn[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) add(e[u], fx[u], v[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            e[u] = en[u];
            fx[u] = fn[u];
#pragma unroll
            for (int f = 0; f < F; ++f) v[u][f] = vn[u][f];
        }
    }
    for (; i < end; i += NT) {
        load(i, e[0], fx[0], v[0]);
        add(e[0], fx[0], v[0]);
    }
    __syncthreads();
    for (int i2 = threadIdx.x; i2 < nf; i2 += NT) {
        const int at = (i2 % F) * (int)S + i2 / F;
        if constexpr (FIXED) {
            const long long a = (long long)acc[at];
            if (a == 0) continue;
            const float v = ldexpf(__ll2float_rn(a), -kx);
            if (odd) unsafeAtomicAdd(dst + i2, v);     // beside this block's float adds
            else dst[i2] += v;
        } else {
            const double a = acc[at];
            if (a != 0.0) dst[i2] += (float)a;
        }
    }
}

// Which levels are binned, and the sizes of the pass: every hashed level of
// an unordered batch; of a spatially ordered one, the hashed levels with
// D_l >= kBinMinResOrdered (coarser ones share lines within a chunk).
bool bin_plan(const Net &net, int64_t n, bool ordered, BinDesc *out)
{
    const GridDesc &g = net.grid;
    const int F = g.feat;
    if (n <= 0 || !g.hashed_mask || (F != 1 && F != 2 && F != 4)) return false;
    BinDesc b{};
    for (int l = 0; l < g.n_levels; ++l)
        if (((g.hashed_mask >> l) & 1u) && (!ordered || g.res[l] >= kBinMinResOrdered))
            b.lv[b.nb++] = l;
    if (b.nb == 0) return false;
    int log2t = 0;
    while ((1u << log2t) <= g.table_mask) ++log2t;
    static_assert(kBinSliceFloats <= 65536, "slice entries and their xor are stored in 16 bits");
    int log2s = 0;
    while ((1 << (log2s + 1)) * F <= kBinSliceFloats) ++log2s;
    b.log2s = std::min(log2s, log2t);
    b.ns = 1 << (log2t - b.log2s);
    b.nbins = b.nb * b.ns;
    if (b.ns > kBinMaxSlices || b.nbins > kBinMaxBins) return false;
    // an x-neighbour pair shares a slice while x + 1 <= D_l < 2^log2s
    for (int j = 0; j < b.nb; ++j)
        if ((int64_t)g.res[b.lv[j]] >= ((int64_t)1 << b.log2s)) return false;
    b.n_chunks = (n + kBinChunk - 1) / kBinChunk;
    b.cap = n * 4 * b.nb;
    if (b.cap >= ((int64_t)1 << 32) - 1 || (int64_t)b.nbins * b.n_chunks + 1 >= ((int64_t)1 << 31))
        return false;
    *out = b;
    return true;
}

// the bins' totals and the batch's two words (bin_clear_words, zero before the
// pass), the bins' starts, then the chunks' runs (two words per bin and chunk)
int bin_clear_words(const BinDesc &b) { return b.nbins + 2; }
static size_t bin_head_words(const BinDesc &b) { return 2 * (size_t)b.nbins + 2; }   // even: uint2 runs

size_t bin_count_words(const BinDesc &b)
{
    return bin_head_words(b) + 2 * (size_t)b.nbins * (size_t)b.n_chunks;
}

// items: cap records of (key, x fraction, F FP32 values)
size_t bin_item_words(const BinDesc &b, int feat)
{
    return (size_t)b.cap * (size_t)(2 + feat);
}

template <int F>
static void launch_bins(const GridDesc &g, const BinDesc &b, int64_t n, const float *pos,
                        const uint32_t *perm, const float *rec, int rec_stride, const float *dgt,
                        int rows, float *grad, uint32_t *cnt, uint32_t *items, int phase,
                        bool fixed, hipStream_t s)
{
    uint32_t *tot = cnt, *base = cnt + bin_clear_words(b);
    uint2 *run = reinterpret_cast<uint2 *>(cnt + bin_head_words(b));
    // a chunk's levels go to one block, or are shared by several where the
    // chunks alone are fewer than two blocks a CU (32,771 vertices, 12 levels:
    // place 37 -> 10 us; 100,003 vertices, 10 levels: 36 -> 26)
    const int gy = (int)std::min<int64_t>(b.nb, (511 + b.n_chunks) / b.n_chunks);
    const dim3 grid((unsigned)b.n_chunks, (unsigned)gy);
    switch (phase) {
    case 0:
        hipLaunchKernelGGL(k_bin_zero, dim3((bin_clear_words(b) + 255) / 256), dim3(256), 0, s, tot,
                           bin_clear_words(b));
        break;
    case 1:
        hipLaunchKernelGGL(k_bin_count<F>, grid, dim3(kBinChunk), 0, s, g, b, n, pos, perm, rec,
                           rec_stride, dgt, rows, run, tot);
        break;
    case 2:
        hipLaunchKernelGGL(k_bin_place<F>, grid, dim3(kBinChunk),
                           (size_t)(2 * b.nbins + 2 * b.ns + 1) * 4, s, g, b, n, pos, perm, rec,
                           rec_stride, dgt, rows, run, tot, base, items);
        break;
    default:
        if (fixed)
            hipLaunchKernelGGL((k_bin_reduce<F, true>), dim3(b.nbins), dim3(kBinReduceThreads), 0, s,
                               g, b, tot, base, items, grad);
        else
            hipLaunchKernelGGL((k_bin_reduce<F, false>), dim3(b.nbins), dim3(kBinReduceThreads), 0, s,
                               g, b, tot, base, items, grad);
        break;
    }
}

hipError_t binned_scatter(npm_ctx *ctx, const BinDesc &b, int64_t n, const float *pos,
                          const uint32_t *perm, const float *rec, int rec_stride,
                          const float *dgt, int rows, float *grad, uint32_t *cnt,
                          uint32_t *items, bool cleared, hipStream_t s)
{
    const GridDesc &g = ctx->net.grid;
    // the precision form sums in fixed point (no FP64)
    const bool fx = ctx->net.cfg.precision == NPM_PREC_BF16;
    static const char *names[4] = {"bin_zero", "bin_count", "bin_place", "bin_reduce"};
    for (int phase = cleared ? 1 : 0; phase < 4; ++phase) {
        int tok;
        timed_begin(ctx, names[phase], s, &tok);
        switch (g.feat) {
        case 1: launch_bins<1>(g, b, n, pos, perm, rec, rec_stride, dgt, rows, grad, cnt, items, phase, fx, s); break;
        case 2: launch_bins<2>(g, b, n, pos, perm, rec, rec_stride, dgt, rows, grad, cnt, items, phase, fx, s); break;
        default: launch_bins<4>(g, b, n, pos, perm, rec, rec_stride, dgt, rows, grad, cnt, items, phase, fx, s); break;
        }
        timed_end(ctx, tok, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace npm
