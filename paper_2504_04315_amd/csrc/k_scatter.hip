// Grid scatter of the levels the binned pass does not take: the transpose of
// the trilinear interpolation (Sec. 5.1), from the per-tile dG into the grid
// gradient.
//
// Memory-side FP32 atomics (21 G line requests/s on this chip) bound a scatter
// that sends every corner there.  In a spatially ordered batch neighbouring
// vertices share corners and neighbouring corners share 64-byte lines, so a
// block sums a chunk of consecutive slots in LDS first and sends each touched
// line once.  A window over the chunk's bounding box would be too large from
// resolutions of about 100 on (Morton runs of 1,024 vertices of a scene span
// thousands of lattice points there, and touch a few hundred lines), so the
// block keeps a hash table of lines: 512 slots of 16 floats.
//
// Work is dealt lane = vertex: a lane forms a vertex's eight corners once,
// keeps the sums of its run of vertices in registers while they stay in one
// cell, and merges with its neighbours' when those ended in the same cell; LDS
// adds to one address execute one after the other (11 cycles each, FP64), and
// on the coarse levels a whole wave lies in one cell.  Measured against one
// window per 32-vertex tile with a lane per (corner, feature): 8-level dense
// grid, 2^18 vertices, 174 -> 96 us; the six levels below resolution 100 of
// the 16-level hash grid, 2^20 vertices, 320 -> 170 us; 4-level dense grid,
// 16,384 vertices in the caller's order, 46 -> 19 us.  At 2^18 vertices the
// LDS adds are 40 us of it, the table lookups 25, loads and corner weights 40.
#include <type_traits>

#include "fused_tiles.h"

namespace npm {

namespace {

constexpr int kScThreads = 512;
constexpr int kScSlots = 512;              // lines a block holds
constexpr int kScLine = 16;                // floats per line (64 bytes)
constexpr int kScProbes = 6;
constexpr int kScSpill = 32;               // spilled corner pairs a wave writes at once
constexpr int64_t kScBlocks = 512;          // two blocks (76 KB of LDS each) on every CU
static_assert(2 * kScThreads <= 1 << 10, "headroom of the fixed-point sums");
constexpr uint32_t kScEmpty = 0xffffffffu;

// The sums are FP64, or in the precision form (FIXED, no FP64) 64-bit fixed
// point: with every |dG| of the chunk's level below 2^e the scale 2^(52 - e)
// keeps a corner's sum over at most 2^10 vertices below 2^62, each
// contribution rounded to a multiple of 2^(e - 53), and the sum is exact in any
// order.  A chunk whose dG holds an infinity or NaN adds that level's corners
// to the gradient as floats.
//
// Cell of a lane's run: lattice corner and whether the run holds anything.
struct RunCell {
    int x, y, z;
    bool have;
};

template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_mov64(uint64_t v)
{
    const uint32_t lo = (uint32_t)dpp_mov<CTRL>((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)dpp_mov<CTRL>((int)(uint32_t)(v >> 32));
    return (uint64_t)hi << 32 | lo;
}

// The sums: FP64, or (FIXED) 64-bit fixed point at the scale 2^k.
template <bool FIXED> struct ChunkSum {
    using T = double;
    int k = 0;
    __device__ __forceinline__ float scaled(float d) const { return d; }
    __device__ __forceinline__ static void add(T &a, float v) { a += (double)v; }
    __device__ __forceinline__ float value(T a) const { return (float)a; }
    __device__ __forceinline__ static uint64_t bits(T a) { return __builtin_bit_cast(uint64_t, a); }
    __device__ __forceinline__ static T from_bits(uint64_t b) { return __builtin_bit_cast(T, b); }
};
template <> struct ChunkSum<true> {
    using T = long long;
    int k = 0;
    __device__ __forceinline__ float scaled(float d) const { return ldexpf(d, k); }
    // v (below 2^52) rounded to an integer: a multiple of 2^30 and the rest,
    // both exact in float
    __device__ __forceinline__ static void add(T &a, float v)
    {
        const float hi = truncf(v * 0x1p-30f);
        const float lo = fmaf(-0x1p30f, hi, v);
        a += (long long)(int)hi * (1ll << 30) + (long long)(int)rintf(lo);
    }
    __device__ __forceinline__ float value(T a) const { return ldexpf(__ll2float_rn(a), -k); }
    __device__ __forceinline__ static uint64_t bits(T a) { return (uint64_t)a; }
    __device__ __forceinline__ static T from_bits(uint64_t b) { return (T)b; }
};

// One step of the lanes' merge: lane i (a multiple of 2 M within its 16-lane
// row) takes over lane i + M's sums if both runs ended in the same cell.
template <int M, int N, typename Sum>
__device__ __forceinline__ void merge_lanes(RunCell &c, typename Sum::T (&a)[N], int lane)
{
    constexpr int SHL = 0x100 + M, SHR = 0x110 + M;
    const bool lower = (lane & (2 * M - 1)) == 0, upper = (lane & (2 * M - 1)) == M;
    // (every lane takes part in the moves: no short circuit around them)
    const int uh = dpp_mov<SHL>((int)c.have), ux = dpp_mov<SHL>(c.x), uy = dpp_mov<SHL>(c.y),
              uz = dpp_mov<SHL>(c.z);
    const bool take = lower & c.have & (uh != 0) & (ux == c.x) & (uy == c.y) & (uz == c.z);
    if (!__any(take)) return;
    const int taken = dpp_mov<SHR>((int)take);
    const bool gone = upper & (taken != 0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const typename Sum::T t = Sum::from_bits(dpp_mov64<SHL>(Sum::bits(a[i])));
        if (take) a[i] += t;
    }
    if (gone) c.have = false;
}

}  // namespace

template <int F, bool FIXED, int R>
__global__ __launch_bounds__(kScThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void
k_scatter_chunk(GridDesc g, int64_t n, const float *__restrict__ pos, const uint32_t *perm,
                const float *__restrict__ rec, int rec_stride, const float *__restrict__ dgt,
                int rows, float *__restrict__ grad, uint32_t level_mask)
{
    using Sum = ChunkSum<FIXED>;
    using T = typename Sum::T;
    constexpr int LE = kScLine / F;                    // entries per line
    constexpr int LOG_LE = F == 1 ? 4 : F == 2 ? 3 : 2;
    constexpr int SPW = 2 + 2 * F;                     // words per spilled pair
    __shared__ __attribute__((aligned(16))) T acc[kScSlots * kScLine];
    __shared__ uint32_t keys[kScSlots];
    __shared__ uint32_t spill[kScThreads / 64][kScSpill * SPW];
    __shared__ uint32_t s_max[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < kScSlots * kScLine; i += kScThreads) acc[i] = T(0);
    for (int i = tid; i < kScSlots; i += kScThreads) keys[i] = kScEmpty;
    if (tid < 3) s_max[tid] = 0u;

    // the lane's run of R consecutive slots of the visiting order
    const int64_t v0 = ((int64_t)blockIdx.x * kScThreads + tid) * R;
    float px[R], py[R], pz[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t v = v0 + r < n ? v0 + r : n - 1;
        if (rec) {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(rec + (size_t)v * rec_stride);
            px[r] = a[0]; py[r] = a[1]; pz[r] = a[2];
        } else {
            const int64_t vv = visit(perm, v);
            px[r] = pos[vv]; py[r] = pos[n + vv]; pz[r] = pos[2 * n + vv];
        }
    }
    const float *dsrc = dgt + (size_t)((v0 < n ? v0 : 0) >> 5) * rows * 32 + (v0 & 31);
    __syncthreads();

    // levels blockIdx.y, blockIdx.y + gridDim.y, ... of the mask
    uint32_t mask = level_mask;
    for (int skip = blockIdx.y; skip > 0 && mask; --skip) mask &= mask - 1;
    for (int it = 0; mask; ++it) {
        const int l = __builtin_ctz(mask);
        for (int skip = gridDim.y; skip > 0 && mask; --skip) mask &= mask - 1;
        const int D = g.res[l];
        const uint32_t d1 = (uint32_t)D + 1u, off = g.offset[l];
        const bool hashed = (g.hashed_mask >> l) & 1u;
        float d[R][F];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int f = 0; f < F; ++f) d[r][f] = v0 + r < n ? dsrc[(l * F + f) * 32 + r] : 0.0f;
        Sum sum;
        bool direct = false;
        if constexpr (FIXED) {
            uint32_t m = 0u;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int f = 0; f < F; ++f) m = max(m, __float_as_uint(d[r][f]) & 0x7fffffffu);
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
            if (lane == 0) atomicMax(&s_max[it % 3], m);
            __syncthreads();
            m = s_max[it % 3];
            // the slot of two levels on: last read before this barrier
            if (tid == 0) s_max[(it + 2) % 3] = 0u;
            if (m == 0u) continue;                     // nothing at this level (uniform)
            direct = m >= 0x7f800000u;                 // infinities and NaN add as floats
            int e;
            frexpf(__uint_as_float(m), &e);            // |d| < 2^e
            sum.k = 52 - e;
        }
        auto entry = [&](uint32_t X, uint32_t Y, uint32_t Z) {
            return off + (hashed ? ((X ^ (Y * 2654435761u) ^ (Z * 805459861u)) & g.table_mask)
                                 : X + d1 * (Y + d1 * Z));
        };
        auto find = [&](uint32_t line) -> int {
            uint32_t s = (line * 2654435769u) >> 23;
            static_assert(kScSlots == 1 << 9, "slots of the line table");
#pragma unroll 1
            for (int p = 0; p < kScProbes; ++p) {
                uint32_t k = __hip_atomic_load(&keys[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (k == kScEmpty) {
                    k = atomicCAS(&keys[s], kScEmpty, line);
                    if (k == kScEmpty) k = line;
                }
                if (k == line) return (int)s;
                s = (s + 1) & (kScSlots - 1);
            }
            return -1;
        };
        // position of feature f of entry e in its line's slot, spread over the
        // banks by the slot
        auto place = [&](int s, uint32_t e, int f) {
            return s * kScLine + ((f * LE + (int)(e & (LE - 1))) ^ ((s >> 1) & (kScLine - 1)));
        };
        // adds the run's sums of its cell's corners to their lines' slots
        auto flush = [&](const RunCell &c, const T (&a)[8 * F], bool on) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t Y = c.y + (p & 1), Z = c.z + (p >> 1);
                const uint32_t e0 = entry(c.x, Y, Z), e1 = entry(c.x + 1, Y, Z);
                int s0 = -1, s1 = -1;
                if (on) {
                    s0 = find(e0 >> LOG_LE);
                    s1 = (e1 >> LOG_LE) == (e0 >> LOG_LE) ? s0 : find(e1 >> LOG_LE);
#pragma unroll
                    for (int f = 0; f < F; ++f) {
                        if (s0 >= 0) __hip_atomic_fetch_add(&acc[place(s0, e0, f)], a[2 * p * F + f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (s1 >= 0) __hip_atomic_fetch_add(&acc[place(s1, e1, f)], a[(2 * p + 1) * F + f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
                // pairs that found no slot: 2 F lanes per pair add them to the
                // gradient, so that a pair's entries share line requests
                uint64_t todo = __ballot(on && (s0 < 0 || s1 < 0));
                while (todo) {
                    const int rank = __popcll(todo & ((1ull << lane) - 1ull));
                    const bool mine = (todo >> lane) & 1ull && rank < kScSpill;
                    const int cnt = min(__popcll(todo), kScSpill);
                    if (mine) {
                        uint32_t *q = spill[wave] + rank * SPW;
                        q[0] = s0 < 0 ? e0 : kScEmpty;
                        q[1] = s1 < 0 ? e1 : kScEmpty;
#pragma unroll
                        for (int i = 0; i < 2 * F; ++i)
                            q[2 + i] = __float_as_uint(sum.value(a[2 * p * F + i]));
                    }
                    wave_lds_fence();
                    for (int i = lane; i < cnt * 2 * F; i += 64) {
                        const uint32_t *q = spill[wave] + (i / (2 * F)) * SPW;
                        const int j = i % (2 * F);
                        const uint32_t e = q[j / F];
                        if (e != kScEmpty) unsafeAtomicAdd(grad + (size_t)e * F + j % F, __uint_as_float(q[2 + j]));
                    }
                    wave_lds_fence();
                    todo &= ~__ballot(mine);
                }
            }
        };
        T a[8 * F];
#pragma unroll
        for (int i = 0; i < 8 * F; ++i) a[i] = T(0);
        RunCell cur = {0, 0, 0, false};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            bool any = false;
#pragma unroll
            for (int f = 0; f < F; ++f) any |= d[r][f] != 0.0f;
            int cx, cy, cz;
            float fx, fy, fz;
            lattice_cell(px[r], D, cx, fx);
            lattice_cell(py[r], D, cy, fy);
            lattice_cell(pz[r], D, cz, fz);
            if (r > 0) {
                const bool out = any && cur.have && (cx != cur.x || cy != cur.y || cz != cur.z);
                if (__any(out)) {
                    flush(cur, a, out);
                    if (out)
#pragma unroll
                        for (int i = 0; i < 8 * F; ++i) a[i] = T(0);
                }
            }
            if (any) {
                cur = {cx, cy, cz, true};
                if (FIXED && direct) {
#pragma unroll
                    for (int b = 0; b < 8; ++b) {
                        const float w = (b & 1 ? fx : 1.0f - fx) * (b & 2 ? fy : 1.0f - fy) *
                                        (b & 4 ? fz : 1.0f - fz);
                        const uint32_t e = entry(cx + (b & 1), cy + ((b >> 1) & 1), cz + (b >> 2));
#pragma unroll
                        for (int f = 0; f < F; ++f) unsafeAtomicAdd(grad + (size_t)e * F + f, w * d[r][f]);
                    }
                    cur.have = false;
                } else {
                    float ds[F];
#pragma unroll
                    for (int f = 0; f < F; ++f) ds[f] = sum.scaled(d[r][f]);
#pragma unroll
                    for (int b = 0; b < 8; ++b) {
                        const float w = (b & 1 ? fx : 1.0f - fx) * (b & 2 ? fy : 1.0f - fy) *
                                        (b & 4 ? fz : 1.0f - fz);
#pragma unroll
                        for (int f = 0; f < F; ++f) Sum::add(a[b * F + f], w * ds[f]);
                    }
                }
            }
        }
        // neighbouring lanes whose runs ended in one cell merge their sums (8
        // lanes at most), and what is left goes to the lines
        merge_lanes<1, 8 * F, Sum>(cur, a, lane);
        merge_lanes<2, 8 * F, Sum>(cur, a, lane);
        merge_lanes<4, 8 * F, Sum>(cur, a, lane);
        flush(cur, a, cur.have);
        __syncthreads();
        // ---- every line once, and the table left empty for the next level
        for (int i = tid; i < kScSlots * kScLine; i += kScThreads) {
            const int s = i / kScLine, j = i % kScLine;
            const uint32_t k = keys[s];
            if (k == kScEmpty) continue;
            const T v = acc[i];
            if (v != T(0)) {
                const int o = j ^ ((s >> 1) & (kScLine - 1));
                const uint32_t e = (k << LOG_LE) | (o & (LE - 1));
                unsafeAtomicAdd(grad + (size_t)e * F + (o >> LOG_LE), sum.value(v));
                acc[i] = T(0);
            }
        }
        __syncthreads();
        for (int i = tid; i < kScSlots; i += kScThreads) keys[i] = kScEmpty;
        __syncthreads();
    }
}

hipError_t chunk_scatter(const Net &net, int64_t n, const float *pos, const uint32_t *perm,
                         const float *rec, int rec_stride, const float *dgt, int rows,
                         float *grad, uint32_t level_mask, hipStream_t s)
{
    const bool fixed = net.cfg.precision == NPM_PREC_BF16;
    const int nl = __builtin_popcount(level_mask);
    if (nl == 0 || n == 0) return hipSuccess;
    // A lane takes two slots where that still gives every CU two blocks: longer
    // runs merge more (8-level dense grid, 2^18 vertices: one slot 125 us, two
    // 96, four 103, eight 147; the hash grid's six levels at 2^20: 222, 170,
    // 151..181, 166), short batches need the blocks (4 levels, 16,384 vertices:
    // one 19 us, two 30).  Blocks take all levels of a chunk, or a share of
    // them where the chunks alone are fewer than two blocks a CU.
    const int R = n * nl >= 2 * kScBlocks * kScThreads ? 2 : 1;
    const int64_t chunks = (n + kScThreads * R - 1) / (kScThreads * R);
    const int gy = (int)std::min<int64_t>(nl, std::max<int64_t>(1, (kScBlocks + chunks - 1) / chunks));
    const dim3 grid((unsigned)chunks, (unsigned)gy), block(kScThreads);
#define NPM_SC_LAUNCH(FV, FX, RV)                                                                  \
    hipLaunchKernelGGL((k_scatter_chunk<FV, FX, RV>), grid, block, 0, s, net.grid, n, pos, perm,   \
                       rec, rec_stride, dgt, rows, grad, level_mask)
#define NPM_SC_RUN(FV)                                                                             \
    do {                                                                                           \
        if (fixed && R == 2) NPM_SC_LAUNCH(FV, true, 2);                                           \
        else if (fixed) NPM_SC_LAUNCH(FV, true, 1);                                                \
        else if (R == 2) NPM_SC_LAUNCH(FV, false, 2);                                              \
        else NPM_SC_LAUNCH(FV, false, 1);                                                          \
    } while (0)
    switch (net.grid.feat) {
    case 1: NPM_SC_RUN(1); break;
    case 2: NPM_SC_RUN(2); break;
    default: NPM_SC_RUN(4); break;
    }
#undef NPM_SC_RUN
#undef NPM_SC_LAUNCH
    return hipGetLastError();
}

}  // namespace npm
