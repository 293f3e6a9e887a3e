// HIP kernels for gfx950 and their C-ABI launchers: random-access sampling of
// the compressed VDB and of the dense baseline (Section 3.2.2), integer
// lookups, the compression-error statistics of Section 5.2, and Philox words.
#include "kcommon.h"

namespace vdbc {

// ---------------------------------------------------------------- sampling

template <class Acc, class View>
__global__ __launch_bounds__(kBlock) void sample_kernel(View view, const float* __restrict__ pos,
                                                        uint64_t n, int filter,
                                                        float* __restrict__ out)
{
    Acc acc{view};
    acc.reset();
    const uint64_t i = (uint64_t)wide_block() * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
    out[i] = filter ? trilinear(acc, x, y, z) : nearest(acc, x, y, z);
}

// Trilinear samples of a VDB.  A third of the footprints reach into another
// leaf region, and with a descent of each lane's own per region the wave ran
// the code of all eight corners, the last seven for an eighth of its lanes.
// Here every lane descends for its lower corner, then the wave's further
// regions (some 27 for 64 random positions) are listed in LDS and the lanes
// take one descent each, whoever's it is, from the lower node that its owner
// found.  The two corners of a row come in one 8-byte load.  16.8 million
// positions in a 512^3 tree at 1:10: 403 -> 282 us, the address units of the
// caches busy for three quarters of it, the vector units for two thirds.
// Ordered positions are bound by VALU issue, and a wave without a crossing, or
// with 64 lanes in a few leaves, must not pay for the sharing: the first reads
// its one region, the second descends once a leaf and region.  Positions past
// the volume cross nothing.  With one descent a lane and region, with the sharing
// alone, and so: a lattice of 512 x 512 x 32 102, 106 and 93 us, 4.2 million
// positions on a line 30.3, 35.6 and 31.7, nearly all outside 30.7, 39.2 and 22.
struct SampleWave {
    uint64_t region[7][64];   // by crossed axes - 1: where its values are | 1 (a stored leaf)
    uint16_t item[7 * 64];    // lane | crossed axes << 6
};

// (A pointer made from an integer would be read by flat loads.)
typedef const __attribute__((address_space(1))) float GlobalFloat;
typedef const __attribute__((address_space(1))) Word GlobalWord;
typedef float f32x2 __attribute__((ext_vector_type(2), aligned(4)));
typedef const __attribute__((address_space(1))) f32x2 GlobalPair;

__device__ __forceinline__ uint64_t region_word(const LeafH& h) { return reinterpret_cast<uint64_t>(h.p) | (h.m & 1u); }
__device__ __forceinline__ GlobalFloat* region_values(uint64_t r) { return reinterpret_cast<GlobalFloat*>(r & ~1ull); }

__global__ __launch_bounds__(kBlock) void sample_tree_kernel(VdbView view, const float* __restrict__ pos, uint64_t n,
                                                             float* __restrict__ out)
{
    __shared__ SampleWave waves[kBlock / 64];
    SampleWave& sw = waves[threadIdx.x >> 6];
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t id = (uint64_t)wide_block() * blockDim.x + threadIdx.x, at = id < n ? id : n - 1;
    const float px = __builtin_amdgcn_fmed3f(pos[3 * at], -2.0f, (float)view.nx + 1.0f);   // as trilinear()
    const float py = __builtin_amdgcn_fmed3f(pos[3 * at + 1], -2.0f, (float)view.ny + 1.0f);
    const float pz = __builtin_amdgcn_fmed3f(pos[3 * at + 2], -2.0f, (float)view.nz + 1.0f);
    const float fx0 = floorf(px), fy0 = floorf(py), fz0 = floorf(pz);
    const int i = (int)fx0, j = (int)fy0, k = (int)fz0;
    // no corner inside the volume: the background for all, without a descent
    const bool none = (unsigned)(i + 1) > (unsigned)view.nx || (unsigned)(j + 1) > (unsigned)view.ny ||
                      (unsigned)(k + 1) > (unsigned)view.nz;
    const int lx = none ? -1 : i >> 3, ly = j >> 3, lz = k >> 3;
    const bool sx = !none && (i & 7) == 7;
    const uint32_t cross = none ? 0u : (sx ? 1u : 0u) | ((j & 7) == 7 ? 2u : 0u) | ((k & 7) == 7 ? 4u : 0u);
    VdbAcc acc{view};
    acc.reset();
    const uint64_t own = region_word(acc.resolve(lx, ly, lz));
    const uint64_t crossing = __ballot(cross != 0u);
    float c[8];
    if (crossing == 0) {
        // every footprint of the wave in one region
        if (own & 1u) {
            GlobalFloat* const q = region_values(own) + ((i & 7) + 8 * (j & 7) + 64 * (k & 7));
#pragma unroll
            for (int row = 0; row < 4; ++row) {
                const f32x2 v = *(GlobalPair*)(q + 8 * (row & 1) + 64 * (row >> 1));
                c[2 * row] = v.x;
                c[2 * row + 1] = v.y;
            }
        } else {
            const float v = *region_values(own);
#pragma unroll
            for (int q = 0; q < 8; ++q) c[q] = v;
        }
    } else {
        // 1, 3 or 7 further regions: the non-empty subsets of the crossed axes
        uint32_t mine = cross;
        int head = (int)lane;
        uint64_t m1 = crossing, m2 = __ballot((mine & (mine - 1u)) != 0u), m4 = __ballot(mine == 7u);
        uint32_t total = (uint32_t)(__popcll(m1) + 2 * __popcll(m2) + 4 * __popcll(m4));
        if (total >= 64) {
            // ordered positions: lanes in a row with one leaf share its first
            // lane's descents, for the axes that any of them crosses
            const uint64_t c1 = __ballot(cross & 1u), c2 = __ballot(cross & 2u), c4 = __ballot(cross & 4u);
            const int bx = __shfl_up(lx, 1), by = __shfl_up(ly, 1), bz = __shfl_up(lz, 1);
            const uint64_t heads = __ballot(lane == 0u || bx != lx || by != ly || bz != lz);
            const uint64_t above = ~1ull << lane;   // lanes past this one
            head = 63 - __clzll((long long)(heads & ~above));
            const uint64_t later = heads & above, run = (later ? (later & (0ull - later)) - 1u : ~0ull) & (~0ull << head);
            mine = head != (int)lane ? 0u : ((c1 & run) ? 1u : 0u) | ((c2 & run) ? 2u : 0u) | ((c4 & run) ? 4u : 0u);
            m1 = __ballot(mine != 0u);
            m2 = __ballot((mine & (mine - 1u)) != 0u);
            m4 = __ballot(mine == 7u);
            total = (uint32_t)(__popcll(m1) + 2 * __popcll(m2) + 4 * __popcll(m4));
        }
        const uint64_t lower = (1ull << lane) - 1u;
        uint32_t o = (uint32_t)(__popcll(m1 & lower) + 2 * __popcll(m2 & lower) + 4 * __popcll(m4 & lower));
        for (uint32_t r = (0u - mine) & mine; r; r = (r - mine) & mine) sw.item[o++] = (uint16_t)(lane | (r << 6));
        // the lower node, or the constant in its place | 1
        const uint64_t node =
            acc.cnode ? reinterpret_cast<uint64_t>(acc.cnode) : reinterpret_cast<uint64_t>(acc.cconst) | 1u;
        wave_lds_fence();
        for (uint32_t q0 = 0; q0 < total; q0 += 64) {
            const uint32_t q = q0 + lane, e = q < total ? sw.item[q] : lane, r = e >> 6;
            const int owner = (int)(e & 63u);
            const int x = __shfl(lx, owner), y = __shfl(ly, owner), z = __shfl(lz, owner);
            const uint64_t found = __shfl((unsigned long long)node, owner);
            if (r) {
                VdbAcc from{view};
                from.reset();
                from.cLx = x >> 4;
                from.cLy = y >> 4;
                from.cLz = z >> 4;
                from.cnode = (found & 1u) ? nullptr : (const Word*)reinterpret_cast<GlobalWord*>(found);
                from.cconst = (const float*)region_values(found);
                sw.region[r - 1][owner] =
                    region_word(from.resolve(x + (int)(r & 1u), y + (int)((r >> 1) & 1u), z + (int)(r >> 2)));
            }
        }
        wave_lds_fence();
        // the rows' pairs, then what a row holds in the next region
        const int x0 = sx ? 6 : i & 7;
        uint64_t h[4];
        int a[4];
        f32x2 v[4];
        float w[4];
#pragma unroll
        for (int row = 0; row < 4; ++row) {
            const uint32_t r = cross & ((uint32_t)row << 1);
            h[row] = r ? sw.region[r - 1][head] : own;
        }
#pragma unroll
        for (int row = 0; row < 4; ++row) {
            // one value (a tile, the background) is read as the second of a pair:
            // the buffer's header is ahead of it
            a[row] = 8 * ((j + (row & 1)) & 7) + 64 * ((k + (row >> 1)) & 7);
            v[row] = *(GlobalPair*)(region_values(h[row]) + ((h[row] & 1u) ? a[row] + x0 : -1));
            w[row] = 0.0f;
        }
        if (sx) {
#pragma unroll
            for (int row = 0; row < 4; ++row) {
                const uint64_t h1 = sw.region[cross & ((uint32_t)row << 1)][head];
                w[row] = region_values(h1)[(h1 & 1u) ? a[row] : 0];
            }
        }
#pragma unroll
        for (int row = 0; row < 4; ++row) {
            c[2 * row] = (h[row] & 1u) && !sx ? v[row].x : v[row].y;
            c[2 * row + 1] = sx ? w[row] : v[row].y;
        }
    }
    const float fx = px - fx0, fy = py - fy0, fz = pz - fz0;
    const float c00 = lerp(c[0], c[1], fx), c10 = lerp(c[2], c[3], fx);
    const float c01 = lerp(c[4], c[5], fx), c11 = lerp(c[6], c[7], fx);
    if (id < n) out[id] = lerp(lerp(c00, c10, fy), lerp(c01, c11, fy), fz);
}

__global__ __launch_bounds__(kBlock) void lookup_kernel(VdbView view, const int32_t* __restrict__ ijk,
                                                        uint64_t n, float* __restrict__ out)
{
    VdbAcc acc{view};
    acc.reset();
    const uint64_t i = (uint64_t)wide_block() * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int x = ijk[3 * i], y = ijk[3 * i + 1], z = ijk[3 * i + 2];
    // voxels beyond the volume read B (edge leaves store B there, regions
    // past the last leaf or outside the root table resolve to B)
    out[i] = acc.voxel(x, y, z);
}

// ---------------------------------------------------------------- quality

// Error statistics of the compressed grid against the dense volume it was
// encoded from (the MSE / PSNR evaluation of Section 5.2).  A workgroup of
// 512 threads takes a 64 x 8 x 8 voxel region (eight leaves along x) in a
// grid-stride loop: thread (x, y) walks the region's 8 slices, so each wave
// reads 256 contiguous bytes of a dense row per slice and every thread stays
// in one leaf (one descent, then its leaf cache).  Per workgroup: {sum of
// squared differences, max |diff|, differing voxels, min dense, max dense}
// into part[5 * block]; a second kernel folds the partials in a fixed order
// (deterministic for a given size).
constexpr int kCmpThreads = 512;
constexpr int kCmpBlocks = 4096;

__global__ __launch_bounds__(kCmpThreads) void compare_kernel(VdbView view, const float* __restrict__ dense,
                                                              double* __restrict__ part)
{
    VdbAcc acc{view};
    acc.reset();
    const int t = threadIdx.x;
    const int lx = t & 63, ly = t >> 6;
    const uint64_t rx = (uint64_t)(view.nx + 63) / 64, ry = (uint64_t)(view.ny + 7) / 8,
                   rz = (uint64_t)(view.nz + 7) / 8;
    double sse = 0.0, mx = 0.0, nd = 0.0, lo = INFINITY, hi = -INFINITY;
    for (uint64_t r = blockIdx.x; r < rx * ry * rz; r += gridDim.x) {
        const int x = (int)(r % rx) * 64 + lx, y = (int)((r / rx) % ry) * 8 + ly;
        const int z0 = (int)(r / (rx * ry)) * 8;
        if (x >= view.nx || y >= view.ny) continue;
        for (int z = z0; z < z0 + 8 && z < view.nz; ++z) {
            const float dv =
                dense[(uint64_t)x + (uint64_t)view.nx * ((uint64_t)y + (uint64_t)view.ny * (uint64_t)z)];
            const float vv = acc.voxel(x, y, z);
            const double e = (double)vv - (double)dv;
            sse = fma(e, e, sse);
            mx = fmax(mx, fabs(e));
            nd += (__float_as_uint(vv) != __float_as_uint(dv)) ? 1.0 : 0.0;
            lo = fmin(lo, (double)dv);
            hi = fmax(hi, (double)dv);
        }
    }
    __shared__ double red[5][kCmpThreads];
    red[0][t] = sse;
    red[1][t] = mx;
    red[2][t] = nd;
    red[3][t] = lo;
    red[4][t] = hi;
    __syncthreads();
    for (int h = kCmpThreads / 2; h > 0; h >>= 1) {
        if (t < h) {
            red[0][t] += red[0][t + h];
            red[1][t] = fmax(red[1][t], red[1][t + h]);
            red[2][t] += red[2][t + h];
            red[3][t] = fmin(red[3][t], red[3][t + h]);
            red[4][t] = fmax(red[4][t], red[4][t + h]);
        }
        __syncthreads();
    }
    if (t < 5) part[5 * blockIdx.x + t] = red[t][0];
}

// Folds the per-workgroup partials: workgroup s reduces statistic s, each
// thread a fixed stride of partials, then a fixed-order tree in LDS.
__global__ __launch_bounds__(256) void compare_fold_kernel(const double* __restrict__ part, int blocks,
                                                           double* __restrict__ out)
{
    const int s = blockIdx.x, t = threadIdx.x;
    const bool sum = (s == 0 || s == 2), mn = (s == 3);
    double a = sum ? 0.0 : mn ? INFINITY : (s == 1 ? 0.0 : -INFINITY);
    for (int b = t; b < blocks; b += 256) {
        const double v = part[5 * b + s];
        a = sum ? a + v : mn ? fmin(a, v) : fmax(a, v);
    }
    __shared__ double red[256];
    red[t] = a;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
            const double v = red[t + h];
            red[t] = sum ? red[t] + v : mn ? fmin(red[t], v) : fmax(red[t], v);
        }
        __syncthreads();
    }
    if (t == 0) out[s] = red[0];
}

__global__ void philox_kernel(const uint32_t* __restrict__ ctr, const uint32_t* __restrict__ key,
                              uint64_t n, uint32_t* __restrict__ out)
{
    const uint64_t i = (uint64_t)wide_block() * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t c0 = ctr[4 * i], c1 = ctr[4 * i + 1], c2 = ctr[4 * i + 2], c3 = ctr[4 * i + 3];
    philox4x32_10(c0, c1, c2, c3, key[2 * i], key[2 * i + 1]);
    out[4 * i] = c0;
    out[4 * i + 1] = c1;
    out[4 * i + 2] = c2;
    out[4 * i + 3] = c3;
}

static vdbc_status check_samples(const float* pos, uint64_t n, uint32_t filter, float* out)
{
    if (filter > 1) return fail(VDBC_E_INVALID, "filter must be 0 or 1");
    if (n && (!pos || !out)) return fail(VDBC_E_INVALID, "null positions or output");
    if (n > (uint64_t)0x7FFFFFFFull * kBlock) return fail(VDBC_E_INVALID, "too many samples");
    return VDBC_OK;
}

}  // namespace vdbc

using namespace vdbc;

extern "C" vdbc_status vdbc_sample(const vdbc_grid* g, const float* pos, uint64_t n,
                                   uint32_t filter, float* out, void* stream)
{
    clear_error();
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    if ((s = check_samples(pos, n, filter, out))) return s;
    if (n == 0) return VDBC_OK;
    const dim3 grid = wide_grid((n + kBlock - 1) / kBlock);
    if (filter)
        hipLaunchKernelGGL(sample_tree_kernel, grid, dim3(kBlock), 0, static_cast<hipStream_t>(stream), v, pos, n, out);
    else
        hipLaunchKernelGGL((sample_kernel<VdbAcc, VdbView>), grid, dim3(kBlock), 0, static_cast<hipStream_t>(stream), v,
                           pos, n, (int)filter, out);
    return launch_check("vdbc_sample");
}

extern "C" vdbc_status vdbc_sample_dense(const float* dense, vdbc_dims d, float background,
                                         const float* pos, uint64_t n, uint32_t filter, float* out,
                                         void* stream)
{
    clear_error();
    DenseView v;
    vdbc_status s = make_dense(dense, d, background, &v);
    if (s) return s;
    if ((s = check_samples(pos, n, filter, out))) return s;
    if (n == 0) return VDBC_OK;
    hipLaunchKernelGGL((sample_kernel<DenseAcc, DenseView>),
                       wide_grid((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                       static_cast<hipStream_t>(stream), v, pos, n, (int)filter, out);
    return launch_check("vdbc_sample_dense");
}

extern "C" vdbc_status vdbc_lookup(const vdbc_grid* g, const int32_t* ijk, uint64_t n, float* out,
                                   void* stream)
{
    clear_error();
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    if (n && (!ijk || !out)) return fail(VDBC_E_INVALID, "null coordinates or output");
    if (n > (uint64_t)0x7FFFFFFFull * kBlock) return fail(VDBC_E_INVALID, "too many lookups");
    if (n == 0) return VDBC_OK;
    hipLaunchKernelGGL(lookup_kernel, wide_grid((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                       static_cast<hipStream_t>(stream), v, ijk, n, out);
    return launch_check("vdbc_lookup");
}

static uint64_t compare_regions(uint64_t nx, uint64_t ny, uint64_t nz)
{
    return ((nx + 63) / 64) * ((ny + 7) / 8) * ((nz + 7) / 8);
}

static uint32_t compare_blocks(const VdbView& v)
{
    const uint64_t regions = compare_regions((uint64_t)v.nx, (uint64_t)v.ny, (uint64_t)v.nz);
    return (uint32_t)std::min<uint64_t>(regions, kCmpBlocks);
}

extern "C" vdbc_status vdbc_compare_workspace(vdbc_dims d, uint64_t* bytes)
{
    clear_error();
    if (!bytes) return fail(VDBC_E_INVALID, "null argument");
    if (d.nx == 0 || d.ny == 0 || d.nz == 0) return fail(VDBC_E_INVALID, "zero dims");
    const uint64_t regions = compare_regions(d.nx, d.ny, d.nz);
    *bytes = 5ull * 8ull * std::min<uint64_t>(regions, kCmpBlocks);
    return VDBC_OK;
}

extern "C" vdbc_status vdbc_compare_dense(const vdbc_grid* g, const float* dense, double* out, void* ws,
                                          uint64_t ws_bytes, void* stream)
{
    clear_error();
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    if (!dense || !out) return fail(VDBC_E_INVALID, "null dense volume or output");
    const uint32_t blocks = compare_blocks(v);
    if (!ws || ws_bytes < 40ull * blocks)
        return fail(VDBC_E_BUFFER_TOO_SMALL, "workspace needs %llu bytes", 40ull * blocks);
    if (reinterpret_cast<uintptr_t>(ws) % 8) return fail(VDBC_E_INVALID, "workspace must be 8-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    double* part = static_cast<double*>(ws);
    hipLaunchKernelGGL(compare_kernel, dim3(blocks), dim3(kCmpThreads), 0, st, v, dense, part);
    if ((s = launch_check("compare"))) return s;
    hipLaunchKernelGGL(compare_fold_kernel, dim3(5), dim3(256), 0, st, part, (int)blocks, out);
    return launch_check("compare fold");
}

extern "C" vdbc_status vdbc_philox(const uint32_t* ctr, const uint32_t* key, uint64_t n,
                                   uint32_t* out, void* stream)
{
    clear_error();
    if (n && (!ctr || !key || !out)) return fail(VDBC_E_INVALID, "null argument");
    if (n > (uint64_t)0x7FFFFFFFull * kBlock) return fail(VDBC_E_INVALID, "too many counters");
    if (n == 0) return VDBC_OK;
    hipLaunchKernelGGL(philox_kernel, wide_grid((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                       static_cast<hipStream_t>(stream), ctr, key, n, out);
    return launch_check("vdbc_philox");
}
