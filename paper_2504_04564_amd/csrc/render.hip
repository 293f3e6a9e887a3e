// HIP kernels for gfx950 and their C-ABI launchers: majorant macrocells,
// emission-absorption and iso-surface marching, and the delta-tracking path
// tracer (Section 4), each for the compressed VDB and for the dense float32
// baseline through the same templated code, plus batched rendering.
#include <climits>
#include <mutex>
#include <type_traits>

#include "kcommon.h"
#include "pt.h"

namespace vdbc {

// Clears the workspace's counters: sample and cell counts, PT tile queue,
// path segment count.
__global__ void zero_u64(unsigned long long* p)
{
    if (threadIdx.x < 4 && blockIdx.x == 0) p[threadIdx.x] = 0ull;
}

// ---------------------------------------------------------------- majorant

// A macrocell's majorant is ds times the largest alpha over [min, max] of the
// values of its (C+2)^3 dilated footprint (the reconstruction, B outside).

// max of the piecewise-linear alpha over [vmin, vmax]: the two ends and every
// control point strictly inside.
__device__ __forceinline__ float majorant_of(const MediumK& m, float vmin, float vmax)
{
    float a = fmaxf(tf_alpha(m, vmin), tf_alpha(m, vmax));
    const float p0 = (vmin - m.tf_lo) * m.tf_inv, p1 = (vmax - m.tf_lo) * m.tf_inv;
    for (int q = 0; q < m.tf_n; ++q)
        if ((float)q > p0 && (float)q < p1) a = fmaxf(a, m.tf[q].w);
    return m.ds * a;
}

// VDB.  The 8^3 blocks of the footprint (at most 10^3: the 66 voxels of a
// macrocell of 64 from the last of a block on; 4^3 up to 16) are resolved one per thread: a tile or an empty region enters
// the min and max at once, a stored leaf is queued in LDS, whole leaves at the
// front and the slices of a border at the back.  A whole leaf is two 16-byte
// loads a lane, two leaves at a time; eight borders, 64 values or fewer each,
// are read at a time.  Up to macrocells of 16 a wave takes one each: such a
// cell is a few latencies long, and a workgroup left three waves idle while
// one resolved.  (One leaf at a time, eight masked 4-byte loads for a border
// too: 186 us at 512^3 with cells of 16, 702 us at 994x676x1225 with 64; 44 and
// 125 us so.  The leaves' bytes at the copy rate are 11 and 70 us.)
constexpr int kMajorantQueue = 10 * 10 * 10;
static_assert((7 + 64 + 2 + 7) / 8 == 10, "blocks an axis of the largest macrocell");
constexpr int kMajorantWaveCell = 16;

struct MajorantShared {
    const float* leaf[kMajorantQueue];
    uint32_t box[kMajorantQueue];   // first voxel and extent - 1 per axis, 3 bits each
    int n[kBlock / 64][2];
    float red[2][kBlock / 64];
};

// Macrocell `cell` by a wave (WAVE) or by the workgroup.
template <bool WAVE>
__device__ __forceinline__ void majorant_tree(const VdbView& view, const MediumK& m, int C, int gx, int gy,
                                              uint32_t cell, float* __restrict__ out, MajorantShared& sh)
{
    constexpr int T = WAVE ? 64 : kBlock, W = T / 64, N = WAVE ? 64 : kMajorantQueue;
    constexpr uint32_t kWhole = 0x3FE00u;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tid = WAVE ? lane : (int)threadIdx.x, w0 = WAVE ? 0 : wave;
    const float** const qleaf = sh.leaf + (WAVE ? 64 * wave : 0);
    uint32_t* const qbox = sh.box + (WAVE ? 64 * wave : 0);
    int* const qn = sh.n[WAVE ? wave : 0];
    const int cx = (int)(cell % (uint32_t)gx), cy = (int)((cell / (uint32_t)gx) % (uint32_t)gy),
              cz = (int)(cell / ((uint32_t)gx * (uint32_t)gy));
    const int E = C + 2, x0 = C * cx - 1, y0 = C * cy - 1, z0 = C * cz - 1;
    float vmin = INFINITY, vmax = -INFINITY;
    if (tid < 2) qn[tid] = 0;
    if (WAVE) wave_lds_fence();
    else __syncthreads();
    VdbAccT<kCacheNone> acc{view};
    acc.reset();
    const int bx0 = x0 >> 3, by0 = y0 >> 3, bz0 = z0 >> 3;
    const int nbx = ((x0 + E - 1) >> 3) - bx0 + 1, nby = ((y0 + E - 1) >> 3) - by0 + 1,
              nbz = ((z0 + E - 1) >> 3) - bz0 + 1;
    for (int b = tid; b < nbx * nby * nbz; b += T) {
        const int l[3] = {bx0 + b % nbx, by0 + (b / nbx) % nby, bz0 + b / (nbx * nby)};
        const LeafH h = acc.resolve(l[0], l[1], l[2]);
        if (h.m == 0u) {
            vmin = fminf(vmin, h.p[0]);
            vmax = fmaxf(vmax, h.p[0]);
            continue;
        }
        const int c0[3] = {x0, y0, z0};
        uint32_t box = 0;
        int bits = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int lo = max(0, c0[a] - 8 * l[a]), n1 = min(7, c0[a] + E - 1 - 8 * l[a]) - lo;
            box |= (uint32_t)lo << (3 * a) | (uint32_t)n1 << (9 + 3 * a);
            bits += 32 - __clz(n1);
        }
        const int q = bits > 6 ? atomicAdd(&qn[0], 1) : N - 1 - atomicAdd(&qn[1], 1);
        qleaf[q] = h.p;
        qbox[q] = box;
    }
    if (WAVE) wave_lds_fence();
    else __syncthreads();
    const int nbig = qn[0], nsmall = qn[1];
    for (int q = w0; q < nbig; q += 2 * W) {
        const int q1 = min(q + W, nbig - 1);   // the same leaf twice at the end
        const uint32_t box[2] = {qbox[q], qbox[q1]};
        const float* p[2] = {qleaf[q], qleaf[q1]};
        if (__all(box[0] == kWhole && box[1] == kWhole)) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const float4*>(p[u >> 1])[lane + 64 * (u & 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                vmin = fminf(fminf(fminf(vmin, v[u].x), fminf(v[u].y, v[u].z)), v[u].w);
                vmax = fmaxf(fmaxf(fmaxf(vmax, v[u].x), fmaxf(v[u].y, v[u].z)), v[u].w);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float v[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) v[s] = p[u][lane + 64 * s];
                const uint32_t i = (uint32_t)(lane & 7) - (box[u] & 7u), j = (uint32_t)(lane >> 3) - ((box[u] >> 3) & 7u);
                const bool in = i <= ((box[u] >> 9) & 7u) && j <= ((box[u] >> 12) & 7u);
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    if (in && (uint32_t)s - ((box[u] >> 6) & 7u) <= (box[u] >> 15)) {
                        vmin = fminf(vmin, v[s]);
                        vmax = fmaxf(vmax, v[s]);
                    }
            }
        }
    }
    for (int q = w0; q < nsmall; q += 8 * W) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int at = N - 1 - min(q + u * W, nsmall - 1);
            const uint32_t box = (uint32_t)__builtin_amdgcn_readfirstlane((int)qbox[at]);
            const uint32_t nx = (box >> 9) & 7u, ny = (box >> 12) & 7u, nz = box >> 15;
            const int sx = 32 - __clz((int)nx), sy = 32 - __clz((int)ny);
            // lanes past the extents read its last voxels again
            const uint32_t i = min((uint32_t)lane & ((1u << sx) - 1u), nx),
                           j = min(((uint32_t)lane >> sx) & ((1u << sy) - 1u), ny),
                           k = min((uint32_t)lane >> (sx + sy), nz);
            v[u] = qleaf[at][(box & 0x1FFu) + i + 8u * j + 64u * k];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            vmin = fminf(vmin, v[u]);
            vmax = fmaxf(vmax, v[u]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        vmin = fminf(vmin, __shfl_xor(vmin, o));
        vmax = fmaxf(vmax, __shfl_xor(vmax, o));
    }
    if (!WAVE) {
        if (lane == 0) {
            sh.red[0][wave] = vmin;
            sh.red[1][wave] = vmax;
        }
        __syncthreads();
        if (threadIdx.x != 0) return;
        for (int q = 1; q < W; ++q) {
            vmin = fminf(vmin, sh.red[0][q]);
            vmax = fmaxf(vmax, sh.red[1][q]);
        }
    }
    if (tid == 0) out[cell] = majorant_of(m, vmin, vmax);
}

// Workgroup `blk` of a volume's majorants (majorant_groups of them).
__device__ __forceinline__ void majorant_tree_group(const VdbView& view, const MediumK& m, int C, int gx, int gy, int gz,
                                                    uint32_t blk, float* __restrict__ out)
{
    __shared__ MajorantShared sh;
    if (C <= kMajorantWaveCell) {
        const uint32_t cell = blk * (kBlock / 64) + (threadIdx.x >> 6);
        if (cell < (uint32_t)gx * (uint32_t)gy * (uint32_t)gz) majorant_tree<true>(view, m, C, gx, gy, cell, out, sh);
    } else if (blk < (uint32_t)gx * (uint32_t)gy * (uint32_t)gz) {
        majorant_tree<false>(view, m, C, gx, gy, blk, out, sh);
    }
}

static uint64_t majorant_groups(int C, uint64_t cells)
{
    return C <= kMajorantWaveCell ? (cells + kBlock / 64 - 1) / (kBlock / 64) : cells;
}

__global__ __launch_bounds__(kBlock) void majorant_tree_kernel(VdbView view, MediumK m, int C, int gx, int gy, int gz,
                                                               float* __restrict__ out)
{
    majorant_tree_group(view, m, C, gx, gy, gz, wide_block(), out);
}

// Dense array.  A workgroup takes a run of macrocells along x, 256 voxels at
// most: 2^wl lanes read a row of the run (contiguous, a wave and row 256 bytes
// of it), the others its further rows, and a thread has six rows in flight; the
// cells fold the columns in LDS.  NARROW: less than a wave reads a row, and the
// wave folds its rows first.  Bound by the array's bytes, (C+2)^2 / C^2 times.
// (A thread per row of a cell's own footprint read 72-byte rows, column by
// column: 362 us at 512^3 with cells of 16; 122 us so, where the array at the copy
// rate takes 113.  Rows outside the volume read again and 64 lanes a row for 16
// voxels: 16 x 900 x 900 with cells of 8 62 us by the thread's rows, 78 then, 36 so;
// 900 x 900 x 16 with cells of 64 126, 214 and 50.)
template <bool NARROW>
__global__ __launch_bounds__(kBlock) void majorant_dense_kernel(DenseView view, MediumK m, int C, int gx, int gy, int gz,
                                                                int run, int runs, int wl, float* __restrict__ out)
{
    __shared__ float col[2][kBlock];   // min, max of the run's columns, by row set
    __shared__ float ends[2][2][kBlock / 64];
    const uint32_t blk = wide_block();
    const int rx = (int)(blk % (unsigned)runs), cy = (int)((blk / (unsigned)runs) % (unsigned)gy),
              cz = (int)(blk / ((unsigned)runs * (unsigned)gy));
    if (cz >= gz) return;   // the whole workgroup
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int width = run * C, lanes = 1 << wl, sets = kBlock >> wl;
    const int E = C + 2, x0 = rx * width, y0 = C * cy - 1, z0 = C * cz - 1;
    const float B = view.background;
    // the footprint's rows inside the volume; B stands for those outside
    const int ya = max(y0, 0), za = max(z0, 0), ny = min(y0 + E, view.ny) - ya,
              nz = min(z0 + E, view.nz) - za, rows = ny * nz;
    const bool rows_out = rows < E * E;
    const uint32_t inv = ((1u << 20) + (uint32_t)ny - 1u) / (uint32_t)ny;   // r / ny = r inv >> 20 for r < 66^2
    const auto row_at = [&](int r) {
        const int k = (int)(((uint32_t)r * inv) >> 20);
        return view.data + (int64_t)view.nx * ((ya + r - k * ny) + (int64_t)view.ny * (za + k));
    };
    const int c = t & (lanes - 1), x = x0 + c, set = NARROW ? t >> wl : __builtin_amdgcn_readfirstlane(t >> wl);
    float vmin = INFINITY, vmax = -INFINITY;
    if (x >= view.nx) {
        vmin = vmax = B;
    } else if (NARROW) {
        for (int r = set; r < rows; r += 6 * sets) {
            float v[6];
#pragma unroll
            for (int u = 0; u < 6; ++u) v[u] = row_at(min(r + u * sets, rows - 1))[x];
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                vmin = fminf(vmin, v[u]);
                vmax = fmaxf(vmax, v[u]);
            }
        }
    } else {
        // (a plane at a time: the rows' addresses are scalar and cost little)
        const float* plane = view.data + x + (int64_t)view.nx * (ya + (int64_t)view.ny * za);
        for (int k = 0; k < nz; ++k, plane += (int64_t)view.nx * view.ny)
            for (int j = set; j < ny; j += 6 * sets) {
                float v[6];
#pragma unroll
                for (int u = 0; u < 6; ++u) v[u] = plane[(int64_t)view.nx * min(j + u * sets, ny - 1)];
#pragma unroll
                for (int u = 0; u < 6; ++u) {
                    vmin = fminf(vmin, v[u]);
                    vmax = fmaxf(vmax, v[u]);
                }
            }
    }
    if (NARROW)
        for (int o = 32; o >= lanes; o >>= 1) {
            vmin = fminf(vmin, __shfl_xor(vmin, o));
            vmax = fmaxf(vmax, __shfl_xor(vmax, o));
        }
    const int kept = NARROW ? kBlock / 64 : sets;   // row sets in LDS
    if (!NARROW || lane < lanes) {
        col[0][(NARROW ? wave : set) * lanes + c] = vmin;
        col[1][(NARROW ? wave : set) * lanes + c] = vmax;
    }
    // the columns x0 - 1 and x0 + width
    const int xe[2] = {x0 - 1, x0 + width};
    const bool in[2] = {xe[0] >= 0, xe[1] < view.nx};
    float e[2][2] = {{in[0] ? INFINITY : B, in[0] ? -INFINITY : B}, {in[1] ? INFINITY : B, in[1] ? -INFINITY : B}};
    if (in[0] || in[1])
        for (int r = t; r < rows; r += kBlock) {
            const float* const row = row_at(r);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float v = in[s] ? row[xe[s]] : B;
                e[s][0] = fminf(e[s][0], v);
                e[s][1] = fmaxf(e[s][1], v);
            }
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            e[s][0] = fminf(e[s][0], __shfl_xor(e[s][0], o));
            e[s][1] = fmaxf(e[s][1], __shfl_xor(e[s][1], o));
        }
    if (lane == 0)
        for (int s = 0; s < 2; ++s) {
            ends[0][s][wave] = e[s][0];
            ends[1][s][wave] = e[s][1];
        }
    __syncthreads();
    const int cx = rx * run + t;
    if (t >= run || cx >= gx) return;
    float lo = rows_out ? B : INFINITY, hi = rows_out ? B : -INFINITY;
    for (int q = C * t; q < C * t + E; ++q) {
        if (q == 0 || q == width + 1) {
            for (int w = 0; w < kBlock / 64; ++w) {
                lo = fminf(lo, ends[0][q != 0][w]);
                hi = fmaxf(hi, ends[1][q != 0][w]);
            }
        } else if (q > lanes) {   // past the volume
            lo = fminf(lo, B);
            hi = fmaxf(hi, B);
        } else {
            for (int w = 0; w < kept; ++w) {
                lo = fminf(lo, col[0][w * lanes + q - 1]);
                hi = fmaxf(hi, col[1][w * lanes + q - 1]);
            }
        }
    }
    out[(uint32_t)cx + (uint32_t)gx * ((uint32_t)cy + (uint32_t)gy * (uint32_t)cz)] = majorant_of(m, lo, hi);
}

// ---------------------------------------------------------------- region index

// Entry t of the region index: the region's place in the buffer as the tree
// resolves it.
__device__ __forceinline__ void index_entry(const VdbView& view, const IndexView& iv, uint32_t t,
                                            uint32_t* __restrict__ tab, int shift)
{
    if (t >= (uint32_t)iv.tx * (uint32_t)iv.ty * (uint32_t)iv.tz) return;
    const uint32_t r = t / (uint32_t)iv.tx;
    VdbAccT<kCacheNone> acc{view};
    acc.reset();
    const LeafH h = acc.resolve((int)(t - r * (uint32_t)iv.tx) - 1, (int)(r % (uint32_t)iv.ty) - 1,
                                (int)(r / (uint32_t)iv.ty) - 1);
    tab[t] = (uint32_t)((uint64_t)(reinterpret_cast<const uint8_t*>(h.p) - iv.base) >> shift);
}

// One thread per entry (x fastest, so that the threads of a wave read the
// same node words; 287,496 entries of a 512^3 tree: 7 us, latency).
__global__ __launch_bounds__(kBlock) void index_kernel(VdbView view, IndexView iv, uint32_t* __restrict__ tab, int shift)
{
    index_entry(view, iv, blockIdx.x * kBlock + threadIdx.x, tab, shift);
}

// The same entries with their skip levels (see IndexView::level): a workgroup
// takes 8^3 entries, resolves them and their upper neighbours (9^3), and one
// wave reduces the emptiness of the footprints over 2^3, 4^3 and 8^3 blocks, a
// row of eight entries a lane.  Larger blocks would leave the chip idle (16^3:
// 125 workgroups at 512^3).
__global__ __launch_bounds__(kBlock) void index_level_kernel(VdbView view, IndexView iv, uint32_t* __restrict__ tab,
                                                             uint8_t* __restrict__ level, int shift)
{
    __shared__ uint32_t row[9][9];   // [z][y]: bit x set where a stored leaf or a tile is
    const uint32_t nbx = (uint32_t)(iv.tx + 7) / 8u, nby = (uint32_t)(iv.ty + 7) / 8u, bq = blockIdx.x / nbx;
    const int x0 = (int)(blockIdx.x - bq * nbx) * 8, y0 = (int)(bq % nby) * 8, z0 = (int)(bq / nby) * 8, t = threadIdx.x;
    if (t < 81) (&row[0][0])[t] = 0u;
    __syncthreads();
    VdbAccT<kCacheNone> acc{view};
    acc.reset();
    auto resolve = [&](int i, int j, int k, bool own) {
        const int x = x0 + i, y = y0 + j, z = z0 + k;
        const LeafH h = acc.resolve(x - 1, y - 1, z - 1);
        if (h.p != view.bg) atomicOr(&row[k][j], 1u << i);
        if (own && x < iv.tx && y < iv.ty && z < iv.tz)
            tab[(uint32_t)x + (uint32_t)iv.tx * ((uint32_t)y + (uint32_t)iv.ty * (uint32_t)z)] =
                (uint32_t)((uint64_t)(reinterpret_cast<const uint8_t*>(h.p) - iv.base) >> shift);
    };
    const int u = t & 7, v = (t >> 3) & 7, w = t >> 6;
    resolve(u, v, w, true);
    resolve(u, v, w + 4, true);
    // the faces x = 8, y = 8 and z = 8 (64 each), their edges (8 each), the corner
    if (w < 3) resolve(w == 0 ? 8 : u, w == 1 ? 8 : w == 0 ? u : v, w == 2 ? 8 : v, false);
    else if (v < 3) resolve(v == 0 ? u : 8, v == 1 ? u : 8, v == 2 ? u : 8, false);
    else if (t == 192 + 24) resolve(8, 8, 8, false);
    __syncthreads();
    if (t >= 64) return;
    // lane t: the row of entries y0 + v, z0 + t / 8, bit x
    const int j = u, k = t >> 3;
    const uint32_t m = row[k][j] | row[k][j + 1] | row[k + 1][j] | row[k + 1][j + 1];
    auto block = [&](uint32_t e, int s, uint32_t keep) {   // e over blocks of 2 s entries a side
        e &= __shfl_xor(e, s);
        e &= __shfl_xor(e, 8 * s);
        e &= (e >> s) & keep;
        return e;
    };
    const uint32_t e1 = ~(m | (m >> 1)) & 0xFFu;
    const uint32_t e2 = block(e1, 1, 0x55u) * 0x3u, e3 = block(e2, 2, 0x11u) * 0xFu, e4 = block(e3, 4, 0x01u) * 0xFFu;
    const int y = y0 + j, z = z0 + k;
    if (y >= iv.ty || z >= iv.tz) return;
    uint8_t* out = level + x0 + (size_t)iv.tx * ((size_t)y + (size_t)iv.ty * (size_t)z);
    for (int i = 0; i < 8 && x0 + i < iv.tx; ++i)
        out[i] = (uint8_t)(((e1 >> i) & 1u) + ((e2 >> i) & 1u) + ((e3 >> i) & 1u) + ((e4 >> i) & 1u));
}

// ---------------------------------------------------------------- marching in quads
// The EA and ISO marchers of a dense array, and of a VDB read through the
// region index: four lanes (a quad) share a ray and take four consecutive
// lattice samples at a time, sixteen rays (4 x 4 pixels) a wave.  One thread
// per ray left the chip waiting (a sample's loads, then the next one's) and
// its waves half empty, since 64 rays end at 64 different places.  Per sample
// the arithmetic, and the order of the sums, are those of the kernels below
// with one thread per ray; the images are the same bit for bit.  EA frame of a
// 512^3 cloud, 1024^2 pixels: 6.3 -> 0.92 ms; ISO of 421x500x333, 1277 x 719:
// 3.1 -> 0.32 ms; EA of 64^3, 128^2 pixels: 271 -> 27 us.  Bound by VALU issue on
// the large frames, by one ray's chain of samples on the smallest.

// Lane S of the quad's value of v, in every lane of the quad.
template <int S>
__device__ __forceinline__ float quad_get(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), S * 0x55, 0xF, 0xF, true));
}
template <int S>
__device__ __forceinline__ int quad_get(int v)
{
    return __builtin_amdgcn_mov_dpp(v, S * 0x55, 0xF, 0xF, true);
}

// A quad's ray: the lattice t0 + (k + 1/2) step inside the volume's box.
struct MarchRay {
    float o[3], d[3], id[3], t0, t1;
    int px, py;
    bool live;
};

template <class View>
__device__ __forceinline__ MarchRay march_ray(const View& v, const CameraK& cam)
{
    MarchRay r;
    const int q = (threadIdx.x & 63) >> 2, w = threadIdx.x >> 6;
    const uint32_t blk = wide_block();   // past the image: no ray is live
    const uint32_t across = (uint32_t)(cam.width + 7) / 8u, by = blk / across, bx = blk - by * across;
    r.px = (int)bx * 8 + (w & 1) * 4 + (q & 3);
    r.py = (int)by * 8 + (w >> 1) * 4 + (q >> 2);
    r.live = r.px < cam.width && r.py < cam.height;
    camera_ray(cam, (float)r.px + 0.5f, (float)r.py + 0.5f, r.o, r.d);
    for (int a = 0; a < 3; ++a) r.id[a] = 1.0f / r.d[a];
    if (!box_clip(v.nx, v.ny, v.nz, r.o, r.d, r.id, r.t0, r.t1)) r.live = false;
    return r;
}

// The first lattice index past the empty block of level L (2^(L - 1) entries
// a side) that holds sample k in entry e; at least k + 1.  Every sample
// before it reads the background (kHddaEps: far beyond the rounding of the
// exit and of a sample's position, from as near as skip_is_exact() asks for).
__device__ __forceinline__ int march_skip(const MarchRay& r, int L, const int e[3], int k, float inv_step)
{
    const int keep = -(1 << (L - 1)), size = 8 << (L - 1);
    float te = INFINITY;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = (float)(8 * ((e[a] & keep) - 1));
        const float plane = r.d[a] > 0.0f ? lo + ((float)size - kHddaEps) : lo + kHddaEps;
        te = r.d[a] == 0.0f ? te : fminf(te, (plane - r.o[a]) * r.id[a]);
    }
    const int kn = (int)floorf(fminf(fmaf(te - r.t0, inv_step, -0.5f), 2.0e9f));
    return max(kn, k) + 1;
}

// Ray parameter and position of lattice sample k, with SKIP its index entry
// and that entry's skip level (0 without); false past the end of the ray.
template <bool SKIP, class View>
__device__ __forceinline__ bool march_at(const View& v, const MarchRay& r, int k, float step, float& t, float p[3],
                                         int e[3], int& L)
{
    t = fmaf((float)k + 0.5f, step, r.t0);
    const int n[3] = {v.nx, v.ny, v.nz};
    const bool in = t < r.t1;
    L = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) p[a] = fmaf(t, r.d[a], r.o[a]);
    if constexpr (SKIP) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            e[a] = ((int)floorf(__builtin_amdgcn_fmed3f(p[a], -2.0f, (float)n[a] + 1.0f)) + 8) >> 3;
        if (in) L = v.level[(uint32_t)e[0] + (uint32_t)v.tx * ((uint32_t)e[1] + (uint32_t)v.ty * (uint32_t)e[2])];
    }
    return in;
}

// Emission-absorption.  SKIP: the transfer function is clear at the
// background, so that samples in empty blocks add nothing.
template <class Acc, class View, bool SKIP>
__global__ __launch_bounds__(kBlock) void ea_quad_kernel(View view, CameraK cam, MediumK m, float step,
                                                         float inv_step, float t_term, float* __restrict__ image)
{
    __shared__ float4 tf[64];
    for (int i = threadIdx.x; i < m.tf_n; i += kBlock) tf[i] = m.tf[i];
    __syncthreads();
    Acc acc{view};
    acc.reset();
    const MarchRay r = march_ray(view, cam);
    float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, T = 1.0f;
    const int lane = threadIdx.x & 3;
    bool run = r.live;
    int k = 0;
    while (run) {
        // the next four samples that are not all empty
        float t, p[3];
        int e[3], L;
        bool in;
        for (;;) {
            in = march_at<SKIP>(view, r, k + lane, step, t, p, e, L);
            const int sample = in && L == 0;
            if (quad_get<0>(sample) | quad_get<1>(sample) | quad_get<2>(sample) | quad_get<3>(sample)) break;
            // the quad's samples are all empty or past the end
            const int next = SKIP && in ? march_skip(r, L, e, k + lane, inv_step) : INT_MAX;
            k = quad_get<3>(next);
            if (k == INT_MAX) break;
        }
        if (k == INT_MAX) break;
        float4 c = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float alpha = 0.0f;
        if (in && L == 0) {
            const float s = trilinear(acc, p[0], p[1], p[2]);
            c = tf_eval_at(tf, m, s);
            alpha = 1.0f - expf(-(m.ds * c.w) * step);
        }
#define VDBC_EA_ADD(S)                                                  \
    {                                                                   \
        const float a = run ? quad_get<S>(alpha) : 0.0f, ta = T * a;    \
        c0 = fmaf(ta, quad_get<S>(c.x), c0);                            \
        c1 = fmaf(ta, quad_get<S>(c.y), c1);                            \
        c2 = fmaf(ta, quad_get<S>(c.z), c2);                            \
        T *= 1.0f - a;                                                  \
        run = run && !(T < t_term);                                     \
    }
        VDBC_EA_ADD(0)
        VDBC_EA_ADD(1)
        VDBC_EA_ADD(2)
        VDBC_EA_ADD(3)
#undef VDBC_EA_ADD
        k += 4;
    }
    if (lane == 0 && r.px < cam.width && r.py < cam.height)
        reinterpret_cast<float4*>(image)[(uint64_t)r.py * cam.width + r.px] = make_float4(c0, c1, c2, 1.0f - T);
}

// Iso-surface (see iso_kernel).  With SKIP the samples of empty blocks take
// the background's side without a field read.
template <class Acc, class View, bool SKIP>
__global__ __launch_bounds__(kBlock) void iso_quad_kernel(View view, CameraK cam, float iso, float step, float inv_step,
                                                          int refine, float* __restrict__ image,
                                                          float* __restrict__ aov)
{
    Acc acc{view};
    acc.reset();
    const MarchRay r = march_ray(view, cam);
    const int lane = threadIdx.x & 3;
    const bool bg_side = acc.background() >= iso;
    bool run = r.live, have = false, prev = false, cross = false;
    float lo = 0.0f, hi = 0.0f;
    int k = 0;
    while (run) {
        float t, p[3];
        int e[3], L;
        bool in;
        for (;;) {
            in = march_at<SKIP>(view, r, k + lane, step, t, p, e, L);
            const int sample = in && L == 0;
            if (quad_get<0>(sample) | quad_get<1>(sample) | quad_get<2>(sample) | quad_get<3>(sample)) break;
            // all empty or past the end; an empty sample after one on the
            // other side is a crossing
            const bool first = quad_get<0>((int)in);
            if (!first) k = INT_MAX;
            if (!first || (have && prev != bg_side)) break;
            have = true;
            prev = bg_side;
            const int next = SKIP && in ? march_skip(r, L, e, k + lane, inv_step) : INT_MAX;
            k = quad_get<3>(next);
            if (k == INT_MAX) break;
        }
        if (k == INT_MAX) break;
        bool side = bg_side;
        if (in && L == 0) side = trilinear(acc, p[0], p[1], p[2]) >= iso;
        const int mine = (in ? 1 : 0) | (side ? 2 : 0);
        // the first sample on another side than the one before it
#define VDBC_ISO_STEP(S)                                                                  \
    {                                                                                     \
        const int b = quad_get<S>(mine);                                                  \
        const bool at = run && (b & 1) && have && ((b & 2) != 0) != prev;                 \
        if (at) {                                                                         \
            lo = fmaf((float)(k + S - 1) + 0.5f, step, r.t0);                             \
            hi = fmaf((float)(k + S) + 0.5f, step, r.t0);                                 \
            cross = true;                                                                 \
            run = false;                                                                  \
        }                                                                                 \
        if (run && (b & 1)) {                                                             \
            have = true;                                                                  \
            prev = (b & 2) != 0;                                                          \
        }                                                                                 \
    }
        VDBC_ISO_STEP(0)
        VDBC_ISO_STEP(1)
        VDBC_ISO_STEP(2)
        VDBC_ISO_STEP(3)
#undef VDBC_ISO_STEP
        k += 4;
    }
    float4 out = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float thit = -1.0f;
    if (cross) {
        // two bisection steps a turn: lane 0 takes the midpoint, lanes 1 and 2
        // the midpoints of the halves it can leave
        for (int it = 0; it < refine; it += 2) {
            const float mid = 0.5f * (lo + hi), below = 0.5f * (lo + mid), above = 0.5f * (mid + hi);
            const float q = lane == 1 ? below : lane == 2 ? above : mid;
            const int same =
                (trilinear(acc, fmaf(q, r.d[0], r.o[0]), fmaf(q, r.d[1], r.o[1]), fmaf(q, r.d[2], r.o[2])) >= iso) ==
                prev;
            const bool up = quad_get<0>(same);
            if (up) lo = mid;
            else hi = mid;
            if (it + 1 == refine) break;
            const bool up2 = up ? quad_get<2>(same) : quad_get<1>(same);
            const float mid2 = up ? above : below;
            if (up2) lo = mid2;
            else hi = mid2;
        }
        // the six central-difference samples of the normal in two turns
        thit = 0.5f * (lo + hi);
        const float sh = (lane & 1) ? -0.5f : 0.5f;
        const float p0 = fmaf(thit, r.d[0], r.o[0]), p1 = fmaf(thit, r.d[1], r.o[1]), p2 = fmaf(thit, r.d[2], r.o[2]);
        const float wxy = trilinear(acc, p0 + (lane < 2 ? sh : 0.0f), p1 + (lane < 2 ? 0.0f : sh), p2);
        const float wz = trilinear(acc, p0, p1, p2 + sh);
        const float gx = quad_get<0>(wxy) - quad_get<1>(wxy), gy = quad_get<2>(wxy) - quad_get<3>(wxy),
                    gz = quad_get<0>(wz) - quad_get<1>(wz);
        const float len = sqrtf(gx * gx + gy * gy + gz * gz);
        out = len > 0.0f ? make_float4(0.5f * (1.0f - gx / len), 0.5f * (1.0f - gy / len), 0.5f * (1.0f - gz / len), 1.0f)
                         : make_float4(0.5f, 0.5f, 0.5f, 1.0f);
    }
    if (lane == 0 && r.px < cam.width && r.py < cam.height) {
        const uint64_t pix = (uint64_t)r.py * cam.width + r.px;
        reinterpret_cast<float4*>(image)[pix] = out;
        if (aov) reinterpret_cast<float2*>(aov)[pix] = make_float2(thit, 0.0f);
    }
}

// ---------------------------------------------------------------- EA

template <class Acc, class View, bool HDDA, bool COUNT>
__global__ __launch_bounds__(kBlock) void ea_kernel(View view, CameraK cam, MediumK m, float step,
                                                    float t_term, float* __restrict__ image,
                                                    unsigned long long* counter)
{
    Acc acc{view};
    acc.reset();
    int px, py;
    const bool live = tile_pixel(cam.width, cam.height, 8, blockIdx.x, blockIdx.y, px, py);
    uint32_t nsamp = 0;
    if (live) {
        float o[3], d[3], t0, t1;
        camera_ray(cam, (float)px + 0.5f, (float)py + 0.5f, o, d);
        float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, T = 1.0f;
        const float id[3] = {1.0f / d[0], 1.0f / d[1], 1.0f / d[2]};
        if (box_clip(view.nx, view.ny, view.nz, o, d, id, t0, t1)) {
            for (int k = 0;; ++k) {
                const float t = fmaf((float)k + 0.5f, step, t0);
                if (t >= t1) break;
                const float x = fmaf(t, d[0], o[0]), y = fmaf(t, d[1], o[1]),
                            z = fmaf(t, d[2], o[2]);
                if (HDDA) {
                    const int i = (int)floorf(fmaxf(x, -2.0f)), j = (int)floorf(fmaxf(y, -2.0f)),
                              kk = (int)floorf(fmaxf(z, -2.0f));
                    const int L = acc.in_stored_leaf(i, j, kk) ? 0 : acc.empty_level(i, j, kk);
                    if (L) {
                        const int mask = (1 << L) - 1;
                        if ((i & mask) != mask && (j & mask) != mask && (kk & mask) != mask) {
                            // every sample whose footprint stays inside this
                            // empty node reads B with alpha 0: jump past it
                            const int lo[3] = {i & ~mask, j & ~mask, kk & ~mask};
                            float te = INFINITY;
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                if (d[a] > 0.0f)
                                    te = fminf(te, ((float)(lo[a] + mask) - kHddaEps - o[a]) / d[a]);
                                else if (d[a] < 0.0f)
                                    te = fminf(te, ((float)lo[a] + kHddaEps - o[a]) / d[a]);
                            }
                            const int kn = (int)floorf(fminf((te - t0) / step - 0.5f, 2.0e9f));
                            k = (kn > k + 1 ? kn : k + 1) - 1;
                            continue;
                        }
                    }
                }
                const float s = trilinear(acc, x, y, z);
                if (COUNT) ++nsamp;
                const float4 c = tf_eval(m, s);
                const float a = 1.0f - expf(-(m.ds * c.w) * step);
                const float ta = T * a;
                c0 = fmaf(ta, c.x, c0);
                c1 = fmaf(ta, c.y, c1);
                c2 = fmaf(ta, c.z, c2);
                T *= 1.0f - a;
                if (T < t_term) break;
            }
        }
        float4* img = reinterpret_cast<float4*>(image);
        img[(uint64_t)py * cam.width + px] = make_float4(c0, c1, c2, 1.0f - T);
    }
    if (COUNT) block_count(nsamp, counter);
}

// ---------------------------------------------------------------- ISO

// Implicit iso-surface marcher (the interval-based marcher of Section 5.4):
// the EA lattice t0 + (k + 1/2) step, the first pair of consecutive samples
// on opposite sides of the iso value (side: f >= iso), `refine` bisection
// steps on that interval, normal -grad f / |grad f| by central differences
// of half a voxel.  With HDDA, lattice samples whose trilinear footprint lies
// inside an empty node read B at every corner, so they take B's side without
// a field read; the crossing, the bisection and the image are unchanged.
template <class Acc, class View, bool HDDA, bool COUNT>
__global__ __launch_bounds__(kBlock) void iso_kernel(View view, CameraK cam, float iso, float step,
                                                     int refine, float* __restrict__ image,
                                                     float* __restrict__ aov,
                                                     unsigned long long* counter)
{
    Acc acc{view};
    acc.reset();
    int px, py;
    const bool live = tile_pixel(cam.width, cam.height, 8, blockIdx.x, blockIdx.y, px, py);
    uint32_t nsamp = 0;
    if (live) {
        float o[3], d[3], t0, t1;
        camera_ray(cam, (float)px + 0.5f, (float)py + 0.5f, o, d);
        float4 out = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float thit = -1.0f;
        const float id[3] = {1.0f / d[0], 1.0f / d[1], 1.0f / d[2]};
        if (box_clip(view.nx, view.ny, view.nz, o, d, id, t0, t1)) {
            const bool bg_side = acc.background() >= iso;
            bool have = false, prev = false;
            float tprev = 0.0f;
            for (int k = 0;; ++k) {
                const float t = fmaf((float)k + 0.5f, step, t0);
                if (t >= t1) break;
                const float x = fmaf(t, d[0], o[0]), y = fmaf(t, d[1], o[1]), z = fmaf(t, d[2], o[2]);
                bool side;
                int last = k;   // last lattice sample of this step
                bool skip = false;
                if (HDDA) {
                    const int i = (int)floorf(fmaxf(x, -2.0f)), j = (int)floorf(fmaxf(y, -2.0f)),
                              kk = (int)floorf(fmaxf(z, -2.0f));
                    const int L = acc.in_stored_leaf(i, j, kk) ? 0 : acc.empty_level(i, j, kk);
                    if (L) {
                        const int mask = (1 << L) - 1;
                        if ((i & mask) != mask && (j & mask) != mask && (kk & mask) != mask) {
                            const int lo[3] = {i & ~mask, j & ~mask, kk & ~mask};
                            float te = INFINITY;
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                if (d[a] > 0.0f)
                                    te = fminf(te, ((float)(lo[a] + mask) - kHddaEps - o[a]) / d[a]);
                                else if (d[a] < 0.0f)
                                    te = fminf(te, ((float)lo[a] + kHddaEps - o[a]) / d[a]);
                            }
                            const int kn = (int)floorf(fminf((te - t0) / step - 0.5f, 2.0e9f));
                            last = (kn > k + 1 ? kn : k + 1) - 1;
                            skip = true;
                        }
                    }
                }
                if (skip) {
                    side = bg_side;
                } else {
                    side = trilinear(acc, x, y, z) >= iso;
                    if (COUNT) ++nsamp;
                }
                if (have && side != prev) {
                    // `refine` bisection steps, then the six central-difference
                    // samples of the normal, through one field evaluation
                    float lo = tprev, hi = t, mid = 0.0f;
                    float p0 = 0.0f, p1 = 0.0f, p2 = 0.0f, gx = 0.0f, gy = 0.0f, gz = 0.0f;
                    for (int it = 0; it < refine + 6; ++it) {
                        float q0, q1, q2;
                        const int e = it - refine;   // >= 0: gradient sample e
                        if (e < 0) {
                            mid = 0.5f * (lo + hi);
                            q0 = fmaf(mid, d[0], o[0]);
                            q1 = fmaf(mid, d[1], o[1]);
                            q2 = fmaf(mid, d[2], o[2]);
                        } else {
                            if (e == 0) {
                                thit = 0.5f * (lo + hi);
                                p0 = fmaf(thit, d[0], o[0]);
                                p1 = fmaf(thit, d[1], o[1]);
                                p2 = fmaf(thit, d[2], o[2]);
                            }
                            const float sh = (e & 1) ? -0.5f : 0.5f;
                            q0 = p0 + ((e >> 1) == 0 ? sh : 0.0f);
                            q1 = p1 + ((e >> 1) == 1 ? sh : 0.0f);
                            q2 = p2 + ((e >> 1) == 2 ? sh : 0.0f);
                        }
                        const float w = trilinear(acc, q0, q1, q2);
                        if (COUNT) ++nsamp;
                        if (e < 0) {
                            if ((w >= iso) == prev) lo = mid;
                            else hi = mid;
                        } else {
                            const float sw = (e & 1) ? -w : w;
                            if ((e >> 1) == 0) gx += sw;
                            else if ((e >> 1) == 1) gy += sw;
                            else gz += sw;
                        }
                    }
                    const float len = sqrtf(gx * gx + gy * gy + gz * gz);
                    out = len > 0.0f ? make_float4(0.5f * (1.0f - gx / len), 0.5f * (1.0f - gy / len),
                                                   0.5f * (1.0f - gz / len), 1.0f)
                                     : make_float4(0.5f, 0.5f, 0.5f, 1.0f);
                    break;
                }
                have = true;
                prev = side;
                tprev = last == k ? t : fmaf((float)last + 0.5f, step, t0);
                k = last;
            }
        }
        const uint64_t pix = (uint64_t)py * cam.width + px;
        reinterpret_cast<float4*>(image)[pix] = out;
        if (aov) reinterpret_cast<float2*>(aov)[pix] = make_float2(thit, 0.0f);
    }
    if (COUNT) block_count(nsamp, counter);
}

// ---------------------------------------------------------------- host side

static vdbc_status make_medium(const vdbc_medium* m, int nx, int ny, int nz, MediumK* k)
{
    if (!m) return fail(VDBC_E_INVALID, "null medium");
    if (m->tf_n < 2 || m->tf_n > 64) return fail(VDBC_E_INVALID, "tf_n must be in [2, 64]");
    if (!(m->tf_hi > m->tf_lo) || !std::isfinite(m->tf_lo) || !std::isfinite(m->tf_hi))
        return fail(VDBC_E_INVALID, "need finite tf_lo < tf_hi");
    if (!std::isfinite(m->sigma_scale) || m->sigma_scale < 0.0f)
        return fail(VDBC_E_INVALID, "sigma_scale must be finite and >= 0");
    std::memset(k, 0, sizeof *k);
    const int nmax = nx > ny ? (nx > nz ? nx : nz) : (ny > nz ? ny : nz);
    k->ds = m->sigma_scale / (float)nmax;
    k->albedo = m->albedo;
    k->tf_n = (int)m->tf_n;
    k->tf_lo = m->tf_lo;
    k->tf_inv = (float)(m->tf_n - 1) / (m->tf_hi - m->tf_lo);
    for (uint32_t i = 0; i < m->tf_n; ++i) {
        for (int c = 0; c < 4; ++c)
            if (!std::isfinite(m->tf[i][c])) return fail(VDBC_E_INVALID, "non-finite TF entry");
        if (m->tf[i][3] < 0.0f) return fail(VDBC_E_INVALID, "TF alpha must be >= 0");
        k->tf[i] = make_float4(m->tf[i][0], m->tf[i][1], m->tf[i][2], m->tf[i][3]);
    }
    for (int a = 0; a < 3; ++a) {
        k->light[a] = m->light_dir[a];
        k->light_E[a] = m->light_E[a];
        k->ambient[a] = m->ambient[a];
    }
    if (m->env) {
        if (m->env_w == 0 || m->env_h == 0 || (uint64_t)m->env_w * m->env_h > (1ull << 28))
            return fail(VDBC_E_INVALID, "env map needs 1 <= env_w * env_h <= 2^28 texels");
        k->env = m->env;
        k->env_w = (int)m->env_w;
        k->env_h = (int)m->env_h;
    }
    return VDBC_OK;
}

// Host mirror of the device TF alpha (for the HDDA precondition alpha(B)=0).
static float host_alpha(const MediumK& m, float s)
{
    float pos = (s - m.tf_lo) * m.tf_inv;
    pos = std::fmin(std::fmax(pos, 0.0f), (float)(m.tf_n - 1));
    int i = (int)pos;
    i = i > m.tf_n - 2 ? m.tf_n - 2 : i;
    const float fr = pos - (float)i;
    return std::fma(fr, m.tf[i + 1].w - m.tf[i].w, m.tf[i].w);
}

static vdbc_status make_camera(const vdbc_camera* c, CameraK* k)
{
    if (!c) return fail(VDBC_E_INVALID, "null camera");
    if (c->kind > 1) return fail(VDBC_E_INVALID, "camera kind must be 0 or 1");
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(c->origin[a]) || !std::isfinite(c->lower_left[a]) ||
            !std::isfinite(c->du[a]) || !std::isfinite(c->dv[a]) || !std::isfinite(c->dir[a]))
            return fail(VDBC_E_INVALID, "non-finite camera vector");
    if (c->kind == 0 && c->dir[0] == 0.0f && c->dir[1] == 0.0f && c->dir[2] == 0.0f)
        return fail(VDBC_E_INVALID, "orthographic camera needs a non-zero direction");
    if (c->width == 0 || c->height == 0 || c->width > 65536 * kTile || c->height > 65535u * kTile ||
        (uint64_t)c->width * c->height > (1ull << 31))
        return fail(VDBC_E_INVALID, "bad image size (1..2^31 pixels)");
    k->kind = (int)c->kind;
    k->width = (int)c->width;
    k->height = (int)c->height;
    for (int a = 0; a < 3; ++a) {
        k->o[a] = c->origin[a];
        k->ll[a] = c->lower_left[a];
        k->du[a] = c->du[a];
        k->dv[a] = c->dv[a];
        k->dir[a] = c->dir[a];
    }
    return VDBC_OK;
}

static uint64_t majorant_bytes(uint32_t C, int nx, int ny, int nz)
{
    const uint64_t gx = (nx + C - 1) / C, gy = (ny + C - 1) / C, gz = (nz + C - 1) / C;
    return gx * gy * gz * 4u;
}

// Majorant grid and coarse occupancy geometry.  Coarse blocks are 2^lf
// macrocells per axis, the largest power of two spanning at most 64 voxels
// (2^3 bricks), doubled until the bit mask fits in 32 KB of LDS.
static void pt_geometry(uint32_t C, int nx, int ny, int nz, PtArgs* g)
{
    g->C = (int)C;
    g->invC = 1.0f / (float)C;
    g->gx = (nx + g->C - 1) / g->C;
    g->gy = (ny + g->C - 1) / g->C;
    g->gz = (nz + g->C - 1) / g->C;
    int lf = 0;
    // coarse blocks of at least 4 macrocells and at least 64 voxels per axis
    // (64 voxels up to C = 16, 4 cells from there on)
    const uint32_t edge = std::max<uint32_t>(64u, 4u * C);
    while ((C << (lf + 1)) <= edge) ++lf;
    for (;;) {
        const int F = 1 << lf;
        g->lf = lf;
        g->cgx = (g->gx + F - 1) / F;
        g->cgy = (g->gy + F - 1) / F;
        g->cgz = (g->gz + F - 1) / F;
        const uint64_t cells = (uint64_t)g->cgx * g->cgy * g->cgz;
        g->cwords = (int)((cells + 31) / 32);
        if (g->cwords <= 8192) break;
        ++lf;
    }
}

static uint64_t pt_workspace(uint32_t C, int nx, int ny, int nz)
{
    PtArgs g;
    pt_geometry(C, nx, ny, nz, &g);
    return 256 + align256(majorant_bytes(C, nx, ny, nz)) + align256(4ull * g.cwords);
}

static uint64_t pt_tiles(uint64_t width, uint64_t height, uint64_t tw);

// Samples per work item of a path-traced launch (= spp: its tiles are not
// split): the caller's, or with VDBC_RENDER_SPLIT and none given the most that
// leaves about kSplitItems items.  The card holds 1280 workgroups at once, and
// with a few items each the last ones to end leave most of it idle, while an
// item of few samples drains its own lanes more often: at 4 samples 512^2
// pixels (1024 tiles) take 1.47 ms whole, 0.85 ms by one sample, 1.15 ms by
// two; 1024^2 pixels (4096 tiles) 2.79 ms whole, 2.61 ms by two samples.  More
// than kSplitItems tiles are never split.
constexpr uint64_t kSplitItems = 6144;

static uint32_t pt_chunk(const vdbc_render_params* r, const vdbc_camera* c)
{
    if (r->chunk_spp != 0) return std::min(r->chunk_spp, r->spp);
    if (!(r->flags & VDBC_RENDER_SPLIT) || !c || r->spp < 2) return r->spp;
    const uint64_t n = (uint64_t)r->spp * pt_tiles(c->width, c->height, r->tile_w == 0 ? 8 : r->tile_w) / kSplitItems;
    return (uint32_t)std::min<uint64_t>(std::max<uint64_t>(n, 1), r->spp);
}

// Whether the tiles are split into several work items (which needs the
// per-pixel sums after the occupancy bits).
static bool pt_split(const vdbc_render_params* r, const vdbc_camera* c) { return pt_chunk(r, c) < r->spp; }

// Whether the tiles are queued in cost order: where asked for, and where the
// library chooses the work items and there are more of them than workgroups at
// once (below that all start together and the two launches, some 10 us, gain
// nothing): 512^2 pixels of 4 samples 0.80 -> 0.73 ms, 800x600 of 2 samples 0.76
// -> 0.64, 1024^2 of 4 samples 2.01 -> 1.96, the dense array's 2.30 either way.
constexpr uint64_t kOrderItems = 1280;

static bool pt_ordered(const vdbc_render_params* r, const vdbc_camera* c)
{
    if (r->flags & VDBC_RENDER_COST_ORDER) return true;
    if (r->chunk_spp != 0 || !(r->flags & VDBC_RENDER_SPLIT) || !c || r->spp == 0) return false;
    const uint32_t chunk = pt_chunk(r, c);
    return pt_tiles(c->width, c->height, r->tile_w == 0 ? 8 : r->tile_w) * ((r->spp + chunk - 1) / chunk) > kOrderItems;
}

// Bytes of the per-pixel sums of a split launch: 32 (red, green, blue,
// hits | escapes) + 8 (AOV depth) per pixel.
static uint64_t pt_sums_bytes(uint64_t npix) { return align256(40ull * npix); }

// 256-pixel tiles of a path-traced image: 4 tw x 64 / tw pixels each.
static uint64_t pt_tiles_x(uint64_t width, uint64_t tw) { return (width + 4 * tw - 1) / (4 * tw); }
static uint64_t pt_tiles(uint64_t width, uint64_t height, uint64_t tw)
{
    return pt_tiles_x(width, tw) * ((height + 64 / tw - 1) / (64 / tw));
}

// Bytes of the cost order (VDBC_RENDER_COST_ORDER): 2 kCostBins u32 unused,
// then per tile its bin and the tile at its place in the order (u32 each).
static uint64_t pt_order_bytes(uint64_t tiles) { return align256(8ull * kCostBins + 8ull * tiles); }

// Region index of a VDB render (VDBC_RENDER_INDEX): its table follows the
// rest of the workspace.
struct IndexPlan {
    IndexView v{};
    bool on = false, wide = false;
};

static vdbc_status launch_index(const VdbView& v, const IndexPlan& ix, hipStream_t st)
{
    if (ix.v.level) {
        const unsigned blocks = (unsigned)((ix.v.tx + 7) / 8) * (unsigned)((ix.v.ty + 7) / 8) * (unsigned)((ix.v.tz + 7) / 8);
        hipLaunchKernelGGL(index_level_kernel, dim3(blocks), dim3(kBlock), 0, st, v, ix.v, const_cast<uint32_t*>(ix.v.tab),
                           const_cast<uint8_t*>(ix.v.level), ix.wide ? 2 : 0);
        return launch_check("region index");
    }
    const uint32_t n = (uint32_t)ix.v.tx * (uint32_t)ix.v.ty * (uint32_t)ix.v.tz;
    hipLaunchKernelGGL(index_kernel, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, v, ix.v,
                       const_cast<uint32_t*>(ix.v.tab), ix.wide ? 2 : 0);
    return launch_check("region index");
}

static vdbc_status majorant_cells(int nx, int ny, int nz, uint32_t C, int g[3], uint64_t* cells)
{
    if (C < 4 || C > 64) return fail(VDBC_E_INVALID, "macrocell must be in [4, 64]");   // sizes kMajorantQueue
    g[0] = (int)(((int64_t)nx + C - 1) / C);
    g[1] = (int)(((int64_t)ny + C - 1) / C);
    g[2] = (int)(((int64_t)nz + C - 1) / C);
    *cells = (uint64_t)g[0] * g[1] * g[2];
    if (*cells > 0x7FFFFFFFull)
        return fail(VDBC_E_INVALID, "too many macrocells (%llu)", (unsigned long long)*cells);
    return VDBC_OK;
}

static vdbc_status launch_majorant(const VdbView& v, const MediumK& m, uint32_t C, float* out, hipStream_t st)
{
    int g[3];
    uint64_t cells;
    vdbc_status s = majorant_cells(v.nx, v.ny, v.nz, C, g, &cells);
    if (s) return s;
    hipLaunchKernelGGL(majorant_tree_kernel, wide_grid(majorant_groups((int)C, cells)), dim3(kBlock), 0, st, v, m,
                       (int)C, g[0], g[1], g[2], out);
    return launch_check("majorant");
}

static vdbc_status launch_majorant(const DenseView& v, const MediumK& m, uint32_t C, float* out, hipStream_t st)
{
    int g[3];
    uint64_t cells;
    vdbc_status s = majorant_cells(v.nx, v.ny, v.nz, C, g, &cells);
    if (s) return s;
    // 256, 128 or 64 voxels of cells: fewer where the volume is narrower, or where
    // workgroups would be too few for the card (cells of 64 at 512^3: 437 us with
    // 128 workgroups of 256 voxels, 223 with 512 of 64)
    int width = 256, run = 0, runs = 0;
    for (;; width /= 2) {
        run = width / (int)C;
        runs = (g[0] + run - 1) / run;
        if (width == 64 || (v.nx > width / 2 && (uint64_t)runs * g[1] * g[2] >= 512)) break;
    }
    int wl = 4;   // lanes a row
    while (wl < 8 && (1 << wl) < std::min(run * (int)C, v.nx)) ++wl;
    const dim3 grid = wide_grid((uint64_t)runs * g[1] * g[2]);
    if (wl < 6)
        hipLaunchKernelGGL(majorant_dense_kernel<true>, grid, dim3(kBlock), 0, st, v, m, (int)C, g[0], g[1], g[2], run, runs,
                           wl, out);
    else
        hipLaunchKernelGGL(majorant_dense_kernel<false>, grid, dim3(kBlock), 0, st, v, m, (int)C, g[0], g[1], g[2], run, runs,
                           wl, out);
    return launch_check("majorant");
}

static vdbc_status launch_index_of(const VdbView& v, const IndexPlan& ix, hipStream_t st) { return launch_index(v, ix, st); }
static vdbc_status launch_index_of(const DenseView&, const IndexPlan&, hipStream_t) { return VDBC_OK; }

// Compute units of the current device (cached per device; 256 if unknown).
static int device_cus()
{
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
    if (dev < 64 && cache[dev].load(std::memory_order_relaxed) > 0)
        return cache[dev].load(std::memory_order_relaxed);
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    if (dev < 64) cache[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// Whether the marchers may skip empty blocks, asked to or not: the image stays
// the same bit for bit while a sample's position is rounded by far less than
// kHddaEps.  A ray's parameter is at most the distance T from its origin to a
// corner of the volume; the exit's plane distance, its product with the
// reciprocal, the lattice index, the sample's parameter and its position round
// by some 4.5 units in the last place of T together, 0.0088 voxels at 2^15.  (From
// 300,000 voxels away 0.6 % of the skips would pass over a sample that reads more
// than the background.)
static bool skip_is_exact(const CameraK& c, const VdbView& v)
{
    double far2 = 0.0;
    for (int corner = 0; corner < (c.kind == 1 ? 8 : 32); ++corner) {
        const double x[3] = {(corner & 1) ? v.nx - 0.5 : -0.5, (corner & 2) ? v.ny - 0.5 : -0.5,
                             (corner & 4) ? v.nz - 0.5 : -0.5};
        double d2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double o = c.kind == 1 ? (double)c.o[a]
                                         : (double)c.ll[a] + ((corner & 8) ? (double)c.du[a] * c.width : 0.0) +
                                               ((corner & 16) ? (double)c.dv[a] * c.height : 0.0);
            d2 += (x[a] - o) * (x[a] - o);
        }
        far2 = std::max(far2, d2);
    }
    return far2 <= 32768.0 * 32768.0;
}

// Whether a frame with VDBC_RENDER_HDDA that may not skip by the region index
// goes through the tree, whose own skips keep a step of margin: in volumes so
// large that rays pass mostly through empty space.  (Of a smaller one far away
// all samples are taken: 512^2 pixels of a 512^3 cloud from 3 10^5 voxels 1.2 ms,
// 3.3 ms by the tree.)
static bool march_by_tree(bool hdda, bool exact, const VdbView& v)
{
    return hdda && !exact && std::max({v.nx, v.ny, v.nz}) > 8192;
}

// MARCH = false leaves out the EA and ISO kernels (accessor variants that
// only the path tracer uses).
template <class Acc, class View, bool MARCH = true>
static vdbc_status render_impl(const View& v, const vdbc_camera* c, const vdbc_medium* med,
                               const vdbc_render_params* r, float* image, float* aov, void* ws,
                               uint64_t ws_bytes, void* stream, const IndexPlan& ix = IndexPlan())
{
    if (!r || !image) return fail(VDBC_E_INVALID, "null params or image");
    CameraK cam;
    MediumK m;
    vdbc_status s = make_camera(c, &cam);
    if (s) return s;
    if (r->mode > 2) return fail(VDBC_E_INVALID, "mode must be EA (0), PT (1) or ISO (2)");
    if (r->mode != VDBC_MODE_ISO) {
        s = make_medium(med, v.nx, v.ny, v.nz, &m);
        if (s) return s;
    }
    const bool count = (r->flags & VDBC_RENDER_COUNT) != 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned long long* counter = reinterpret_cast<unsigned long long*>(ws);
    vdbc_dims d{(uint32_t)v.nx, (uint32_t)v.ny, (uint32_t)v.nz};
    uint64_t need = 0;
    s = vdbc_render_workspace(r, d, c, &need);
    if (s) return s;
    if (need && (!ws || ws_bytes < need))
        return fail(VDBC_E_BUFFER_TOO_SMALL, "workspace needs %llu bytes", (unsigned long long)need);
    if (ws && reinterpret_cast<uintptr_t>(ws) % 256)
        return fail(VDBC_E_INVALID, "workspace must be 256-byte aligned");
    dim3 grid((cam.width + kTile - 1) / kTile, (cam.height + kTile - 1) / kTile);
    const dim3 quads = wide_grid((uint64_t)((cam.width + 7) / 8) * (uint64_t)((cam.height + 7) / 8));   // 8 x 8 pixels
    if constexpr (MARCH) {
        if (r->mode == VDBC_MODE_ISO) {
            if (!(r->step > 0.0f) || !std::isfinite(r->step))
                return fail(VDBC_E_INVALID, "ISO step must be finite and > 0");
            const double diag = std::sqrt((double)v.nx * v.nx + (double)v.ny * v.ny + (double)v.nz * v.nz);
            if (diag / r->step > 16777216.0)
                return fail(VDBC_E_INVALID, "ISO step too small for this volume (> 2^24 samples per ray)");
            if (!std::isfinite(r->iso)) return fail(VDBC_E_INVALID, "iso value must be finite");
            if (r->refine > 64) return fail(VDBC_E_INVALID, "refine must be <= 64");
            if (count) {
                hipLaunchKernelGGL(zero_u64, dim3(1), dim3(64), 0, st, counter);
                if ((s = launch_check("zero counter"))) return s;
            }
            const bool hdda = (r->flags & VDBC_RENDER_HDDA) != 0;
#define ISO_QUAD(ACC, VIEW, FIELD, SKIP)                                                                          \
    hipLaunchKernelGGL((iso_quad_kernel<ACC, VIEW, SKIP>), quads, dim3(kBlock), 0, st, FIELD, cam, r->iso, r->step, \
                       1.0f / r->step, (int)r->refine, image, aov)
            if constexpr (std::is_same_v<Acc, DenseAcc>) {
                if (count)
                    hipLaunchKernelGGL((iso_kernel<Acc, View, false, true>), grid, dim3(kBlock), 0, st, v, cam, r->iso,
                                       r->step, (int)r->refine, image, aov, counter);
                else
                    ISO_QUAD(DenseAcc, DenseView, v, false);
                return launch_check("iso render");
            } else {
            const bool skip = skip_is_exact(cam, v);
            if (ix.on && !count && !march_by_tree(hdda, skip, v)) {
                if ((s = launch_index(v, ix, st))) return s;
                if (ix.wide && skip) ISO_QUAD(IndexAccT<true>, IndexView, ix.v, true);
                else if (ix.wide) ISO_QUAD(IndexAccT<true>, IndexView, ix.v, false);
                else if (skip) ISO_QUAD(IndexAccT<false>, IndexView, ix.v, true);
                else ISO_QUAD(IndexAccT<false>, IndexView, ix.v, false);
                return launch_check("iso render");
            }
#undef ISO_QUAD
    #define ISO_LAUNCH(H, CNT)                                                                      \
        hipLaunchKernelGGL((iso_kernel<Acc, View, H, CNT>), grid, dim3(kBlock), 0, st, v, cam, r->iso, \
                           r->step, (int)r->refine, image, aov, counter)
            if (hdda) {
                if (count) ISO_LAUNCH(true, true);
                else ISO_LAUNCH(true, false);
            } else {
                if (count) ISO_LAUNCH(false, true);
                else ISO_LAUNCH(false, false);
            }
    #undef ISO_LAUNCH
            return launch_check("iso render");
            }
        }
        if (count && r->mode == VDBC_MODE_EA) {
            hipLaunchKernelGGL(zero_u64, dim3(1), dim3(64), 0, st, counter);
            if ((s = launch_check("zero counter"))) return s;
        }
        if (r->mode == VDBC_MODE_EA) {
            if (!(r->step > 0.0f) || !std::isfinite(r->step))
                return fail(VDBC_E_INVALID, "EA step must be finite and > 0");
            // bound the per-ray loop: box diagonal / step <= 2^24 samples
            const double diag = std::sqrt((double)v.nx * v.nx + (double)v.ny * v.ny + (double)v.nz * v.nz);
            if (diag / r->step > 16777216.0)
                return fail(VDBC_E_INVALID, "EA step too small for this volume (> 2^24 samples per ray)");
            const bool clear = host_alpha(m, v.background) == 0.0f;
            const bool hdda = (r->flags & VDBC_RENDER_HDDA) && clear;
            // past 1 a ray ends at the first sample it takes: which one that is
            // stays with the kernel of one thread per ray and its own skips
            const bool first_only = r->t_terminate > 1.0f;
#define EA_QUAD(ACC, VIEW, FIELD, SKIP)                                                                          \
    hipLaunchKernelGGL((ea_quad_kernel<ACC, VIEW, SKIP>), quads, dim3(kBlock), 0, st, FIELD, cam, m, r->step, \
                       1.0f / r->step, r->t_terminate, image)
            if constexpr (std::is_same_v<Acc, DenseAcc>) {
                if (count)
                    hipLaunchKernelGGL((ea_kernel<Acc, View, false, true>), grid, dim3(kBlock), 0, st, v, cam, m,
                                       r->step, r->t_terminate, image, counter);
                else
                    EA_QUAD(DenseAcc, DenseView, v, false);
                return launch_check("ea render");
            } else {
            const bool exact = skip_is_exact(cam, v), skip = clear && exact;
            if (ix.on && !count && !first_only && !march_by_tree(hdda, exact, v)) {
                if ((s = launch_index(v, ix, st))) return s;
                if (ix.wide && skip) EA_QUAD(IndexAccT<true>, IndexView, ix.v, true);
                else if (ix.wide) EA_QUAD(IndexAccT<true>, IndexView, ix.v, false);
                else if (skip) EA_QUAD(IndexAccT<false>, IndexView, ix.v, true);
                else EA_QUAD(IndexAccT<false>, IndexView, ix.v, false);
                return launch_check("ea render");
            }
#undef EA_QUAD
    #define EA_LAUNCH(H, CNT)                                                                      \
        hipLaunchKernelGGL((ea_kernel<Acc, View, H, CNT>), grid, dim3(kBlock), 0, st, v, cam, m, \
                           r->step, r->t_terminate, image, counter)
            if (hdda) {
                if (count) EA_LAUNCH(true, true);
                else EA_LAUNCH(true, false);
            } else {
                if (count) EA_LAUNCH(false, true);
                else EA_LAUNCH(false, false);
            }
    #undef EA_LAUNCH
            return launch_check("ea render");
            }
        }
    } else if (r->mode != VDBC_MODE_PT) {
        return fail(VDBC_E_UNSUPPORTED, "accessor variant for the path tracer only");
    }
    // the tile's work units (256 x spp) are 32-bit and the bounce is a
    // 16-bit field of the random-number counter
    if (r->spp == 0 || r->spp > kMaxSpp || r->max_bounces == 0 || r->max_bounces > kMaxBounces)
        return fail(VDBC_E_INVALID, "need 1 <= spp <= %u and 1 <= max_bounces <= %u", kMaxSpp, kMaxBounces);
    if (r->tile_w != 0 && r->tile_w != 8 && r->tile_w != 16 && r->tile_w != 32 && r->tile_w != 64)
        return fail(VDBC_E_INVALID, "tile_w must be 0 (default 8), 8, 16, 32 or 64");
    {
        // the work-item queue counts in 32 bits
        const uint64_t tiles = pt_tiles((uint64_t)cam.width, (uint64_t)cam.height, r->tile_w == 0 ? 8 : r->tile_w);
        const uint32_t chunk = pt_chunk(r, c);
        const uint64_t per_tile = (r->spp + chunk - 1) / chunk;
        if (tiles * per_tile > 0xFFFFFFFFull)
            return fail(VDBC_E_INVALID, "more than 2^32 work items: raise chunk_spp");
    }
    {
        const double l = std::sqrt((double)med->light_dir[0] * med->light_dir[0] +
                                   (double)med->light_dir[1] * med->light_dir[1] +
                                   (double)med->light_dir[2] * med->light_dir[2]);
        if (!(std::fabs(l - 1.0) <= 1e-3)) return fail(VDBC_E_INVALID, "light_dir must be a unit vector");
        if (!std::isfinite(med->albedo) || med->albedo < 0.0f)
            return fail(VDBC_E_INVALID, "albedo must be finite and >= 0");
    }
    hipLaunchKernelGGL(zero_u64, dim3(1), dim3(64), 0, st, counter);   // counters and tile queue
    if ((s = launch_check("zero counters"))) return s;
    float* maj = reinterpret_cast<float*>(static_cast<uint8_t*>(ws) + 256);
    if (!(r->flags & VDBC_RENDER_KEEP_MAJORANT)) {
        s = launch_majorant(v, m, r->macrocell, maj, st);
        if (s) return s;
    }
    PtArgs g;
    pt_geometry(r->macrocell, v.nx, v.ny, v.nz, &g);
    g.spp = (int)r->spp;
    g.max_bounces = (int)r->max_bounces;
    g.tw = r->tile_w == 0 ? 8 : (int)r->tile_w;
    g.twl = __builtin_ctz((unsigned)g.tw);
    g.seed_lo = (uint32_t)r->seed;
    g.seed_hi = (uint32_t)(r->seed >> 32);
    g.frame = r->frame;
    g.rr = (r->flags & VDBC_RENDER_RR) ? 1 : 0;
    const bool split = pt_split(r, c);
    g.chunk = pt_chunk(r, c);
    g.chunks = (r->spp + g.chunk - 1) / g.chunk;
    uint32_t* coarse = reinterpret_cast<uint32_t*>(
        static_cast<uint8_t*>(ws) + 256 + align256(majorant_bytes(r->macrocell, v.nx, v.ny, v.nz)));
    const uint64_t npix = (uint64_t)cam.width * (uint64_t)cam.height;
    const uint64_t tiles = pt_tiles((uint64_t)cam.width, (uint64_t)cam.height, (uint64_t)g.tw);
    uint8_t* const tail = static_cast<uint8_t*>(ws) + pt_workspace(r->macrocell, v.nx, v.ny, v.nz);
    PtSums sums{};
    if (split) {
        uint8_t* base = tail;
        sums.rgbn = reinterpret_cast<unsigned long long*>(base);
        sums.depth = sums.rgbn + 4 * npix;
        const uint64_t words = pt_sums_bytes(npix) / 16;
        hipLaunchKernelGGL(pt_sums_clear_kernel, dim3((unsigned)std::min<uint64_t>((words + kBlock - 1) / kBlock, 4096)),
                           dim3(kBlock), 0, st, reinterpret_cast<uint4*>(base), words);
        if ((s = launch_check("clear pixel sums"))) return s;
    }
    {
        const uint64_t ncoarse = (uint64_t)g.cgx * g.cgy * g.cgz;
        hipLaunchKernelGGL(coarse_bits_kernel, dim3((unsigned)((ncoarse + kCoarsePerGroup - 1) / kCoarsePerGroup)),
                           dim3(kBlock), 0, st, maj, g, coarse);
        if ((s = launch_check("coarse occupancy"))) return s;
    }
    const uint32_t* order = nullptr;
    if (pt_ordered(r, c)) {
        uint32_t* key = reinterpret_cast<uint32_t*>(tail + (split ? pt_sums_bytes(npix) : 0)) + 2 * kCostBins;
        uint32_t* ord = key + tiles;
        constexpr uint64_t per_group = kBlock / kCostLanes;
        hipLaunchKernelGGL(pt_tile_cost_kernel, dim3((unsigned)((tiles + per_group - 1) / per_group)), dim3(kBlock), 0, st, cam,
                           g, v.nx, v.ny, v.nz, maj, (uint32_t)pt_tiles_x((uint64_t)cam.width, (uint64_t)g.tw),
                           (uint32_t)tiles, key);
        hipLaunchKernelGGL(pt_cost_order_kernel, dim3(1), dim3(1024), 0, st, key, ord, (uint32_t)tiles);
        if ((s = launch_check("cost order"))) return s;
        order = ord;
    }
    if (ix.on && (s = launch_index_of(v, ix, st))) return s;
    const size_t lds = 4u * (size_t)g.cwords;
    const int per_cu = ix.on ? kPtBlocksPerCu<IndexAccT<false>> : kPtBlocksPerCu<Acc>;
    grid = dim3((unsigned)std::min<uint64_t>(tiles * g.chunks, (uint64_t)device_cus() * (uint64_t)per_cu));
    uint32_t* queue = reinterpret_cast<uint32_t*>(counter + 2);
#define PT_LAUNCH_ACC(ACC, VIEW, FIELD, CNT, AO, EN)                                                  \
    hipLaunchKernelGGL((pt_kernel<ACC, VIEW, CNT, AO, EN>), grid, dim3(kBlock), lds, st, FIELD, cam, m, \
                       g, maj, coarse, image, aov, counter, queue, sums, order)
#define PT_LAUNCH(CNT, AO, EN)                                                          \
    if constexpr (std::is_same_v<Acc, VdbAcc>) {                                        \
        if (ix.on && ix.wide) PT_LAUNCH_ACC(IndexAccT<true>, IndexView, ix.v, CNT, AO, EN); \
        else if (ix.on) PT_LAUNCH_ACC(IndexAccT<false>, IndexView, ix.v, CNT, AO, EN);  \
        else PT_LAUNCH_ACC(Acc, View, v, CNT, AO, EN);                                  \
    } else PT_LAUNCH_ACC(Acc, View, v, CNT, AO, EN)
#define PT_LAUNCH_ENV(CNT, AO)               \
    if (m.env) { PT_LAUNCH(CNT, AO, true); } \
    else { PT_LAUNCH(CNT, AO, false); }
    if (count) {
        if (aov) { PT_LAUNCH_ENV(true, true) }
        else { PT_LAUNCH_ENV(true, false) }
    } else {
        if (aov) { PT_LAUNCH_ENV(false, true) }
        else { PT_LAUNCH_ENV(false, false) }
    }
#undef PT_LAUNCH_ENV
#undef PT_LAUNCH
#undef PT_LAUNCH_ACC
    if (split) {
        if ((s = launch_check("pt render"))) return s;
        hipLaunchKernelGGL(pt_resolve_kernel, dim3((unsigned)((npix + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, sums,
                           image, aov, (uint32_t)npix, g.spp);
        return launch_check("pixel sums to image");
    }
    return launch_check("pt render");
}

}  // namespace vdbc

using namespace vdbc;

extern "C" vdbc_status vdbc_render_workspace(const vdbc_render_params* r, vdbc_dims d,
                                             const vdbc_camera* c, uint64_t* bytes)
{
    if (!r || !bytes) return fail(VDBC_E_INVALID, "null argument");
    if (d.nx == 0 || d.ny == 0 || d.nz == 0) return fail(VDBC_E_INVALID, "zero dims");
    if (r->mode == VDBC_MODE_PT) {
        if (r->macrocell < 4 || r->macrocell > 64 || (r->macrocell & (r->macrocell - 1)))
            return fail(VDBC_E_INVALID, "macrocell must be 4, 8, 16, 32 or 64");
        *bytes = pt_workspace(r->macrocell, (int)d.nx, (int)d.ny, (int)d.nz);
        const bool library = r->chunk_spp == 0 && (r->flags & VDBC_RENDER_SPLIT) != 0;
        if (library || (r->chunk_spp != 0 && r->chunk_spp < r->spp)) {
            if (!c) return fail(VDBC_E_INVALID, "work split: the workspace size needs the camera");
        } else if ((r->flags & VDBC_RENDER_COST_ORDER) && !c) {
            return fail(VDBC_E_INVALID, "VDBC_RENDER_COST_ORDER: the workspace size needs the camera");
        }
        if ((library || (r->flags & VDBC_RENDER_COST_ORDER)) && r->tile_w != 0 && r->tile_w != 8 && r->tile_w != 16 &&
            r->tile_w != 32 && r->tile_w != 64)
            return fail(VDBC_E_INVALID, "tile_w must be 0 (default 8), 8, 16, 32 or 64");
        if (pt_split(r, c)) *bytes += pt_sums_bytes((uint64_t)c->width * (uint64_t)c->height);
        if (pt_ordered(r, c)) *bytes += pt_order_bytes(pt_tiles(c->width, c->height, r->tile_w == 0 ? 8 : r->tile_w));
        if (r->flags & VDBC_RENDER_INDEX) {
            uint64_t t[3];
            *bytes += index_dims(d.nx, d.ny, d.nz, t);
        }
    } else {
        *bytes = (r->flags & VDBC_RENDER_COUNT) ? 256 : 0;
        if (r->flags & VDBC_RENDER_INDEX) {
            uint64_t t[3];
            if (index_dims(d.nx, d.ny, d.nz, t)) *bytes += index_dims(d.nx, d.ny, d.nz, t) + align256(t[0] * t[1] * t[2]);
        }
    }
    return VDBC_OK;
}

static vdbc_status render_vdb(const vdbc_grid* g, const vdbc_camera* c, const vdbc_medium* m,
                              const vdbc_render_params* r, float* image, float* aov, void* ws,
                              uint64_t ws_bytes, void* stream)
{
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    // path tracer only: the accessor's cache policy (a tuning knob; the image
    // does not depend on it)
    const uint32_t pol = r ? (r->flags & (VDBC_RENDER_CACHE_NONE | VDBC_RENDER_CACHE_LEAF)) : 0u;
    if (pol == (VDBC_RENDER_CACHE_NONE | VDBC_RENDER_CACHE_LEAF))
        return fail(VDBC_E_INVALID, "at most one cache-policy flag");
    if (pol && r->mode == VDBC_MODE_PT) {
        if (pol == VDBC_RENDER_CACHE_NONE)
            return render_impl<VdbAccT<kCacheNone>, VdbView, false>(v, c, m, r, image, aov, ws, ws_bytes, stream);
        return render_impl<VdbAccT<kCacheLeaf>, VdbView, false>(v, c, m, r, image, aov, ws, ws_bytes, stream);
    }
    IndexPlan ix;
    if (r && r->mode <= 2 && (r->flags & VDBC_RENDER_INDEX) && ws) {
        // the table is the last part of the workspace (its size is checked
        // with the rest of it below, before anything is enqueued)
        uint64_t need = 0, t[3];
        vdbc_dims d{(uint32_t)v.nx, (uint32_t)v.ny, (uint32_t)v.nz};
        const uint64_t tab = index_dims(d.nx, d.ny, d.nz, t);
        if ((s = vdbc_render_workspace(r, d, c, &need))) return s;
        const uint64_t levels = tab && r->mode != VDBC_MODE_PT ? align256(t[0] * t[1] * t[2]) : 0;
        uint8_t* const at = static_cast<uint8_t*>(ws) + need - tab - levels;
        ix.on = tab && make_index(g, v, reinterpret_cast<uint32_t*>(at), &ix.v, &ix.wide);
        if (levels) ix.v.level = at + tab;
    }
    return render_impl<VdbAcc>(v, c, m, r, image, aov, ws, ws_bytes, stream, ix);
}

// The parameters of a call with VDBC_RENDER_SPLIT taken back where the
// workspace has no room for the pixel sums and the order (it is a choice of the library's,
// not a demand).
static const vdbc_render_params* fit_split(const vdbc_render_params* r, vdbc_dims d, const vdbc_camera* c,
                                           uint64_t ws_bytes, vdbc_render_params* whole)
{
    uint64_t need = 0;
    if (!r || !(r->flags & VDBC_RENDER_SPLIT) || vdbc_render_workspace(r, d, c, &need) || need <= ws_bytes) return r;
    *whole = *r;
    whole->flags &= ~(uint32_t)VDBC_RENDER_SPLIT;
    return whole;
}

extern "C" vdbc_status vdbc_render(const vdbc_grid* g, const vdbc_camera* c, const vdbc_medium* m,
                                   const vdbc_render_params* r, float* image, float* aov, void* ws,
                                   uint64_t ws_bytes, void* stream)
{
    clear_error();
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    vdbc_render_params whole;
    r = fit_split(r, vdbc_dims{(uint32_t)v.nx, (uint32_t)v.ny, (uint32_t)v.nz}, c, ws_bytes, &whole);
    return render_vdb(g, c, m, r, image, aov, ws, ws_bytes, stream);
}

// ---------------------------------------------------------------- render without allocation

// Fixed scratch of vdbc_render_noalloc: the render workspace (counters, tile
// queue, majorant grid, coarse occupancy bits) of one call.  Every GPU the
// library runs on holds its own copy until the process ends.  Host code never
// passes the symbol itself to a kernel: it takes the device address that
// hipGetSymbolAddress returns for the current device.
constexpr uint64_t kScratchBytes = VDBC_NOALLOC_SCRATCH_BYTES;
__device__ __align__(256) uint8_t scratch[kScratchBytes];

// Device address of `scratch` on the current device, resolved once per
// device (with that device current) on its first call.
static vdbc_status scratch_address(void** out)
{
    static std::mutex mu;
    static void* addr[64] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(VDBC_E_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= 64) return fail(VDBC_E_UNSUPPORTED, "device index %d beyond 63", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(VDBC_E_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                        hipGetErrorString(e));
        addr[dev] = p;
    }
    *out = addr[dev];
    return VDBC_OK;
}

extern "C" vdbc_status vdbc_render_noalloc(const vdbc_grid* g, const vdbc_camera* c,
                                           const vdbc_medium* m, const vdbc_render_params* r,
                                           float* image, float* aov, void* stream)
{
    clear_error();
    if (!g || !r) return fail(VDBC_E_INVALID, "null grid or params");
    if (r->flags & VDBC_RENDER_KEEP_MAJORANT)
        return fail(VDBC_E_INVALID, "VDBC_RENDER_KEEP_MAJORANT: the scratch holds no majorant of the caller's");
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    vdbc_dims d{(uint32_t)v.nx, (uint32_t)v.ny, (uint32_t)v.nz};
    vdbc_render_params whole;
    r = fit_split(r, d, c, kScratchBytes, &whole);
    uint64_t need = 0;
    if ((s = vdbc_render_workspace(r, d, c, &need))) return s;
    if (need > kScratchBytes)
        return fail(VDBC_E_BUFFER_TOO_SMALL, "this render needs %llu bytes of scratch; the fixed scratch holds %llu "
                    "(use vdbc_render with a workspace, a larger macrocell or chunk_spp 0)",
                    (unsigned long long)need, (unsigned long long)kScratchBytes);
    void* ws = nullptr;
    if ((s = scratch_address(&ws))) return s;
    return render_vdb(g, c, m, r, image, aov, ws, kScratchBytes, stream);
}

extern "C" vdbc_status vdbc_render_dense(const float* dense, vdbc_dims d, float background,
                                         const vdbc_camera* c, const vdbc_medium* m,
                                         const vdbc_render_params* r, float* image, float* aov,
                                         void* ws, uint64_t ws_bytes, void* stream)
{
    clear_error();
    DenseView v;
    vdbc_status s = make_dense(dense, d, background, &v);
    if (s) return s;
    vdbc_render_params whole;
    r = fit_split(r, d, c, ws_bytes, &whole);
    return render_impl<DenseAcc>(v, c, m, r, image, aov, ws, ws_bytes, stream);
}

extern "C" vdbc_status vdbc_majorant(const vdbc_grid* g, const vdbc_medium* med, uint32_t C,
                                     float* out, void* stream)
{
    clear_error();
    VdbView v;
    vdbc_status s = make_view(g, &v);
    if (s) return s;
    if (!out) return fail(VDBC_E_INVALID, "null output");
    if (C < 4 || C > 64) return fail(VDBC_E_INVALID, "macrocell must be in [4, 64]");
    MediumK m;
    if ((s = make_medium(med, v.nx, v.ny, v.nz, &m))) return s;
    return launch_majorant(v, m, C, out, static_cast<hipStream_t>(stream));
}

extern "C" vdbc_status vdbc_majorant_dense(const float* dense, vdbc_dims d, float background,
                                           const vdbc_medium* med, uint32_t C, float* out,
                                           void* stream)
{
    clear_error();
    DenseView v;
    vdbc_status s = make_dense(dense, d, background, &v);
    if (s) return s;
    if (!out) return fail(VDBC_E_INVALID, "null output");
    if (C < 4 || C > 64) return fail(VDBC_E_INVALID, "macrocell must be in [4, 64]");
    MediumK m;
    if ((s = make_medium(med, v.nx, v.ny, v.nz, &m))) return s;
    return launch_majorant(v, m, C, out, static_cast<hipStream_t>(stream));
}

// ---------------------------------------------------------------- batched majorants
// The majorant grids and the coarse occupancy bits of every volume of a batch
// in one launch each, with the per-cell code of the single-volume kernels (so
// the grids and bits are bitwise those of per-volume launches): workgroup b
// belongs to the volume v with base[v] <= b < base[v + 1], a prefix table of
// the volumes' majorant (coarse-bit) workgroups, and works on its local
// index b - base[v].  Small volumes no longer leave the chip idle one launch
// at a time.

namespace vdbc {

__device__ inline uint32_t batch_volume_of(const uint32_t* __restrict__ base, uint32_t n, uint32_t b)
{
    uint32_t lo = 0, hi = n;   // base[lo] <= b < base[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (base[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(kBlock) void majorant_batch_kernel(const BatchDesc* __restrict__ descs,
                                                                const uint32_t* __restrict__ base, uint32_t n)
{
    __shared__ uint32_t s_v;
    if (threadIdx.x == 0) s_v = batch_volume_of(base, n, blockIdx.x);
    __syncthreads();
    const uint32_t v = s_v;
    const BatchDesc* D = descs + v;
    majorant_tree_group(D->view, D->med, D->g.C, D->g.gx, D->g.gy, D->g.gz, blockIdx.x - base[v],
                        const_cast<float*>(D->maj));
}

__global__ __launch_bounds__(kBlock) void index_batch_kernel(const BatchDesc* __restrict__ descs,
                                                             const uint32_t* __restrict__ base, uint32_t n, int shift)
{
    const uint32_t v = batch_volume_of(base, n, blockIdx.x);
    const BatchDesc* D = descs + v;
    index_entry(D->view, D->index, (blockIdx.x - base[v]) * kBlock + threadIdx.x, const_cast<uint32_t*>(D->index.tab),
                shift);
}

__global__ __launch_bounds__(kBlock) void coarse_bits_batch_kernel(const BatchDesc* __restrict__ descs,
                                                                   const uint32_t* __restrict__ base, uint32_t n)
{
    // every thread finds the volume itself: a workgroup lies in one volume,
    // and no barrier is needed before the ballot
    const uint32_t v = batch_volume_of(base, n, blockIdx.x);
    const BatchDesc* D = descs + v;
    coarse_bits_block(D->maj, D->g, const_cast<uint32_t*>(D->coarse), blockIdx.x - base[v]);
}

}  // namespace vdbc

// ---------------------------------------------------------------- batched PT (host)

struct vdbc_batch {
    uint32_t n = 0;
    vdbc_tuning t{};
    std::vector<VdbView> views;
    std::vector<CameraK> cams;
    std::vector<MediumK> meds;
    std::vector<PtArgs> gs;
    std::vector<float*> majs;
    std::vector<uint32_t*> coarse;
    std::vector<float*> images;
    std::vector<PtSums> sums;          // per volume: pixel sums of split items, or null
    std::vector<int> tiles_x, tiles_y;
    BatchDesc* d_descs = nullptr;
    uint32_t* d_items = nullptr;
    uint32_t* d_counter = nullptr;
    uint32_t* d_cell_base = nullptr;     // prefix tables of majorant and coarse-bit workgroups
    uint32_t* d_coarse_base = nullptr;
    uint32_t* d_index_base = nullptr;    // ... and of index workgroups
    uint64_t mblocks_total = 0, cblocks_total = 0, iblocks_total = 0;
    // region indexes of all volumes (in bytes, or wide where one of them
    // needs it), or of none where one cannot have any
    std::vector<IndexPlan> index;
    bool indexed = false, wide = false, env = false;
    uint32_t n_items = 0;
    int max_cwords = 0;
    int grid_blocks = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace vdbc {

static vdbc_status batch_tuning(const vdbc_tuning* t, vdbc_tuning* out)
{
    vdbc_tuning d{16, 8, 4, 1, 0};
    if (t) d = *t;
    if (d.macrocell < 4 || d.macrocell > 64 || (d.macrocell & (d.macrocell - 1)))
        return fail(VDBC_E_INVALID, "tuning.macrocell must be 4, 8, 16, 32 or 64");
    if (d.tile_w == 0) d.tile_w = 8;
    if (d.tile_w != 8 && d.tile_w != 16 && d.tile_w != 32 && d.tile_w != 64)
        return fail(VDBC_E_INVALID, "tuning.tile_w must be 8, 16, 32 or 64");
    if (d.blocks_per_cu == 0) d.blocks_per_cu = 4;
    if (d.blocks_per_cu > 32) return fail(VDBC_E_INVALID, "tuning.blocks_per_cu must be <= 32");
    *out = d;
    return VDBC_OK;
}

// Bytes of a batch volume's pixel sums (32 per pixel: RGB and the hit and
// escape counts; the batched launch writes no depth).
static uint64_t batch_sums_bytes(uint64_t npix) { return align256(32ull * npix); }

// Validates the items and fills the per-volume launch state; the offsets
// receive the workspace layout (counter, descriptors, item list, then per
// volume majorant, coarse bits and, for a split volume, its pixel sums; 0 for
// a volume that is not split) and the total size.
static vdbc_status batch_plan(const vdbc_batch_item* items, uint32_t n, const vdbc_tuning& t, vdbc_batch* b,
                              std::vector<uint64_t>* maj_off, std::vector<uint64_t>* coarse_off,
                              std::vector<uint64_t>* sums_off, std::vector<uint64_t>* index_off,
                              uint64_t* items_off, uint64_t* total)
{
    if (!items || n == 0 || n > 4096) return fail(VDBC_E_INVALID, "need 1..4096 batch items");
    b->n = n;
    b->t = t;
    uint64_t tiles_total = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const vdbc_batch_item& it = items[i];
        VdbView v;
        CameraK cam;
        MediumK m;
        vdbc_status s = make_view(&it.grid, &v);
        if (!s) s = make_camera(&it.camera, &cam);
        if (!s) s = make_medium(&it.medium, v.nx, v.ny, v.nz, &m);
        if (s) return fail(s, "batch item %u: %s", i, vdbc_last_error());
        if (it.spp == 0 || it.spp > kMaxSpp || it.max_bounces == 0 || it.max_bounces > kMaxBounces || !it.image)
            return fail(VDBC_E_INVALID, "batch item %u: need 1 <= spp <= %u, 1 <= max_bounces <= %u and an image", i,
                        kMaxSpp, kMaxBounces);
        const double l = std::sqrt((double)it.medium.light_dir[0] * it.medium.light_dir[0] +
                                   (double)it.medium.light_dir[1] * it.medium.light_dir[1] +
                                   (double)it.medium.light_dir[2] * it.medium.light_dir[2]);
        if (!(std::fabs(l - 1.0) <= 1e-3)) return fail(VDBC_E_INVALID, "batch item %u: light_dir not unit", i);
        PtArgs g;
        pt_geometry(t.macrocell, v.nx, v.ny, v.nz, &g);
        g.spp = (int)it.spp;
        g.max_bounces = (int)it.max_bounces;
        g.tw = (int)t.tile_w;
        g.twl = __builtin_ctz((unsigned)g.tw);
        g.seed_lo = (uint32_t)it.seed;
        g.seed_hi = (uint32_t)(it.seed >> 32);
        g.frame = it.frame;
        g.rr = 0;
        const bool split = t.chunk_spp != 0 && t.chunk_spp < it.spp;
        g.chunk = split ? t.chunk_spp : (uint32_t)g.spp;
        g.chunks = split ? (it.spp + t.chunk_spp - 1) / t.chunk_spp : 1u;
        const int tx = (int)pt_tiles_x((uint64_t)cam.width, (uint64_t)g.tw),
                  ty = (int)(pt_tiles((uint64_t)cam.width, (uint64_t)cam.height, (uint64_t)g.tw) / (uint64_t)tx);
        if ((uint64_t)tx * ty * g.chunks > 0xFFFFFu)
            return fail(VDBC_E_INVALID, "batch item %u: image too large for %u work items per tile", i, g.chunks);
        b->views.push_back(v);
        b->cams.push_back(cam);
        b->meds.push_back(m);
        b->gs.push_back(g);
        b->images.push_back(it.image);
        b->tiles_x.push_back(tx);
        b->tiles_y.push_back(ty);
        tiles_total += (uint64_t)tx * ty * g.chunks;
        b->max_cwords = std::max(b->max_cwords, g.cwords);
    }
    uint64_t o = 256;                                   // counter
    const uint64_t descs_off = o;
    o += align256((uint64_t)n * sizeof(BatchDesc));
    o += align256(12ull * (n + 1));                     // the prefix tables of the batched set-up launches
    *items_off = o;
    o += align256(tiles_total * 4);
    for (uint32_t i = 0; i < n; ++i) {
        maj_off->push_back(o);
        o += align256(majorant_bytes(t.macrocell, b->views[i].nx, b->views[i].ny, b->views[i].nz));
        coarse_off->push_back(o);
        o += align256(4ull * b->gs[i].cwords);
        if (b->gs[i].chunks > 1) {
            sums_off->push_back(o);
            o += batch_sums_bytes((uint64_t)b->cams[i].width * b->cams[i].height);
        } else {
            sums_off->push_back(0);
        }
        uint64_t e[3];
        index_off->push_back(o);
        o += index_dims((uint64_t)b->views[i].nx, (uint64_t)b->views[i].ny, (uint64_t)b->views[i].nz, e);
    }
    (void)descs_off;
    b->n_items = (uint32_t)tiles_total;
    *total = o;
    return VDBC_OK;
}

// The images of the split volumes from their pixel sums.
static vdbc_status batch_resolve(vdbc_batch* b, hipStream_t st)
{
    for (uint32_t i = 0; i < b->n; ++i) {
        if (!b->sums[i].rgbn) continue;
        const uint64_t npix = (uint64_t)b->cams[i].width * b->cams[i].height;
        hipLaunchKernelGGL(pt_resolve_kernel, dim3((unsigned)((npix + kBlock - 1) / kBlock)), dim3(kBlock), 0, st,
                           b->sums[i], b->images[i], nullptr, (uint32_t)npix, b->gs[i].spp);
        vdbc_status s = launch_check("batch pixel sums to image");
        if (s) return s;
    }
    return VDBC_OK;
}

static vdbc_status batch_enqueue(vdbc_batch* b, hipStream_t st)
{
    vdbc_status s;
    // the persistent launch builds every volume's majorant grid and coarse
    // bits in one launch each (below the grid-size limit); one launch per
    // volume otherwise, and for the per-volume baseline
    const bool batched_pre = b->t.persistent && b->mblocks_total < (1ull << 24) && b->cblocks_total < (1ull << 24) &&
                             b->iblocks_total < (1ull << 24);
    if (batched_pre) {
        hipLaunchKernelGGL(majorant_batch_kernel, dim3((unsigned)b->mblocks_total), dim3(kBlock), 0, st, b->d_descs,
                           b->d_cell_base, b->n);
        if ((s = launch_check("batched majorants"))) return s;
        hipLaunchKernelGGL(coarse_bits_batch_kernel, dim3((unsigned)b->cblocks_total), dim3(kBlock), 0, st,
                           b->d_descs, b->d_coarse_base, b->n);
        if ((s = launch_check("batched coarse occupancy"))) return s;
        if (b->indexed) {
            hipLaunchKernelGGL(index_batch_kernel, dim3((unsigned)b->iblocks_total), dim3(kBlock), 0, st, b->d_descs,
                               b->d_index_base, b->n, b->wide ? 2 : 0);
            if ((s = launch_check("batched region indexes"))) return s;
        }
    }
    for (uint32_t i = 0; i < b->n; ++i) {
        if (!batched_pre) {
            if ((s = launch_majorant(b->views[i], b->meds[i], (uint32_t)b->gs[i].C, b->majs[i], st)))
                return s;
            const PtArgs& g = b->gs[i];
            const uint64_t ncoarse = (uint64_t)g.cgx * g.cgy * g.cgz;
            hipLaunchKernelGGL(coarse_bits_kernel, dim3((unsigned)((ncoarse + kCoarsePerGroup - 1) / kCoarsePerGroup)), dim3(kBlock), 0,
                               st, b->majs[i], g, b->coarse[i]);
            if ((s = launch_check("batch coarse occupancy"))) return s;
            if (b->indexed && (s = launch_index(b->views[i], b->index[i], st))) return s;
        }
        if (b->sums[i].rgbn) {
            const uint64_t words = batch_sums_bytes((uint64_t)b->cams[i].width * b->cams[i].height) / 16;
            hipLaunchKernelGGL(pt_sums_clear_kernel,
                               dim3((unsigned)std::min<uint64_t>((words + kBlock - 1) / kBlock, 4096)), dim3(kBlock), 0,
                               st, reinterpret_cast<uint4*>(b->sums[i].rgbn), words);
            if ((s = launch_check("batch pixel sums clear"))) return s;
        }
    }
    if (b->t.persistent) {
        hipLaunchKernelGGL(zero_u32, dim3(1), dim3(64), 0, st, b->d_counter);
#define BATCH_LAUNCH(ACC, EN)                                                                                   \
    hipLaunchKernelGGL((pt_batch_kernel<ACC, EN>), dim3(b->grid_blocks), dim3(kBlock), 4u * (size_t)b->max_cwords, st, \
                       b->d_descs, b->d_items, b->n_items, b->d_counter)
#define BATCH_LAUNCH_ENV(ACC)          \
    if (b->env) BATCH_LAUNCH(ACC, true); \
    else BATCH_LAUNCH(ACC, false)
        if (b->indexed && b->wide) { BATCH_LAUNCH_ENV(IndexAccT<true>); }
        else if (b->indexed) { BATCH_LAUNCH_ENV(IndexAccT<false>); }
        else { BATCH_LAUNCH_ENV(VdbAcc); }
#undef BATCH_LAUNCH_ENV
#undef BATCH_LAUNCH
        if ((s = launch_check("batched render"))) return s;
        return batch_resolve(b, st);
    }
    // one launch per volume; the launches run in stream order, so they share
    // the tile queue, cleared before each
    for (uint32_t i = 0; i < b->n; ++i) {
        const PtArgs& g = b->gs[i];
        const uint32_t items = (uint32_t)(b->tiles_x[i] * b->tiles_y[i]) * g.chunks;
        hipLaunchKernelGGL(zero_u32, dim3(1), dim3(64), 0, st, b->d_counter);
        const dim3 grid(std::min<uint32_t>(items, (uint32_t)b->grid_blocks));
#define VOLUME_LAUNCH(ACC, VIEW, FIELD, EN)                                                                       \
    hipLaunchKernelGGL((pt_kernel<ACC, VIEW, false, false, EN>), grid, dim3(kBlock), 4u * (size_t)g.cwords, st, FIELD, \
                       b->cams[i], b->meds[i], g, b->majs[i], b->coarse[i], b->images[i], nullptr, nullptr,        \
                       b->d_counter, b->sums[i], nullptr)
#define VOLUME_LAUNCH_ENV(ACC, VIEW, FIELD)                  \
    if (b->meds[i].env) VOLUME_LAUNCH(ACC, VIEW, FIELD, true); \
    else VOLUME_LAUNCH(ACC, VIEW, FIELD, false)
        if (b->indexed && b->wide) { VOLUME_LAUNCH_ENV(IndexAccT<true>, IndexView, b->index[i].v); }
        else if (b->indexed) { VOLUME_LAUNCH_ENV(IndexAccT<false>, IndexView, b->index[i].v); }
        else { VOLUME_LAUNCH_ENV(VdbAcc, VdbView, b->views[i]); }
#undef VOLUME_LAUNCH_ENV
#undef VOLUME_LAUNCH
        if ((s = launch_check("per-volume render"))) return s;
    }
    return batch_resolve(b, st);
}

}  // namespace vdbc

extern "C" vdbc_status vdbc_batch_workspace(const vdbc_batch_item* items, uint32_t n, const vdbc_tuning* t,
                                            uint64_t* bytes)
{
    clear_error();
    if (!bytes) return fail(VDBC_E_INVALID, "null argument");
    vdbc_tuning tt;
    vdbc_status s = batch_tuning(t, &tt);
    if (s) return s;
    vdbc_batch b;
    std::vector<uint64_t> mo, co, so, xo;
    uint64_t io, total;
    if ((s = batch_plan(items, n, tt, &b, &mo, &co, &so, &xo, &io, &total))) return s;
    *bytes = total;
    return VDBC_OK;
}

extern "C" vdbc_status vdbc_batch_create(const vdbc_batch_item* items, uint32_t n, const vdbc_tuning* t, void* ws,
                                         uint64_t ws_bytes, void* stream, vdbc_batch** out)
{
    clear_error();
    if (!out || !ws) return fail(VDBC_E_INVALID, "null argument");
    if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(VDBC_E_INVALID, "workspace must be 256-byte aligned");
    *out = nullptr;
    vdbc_tuning tt;
    vdbc_status s = batch_tuning(t, &tt);
    if (s) return s;
    std::unique_ptr<vdbc_batch> b(new (std::nothrow) vdbc_batch());
    if (!b) return fail(VDBC_E_NOMEM, "no memory");
    std::vector<uint64_t> mo, co, so, xo;
    uint64_t io, total;
    if ((s = batch_plan(items, n, tt, b.get(), &mo, &co, &so, &xo, &io, &total))) return s;
    if (ws_bytes < total)
        return fail(VDBC_E_BUFFER_TOO_SMALL, "batch workspace needs %llu bytes", (unsigned long long)total);
    uint8_t* w = static_cast<uint8_t*>(ws);
    b->d_counter = reinterpret_cast<uint32_t*>(w);
    b->d_descs = reinterpret_cast<BatchDesc*>(w + 256);
    b->d_cell_base = reinterpret_cast<uint32_t*>(w + 256 + align256((uint64_t)n * sizeof(BatchDesc)));
    b->d_coarse_base = b->d_cell_base + (n + 1);
    b->d_index_base = b->d_coarse_base + (n + 1);
    b->d_items = reinterpret_cast<uint32_t*>(w + io);
    for (uint32_t i = 0; i < n; ++i) {
        b->majs.push_back(reinterpret_cast<float*>(w + mo[i]));
        b->coarse.push_back(reinterpret_cast<uint32_t*>(w + co[i]));
        b->sums.push_back(so[i] ? PtSums{reinterpret_cast<unsigned long long*>(w + so[i]), nullptr} : PtSums{});
    }
    // twice where the first pass meets a volume that needs wide entries
    b->index.resize(n);
    b->indexed = true;
    for (int pass = 0; pass < 2; ++pass)
        for (uint32_t i = 0; i < n && b->indexed; ++i) {
            b->indexed = make_index(&items[i].grid, b->views[i], reinterpret_cast<uint32_t*>(w + xo[i]), &b->index[i].v,
                                    &b->wide);
            b->index[i].wide = b->wide;
        }
    for (const MediumK& m : b->meds) b->env = b->env || m.env;
    // descriptors and the cost-ordered work list (largest estimated cost first:
    // samples per pixel x ray length through the volume)
    std::vector<BatchDesc> descs(n);
    std::vector<uint32_t> order(n);
    for (uint32_t i = 0; i < n; ++i) {
        descs[i] = BatchDesc{b->views[i], b->index[i].v, b->cams[i], b->meds[i], b->gs[i], b->majs[i], b->coarse[i], b->images[i],
                             b->sums[i], b->tiles_x[i]};
        order[i] = i;
    }
    auto cost = [&](uint32_t i) {
        return (double)b->gs[i].spp * (double)(b->views[i].nx + b->views[i].ny + b->views[i].nz);
    };
    std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t c) { return cost(a) > cost(c); });
    std::vector<uint32_t> list;
    list.reserve(b->n_items);
    for (uint32_t i : order)
        for (uint32_t k = 0; k < (uint32_t)(b->tiles_x[i] * b->tiles_y[i]) * b->gs[i].chunks; ++k)
            list.push_back((i << 20) | k);
    // prefix tables of the batched majorant launches: macrocells and
    // coarse-bit workgroups per volume (the launch is used only while both
    // totals stay below 2^24 workgroups)
    std::vector<uint32_t> bases(3 * (size_t)(n + 1), 0u);
    for (uint32_t i = 0; i < n; ++i) {
        const PtArgs& g = b->gs[i];
        b->mblocks_total += majorant_groups(g.C, (uint64_t)g.gx * g.gy * g.gz);
        b->cblocks_total += ((uint64_t)g.cgx * g.cgy * g.cgz + kCoarsePerGroup - 1) / kCoarsePerGroup;
        bases[i + 1] = (uint32_t)std::min<uint64_t>(b->mblocks_total, 0xFFFFFFFFull);
        bases[n + 1 + i + 1] = (uint32_t)std::min<uint64_t>(b->cblocks_total, 0xFFFFFFFFull);
        const IndexView& iv = b->index[i].v;
        if (b->indexed) b->iblocks_total += ((uint64_t)iv.tx * iv.ty * iv.tz + kBlock - 1) / kBlock;
        bases[2 * (n + 1) + i + 1] = (uint32_t)std::min<uint64_t>(b->iblocks_total, 0xFFFFFFFFull);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(b->d_cell_base, bases.data(), bases.size() * 4, hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(b->d_descs, descs.data(), n * sizeof(BatchDesc), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(b->d_items, list.data(), list.size() * 4, hipMemcpyHostToDevice, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return fail(VDBC_E_DEVICE, "batch descriptor upload: %s", hipGetErrorString(hipGetLastError()));
    b->grid_blocks = device_cus() * (int)tt.blocks_per_cu;
    *out = b.release();
    return VDBC_OK;
}

extern "C" vdbc_status vdbc_batch_launch(vdbc_batch* b, void* stream)
{
    clear_error();
    if (!b) return fail(VDBC_E_INVALID, "null batch");
    return batch_enqueue(b, static_cast<hipStream_t>(stream));
}

extern "C" vdbc_status vdbc_batch_capture(vdbc_batch* b, void* stream)
{
    clear_error();
    if (!b) return fail(VDBC_E_INVALID, "null batch");
    if (!stream) return fail(VDBC_E_INVALID, "capture needs a non-default stream");
    if (b->exec) return VDBC_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess)
        return fail(VDBC_E_DEVICE, "begin capture: %s", hipGetErrorString(hipGetLastError()));
    vdbc_status s = batch_enqueue(b, st);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(st, &g);
    if (s) {
        if (g) (void)hipGraphDestroy(g);
        return s;
    }
    if (e != hipSuccess || !g) return fail(VDBC_E_DEVICE, "end capture: %s", hipGetErrorString(e));
    hipGraphExec_t ex = nullptr;
    if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGraphDestroy(g);
        return fail(VDBC_E_DEVICE, "graph instantiate failed");
    }
    b->graph = g;
    b->exec = ex;
    return VDBC_OK;
}

extern "C" vdbc_status vdbc_batch_graph_launch(vdbc_batch* b, void* stream)
{
    clear_error();
    if (!b || !b->exec) return fail(VDBC_E_INVALID, "batch has no captured graph");
    if (hipGraphLaunch(b->exec, static_cast<hipStream_t>(stream)) != hipSuccess)
        return fail(VDBC_E_DEVICE, "graph launch: %s", hipGetErrorString(hipGetLastError()));
    return VDBC_OK;
}

extern "C" void vdbc_batch_destroy(vdbc_batch* b)
{
    if (!b) return;
    // teardown: nothing useful can be done with a failure here
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    delete b;
}
