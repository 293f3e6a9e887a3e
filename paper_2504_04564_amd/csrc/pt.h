// Device code of the delta-tracking path tracer (Section 4): majorant-grid
// DDA with coarse-block skipping, the per-tile path pool, the persistent
// single-volume kernel and the batched multi-volume kernel.
#pragma once
#include <type_traits>

#include "kcommon.h"

namespace vdbc {

// Resident PT workgroups per compute unit (the kernel's launch bounds): the
// tree accessor needs the registers of four, the others fit five (512^3 frame
// 5.52 ms with four, 5.22 with five; 994x676x1225 17.0 and 16.1).
template <class Acc>
constexpr int kPtBlocksPerCu = std::is_same_v<Acc, IndexAccT<false>> || std::is_same_v<Acc, IndexAccT<true>> ||
                                       std::is_same_v<Acc, DenseAcc> ? 5 : 4;
// Largest samples per pixel (256 x spp work units per tile fit 32 bits) and
// bounces per path (the bounce is a 16-bit field of the Philox counter).
constexpr uint32_t kMaxSpp = 1u << 16;
constexpr uint32_t kMaxBounces = 0xFFFFu;

// ---------------------------------------------------------------- PT

struct PtArgs {
    int spp, max_bounces, C, gx, gy, gz, tw, twl;   // tw pixels per wave row, twl = log2 tw
    float invC;
    int lf, cgx, cgy, cgz, cwords;   // coarse blocks of 2^lf macrocells per axis, bit words
    uint32_t seed_lo, seed_hi, frame;
    int rr;                          // Russian roulette from bounce 2 on
    uint32_t chunk, chunks;          // samples per work item, work items per tile
};

// Occupancy of the coarse blocks: bit set iff some macrocell of the block has
// a non-zero majorant.  Eight lanes per block, each an eighth of its macrocells;
// a wave's eight bits are one byte.  Latency: a thread per block walked its 64
// cells one load after the other, 11 us at 512^3 with cells of 16 (4 us so).
constexpr int kCoarsePerGroup = kBlock / 8;

// Workgroup `blk` of that launch (the whole workgroup calls it).
__device__ inline void coarse_bits_block(const float* __restrict__ maj, const PtArgs& g, uint32_t* __restrict__ bits,
                                         uint32_t blk)
{
    const int block = (int)blk * kCoarsePerGroup + (int)(threadIdx.x >> 3), part = (int)(threadIdx.x & 7);
    const int ncoarse = g.cgx * g.cgy * g.cgz;
    const int F = 1 << g.lf;
    bool occ = false;
    if (block < ncoarse) {
        const int x0 = block % g.cgx * F, y0 = (block / g.cgx) % g.cgy * F, z0 = block / (g.cgx * g.cgy) * F;
        const int x1 = min(x0 + F, g.gx), ny = min(F, g.gy - y0), rows = ny * min(F, g.gz - z0);
        for (int r = part; r < rows; r += 8) {
            const float* const row = maj + (int64_t)g.gx * (y0 + r % ny + (int64_t)g.gy * (z0 + r / ny));
            for (int x = x0; x < x1; ++x) occ |= row[x] > 0.0f;
        }
    }
    const uint64_t any = __ballot(occ);
    const int lane = threadIdx.x & 63;
    const int first = (int)blk * kCoarsePerGroup + (int)(threadIdx.x >> 6) * 8;   // of the wave's eight
    uint32_t byte = 0;
    for (int q = 0; q < 8; ++q) byte |= ((any >> (8 * q)) & 0xFFull) ? 1u << q : 0u;
    if (lane == 0 && first < 32 * g.cwords) reinterpret_cast<uint8_t*>(bits)[first >> 3] = (uint8_t)byte;
}

__global__ __launch_bounds__(kBlock) void coarse_bits_kernel(const float* __restrict__ maj,
                                                             PtArgs g, uint32_t* __restrict__ bits)
{
    coarse_bits_block(maj, g, bits, blockIdx.x);
}

// Random words of a lane's path segment: key (seed_lo ^ pixel, seed_hi),
// counter (block, sample, stream << 16 | bounce, frame); draw d is word d & 3 of
// block d >> 2, u = (x >> 8) * 2^-24.  Generated ahead of their use: a ring of
// two Philox blocks per lane in LDS, filled at one place of the path loop.  Philox at every draw
// site ran for a handful of lanes each time (11 % lane utilisation in the free
// flights, a third of the kernel's VALU instructions).
struct Stream {
    uint32_t* ring;    // this lane's word 0; words kBlock apart
    uint32_t tag;      // stream << 16 | bounce
    uint32_t d, made;  // words taken, words made
    __device__ __forceinline__ void start(uint32_t bounce, uint32_t stream)
    {
        tag = (stream << 16) | bounce;
        d = made = 0;
    }
    __device__ __forceinline__ void fill(uint32_t k0, uint32_t k1, uint32_t sample, uint32_t frame)
    {
        uint32_t w0 = made >> 2, w1 = sample, w2 = tag, w3 = frame;
        philox4x32_10(w0, w1, w2, w3, k0, k1);
        uint32_t* r = ring + (made & 4u) * kBlock;
        r[0] = w0;
        r[kBlock] = w1;
        r[2 * kBlock] = w2;
        r[3 * kBlock] = w3;
        made += 4u;
    }
    __device__ __forceinline__ float next()
    {
        const uint32_t x = ring[(d & 7u) * kBlock];
        ++d;
        return (float)(x >> 8) * (1.0f / 16777216.0f);
    }
};

// One ray segment being tracked through the majorant grid (Section 4): a 3D
// DDA over macrocells, hierarchical over coarse blocks of macrocells whose
// occupancy bits live in LDS, and delta tracking inside non-empty cells.
struct Flight {
    float o[3], d[3];
    // hardware reciprocal of d, +inf for d == +-0
    float id[3];
    // what the exit plane of a cell adds to C c along each axis: C - 1/2
    // (d > 0), -1/2 (d < 0) or +inf (d == 0: no crossing on this axis)
    float k[3];
    float t, t1, te, mu, imu;
    int c[3], axis;
    bool incell, ok;
    uint32_t budget;
};

// Starts a segment: clip to the box [-0.5, n-0.5]^3 (as box_clip, without
// branches) and find the first macrocell.
__device__ __forceinline__ void flight_begin(Flight& f, const PtArgs& g, int nx, int ny, int nz,
                                             const float o[3], const float d[3], float& t0)
{
    const float C = (float)g.C;
    const float hi[3] = {(float)nx - 0.5f, (float)ny - 0.5f, (float)nz - 0.5f};
    const float last[3] = {(float)(g.gx - 1), (float)(g.gy - 1), (float)(g.gz - 1)};
    float lo_t = -INFINITY, hi_t = INFINITY;
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool flat = d[a] == 0.0f;
        const float r = __builtin_amdgcn_rcpf(d[a]);   // hardware reciprocal (<= 1 ulp)
        const float ta = (-0.5f - o[a]) * r, tb = (hi[a] - o[a]) * r;
        const float mn = fminf(ta, tb), mx = fmaxf(ta, tb);
        lo_t = fmaxf(lo_t, flat ? -INFINITY : mn);
        hi_t = fminf(hi_t, flat ? INFINITY : mx);
        ok = ok && (!flat || !(o[a] < -0.5f || o[a] > hi[a]));
        const float k = d[a] > 0.0f ? C - 0.5f : -0.5f;
        f.k[a] = flat ? INFINITY : k;
        f.id[a] = flat ? INFINITY : r;
        f.o[a] = o[a];
        f.d[a] = d[a];
    }
    t0 = fmaxf(lo_t, 0.0f);
    f.t1 = hi_t;
    // a zero or non-finite direction leaves t1 infinite: no segment
    f.ok = ok && t0 < hi_t && hi_t <= 1.0e30f;
    f.incell = false;
    f.budget = kMaxFlightSamples;
    f.t = t0;
    // the macrocell edge is a power of two: multiplying by its reciprocal is exact
#pragma unroll
    for (int a = 0; a < 3; ++a)
        f.c[a] = (int)__builtin_amdgcn_fmed3f((fmaf(t0, d[a], o[a]) + 0.5f) * g.invC, 0.0f, last[a]);
}

__device__ __forceinline__ bool coarse_occupied(const uint32_t* bits, const PtArgs& g, int bx,
                                                int by, int bz)
{
    // at most 2^18 blocks: 24-bit products
    const uint32_t i = __umul24(__umul24((uint32_t)bz, (uint32_t)g.cgy) + (uint32_t)by, (uint32_t)g.cgx) + (uint32_t)bx;
    return (bits[i >> 5] >> (i & 31u)) & 1u;
}

// Exit distance through the faces of the axis-aligned cell of edge `edge` and
// index c, exit planes at edge c + k; returns the crossing axis or -1 if t1 is
// closer.  (edge c + k is exact, and a NaN loses every comparison.)
__device__ __forceinline__ int cell_exit(const Flight& f, float edge, const int c[3], const float k[3],
                                         float& te)
{
    float ta[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ta[a] = (fmaf(edge, (float)c[a], k[a]) - f.o[a]) * f.id[a];
    te = f.t1;
    int axis = -1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool nearer = ta[a] < te;
        te = nearer ? ta[a] : te;
        axis = nearer ? a : axis;
    }
    return axis;
}

// -log(x) = -ln 2 log2(x) for x in [2^-24, 1], with the hardware's log2.  ln 2 =
// 0x1.62e42fefa39ef...p-1 is split into its first 24 bits and the next 24, and the
// rounding of the head's product is recovered by an fma (Dekker's double-length
// product, Numer. Math. 18, 1971, in the form with one fma).  The last fma rounds
// once from the exact product, so the recovered part enters a second time, below
// half a unit of the last place; it stays because every image depends on the bits.
// On this range they are __logf's, whose care for denormals and infinities costs
// the kernel 4 to 11 % (512^3 frame 5.42 -> 5.62 ms, 994x676x1225 15.9 -> 17.9).
__device__ __forceinline__ float neg_log(float x)
{
    const float head = 0x1.62e42ep-1f, tail = 0x1.efa39ep-25f;
    const float y = __builtin_amdgcn_logf(x);
    const float e = fmaf(y, tail, fmaf(y, head, -(y * head)));
    return -fmaf(y, head, e);
}

// Advances the flight to its next tentative collision: returns 1 with f.t
// at the collision (the caller samples the density there and makes the
// accept test), 0 when the segment leaves the grid without one, or
// kFlightYield after entering `walk` <= kWalkCells macrocells without a
// collision (call again to continue; the walk and its random draws are the
// same as without the pause).  Takes at most walk + 1 draws from `rng`, walk
// when the flight is not inside a cell yet.  Empty cells draw no random
// numbers and coarse-block faces are macrocell faces, so the tentative
// collisions are those of a uniform walk over every macrocell; a flight that
// overshoots a cell restarts at its exit (memorylessness).
//
// Every lane of the wave takes the same kWalkCells + 1 turns (draw and step,
// then look the next cell up) under a flag instead of leaving the loop where
// its own walk ends: the flight's state then stays in place, where exits out
// of the middle cost some fifty register moves a turn.  The turns are unrolled
// (512^3 frame 5.55 -> 5.37 ms, 24-volume batch 4.02 -> 3.69).
__device__ __forceinline__ int flight_advance(Flight& f, const float* __restrict__ maj, const uint32_t* cbits,
                                              const PtArgs& g, Stream& rng, int walk, uint32_t& ncell)
{
    const float C = (float)g.C;
    const int F = 1 << g.lf;
    int result = f.ok ? kFlightYield : 0;
    bool run = f.ok;
#pragma unroll
    for (int turn = 0; turn <= kWalkCells; ++turn) {
        bool step = false;
        if (run && f.incell) {
            f.t = fmaf(neg_log(1.0f - rng.next()), f.imu, f.t);
            f.incell = f.t < f.te;
            step = !f.incell;
            if (f.incell) {
                run = false;
                result = --f.budget == 0 ? 0 : 1;
            }
        }
        if (step) {
            f.t = f.te;
#pragma unroll
            for (int a = 0; a < 3; ++a) f.c[a] += f.axis != a ? 0 : f.k[a] > 0.0f ? 1 : -1;
            if (f.axis < 0 || (unsigned)f.c[0] >= (unsigned)g.gx || (unsigned)f.c[1] >= (unsigned)g.gy ||
                (unsigned)f.c[2] >= (unsigned)g.gz) {
                run = false;
                result = 0;
            }
        }
        run = run && turn < walk;
        if (turn < kWalkCells && run) {
            ++ncell;
            const int b[3] = {f.c[0] >> g.lf, f.c[1] >> g.lf, f.c[2] >> g.lf};
            if (!coarse_occupied(cbits, g, b[0], b[1], b[2])) {
                // cross the empty block in one step
                const float CF = C * (float)F;
                float kf[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) kf[a] = f.k[a] > 0.0f ? f.k[a] + (CF - C) : f.k[a];
                const int axis = cell_exit(f, CF, b, kf, f.t);
                const int n[3] = {g.gx, g.gy, g.gz};
                bool out = axis < 0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float p = (fmaf(f.t, f.d[a], f.o[a]) + 0.5f) * g.invC;
                    const int lo = b[a] * F, hi = lo + F;
                    const int in = min(max((int)floorf(p), lo), min(hi, n[a]) - 1);
                    const int to = f.k[a] > 0.0f ? hi : lo - 1;
                    f.c[a] = axis == a ? to : in;
                    out = out || (unsigned)f.c[a] >= (unsigned)n[a];
                }
                if (out) {
                    run = false;
                    result = 0;
                }
            } else {
                f.axis = cell_exit(f, C, f.c, f.k, f.te);
                f.mu = maj[(uint32_t)f.c[0] + (uint32_t)g.gx * ((uint32_t)f.c[1] + (uint32_t)g.gy * (uint32_t)f.c[2])];
                f.incell = f.mu > 0.0f && f.t < f.te;
                f.imu = __builtin_amdgcn_rcpf(f.mu);   // hardware reciprocal (<= 1 ulp)
                if (!f.incell) {
                    // an empty cell inside an occupied block
                    f.t = f.te;
#pragma unroll
                    for (int a = 0; a < 3; ++a) f.c[a] += f.axis != a ? 0 : f.k[a] > 0.0f ? 1 : -1;
                    if (f.axis < 0 || (unsigned)f.c[0] >= (unsigned)g.gx || (unsigned)f.c[1] >= (unsigned)g.gy ||
                        (unsigned)f.c[2] >= (unsigned)g.gz) {
                        run = false;
                        result = 0;
                    }
                }
            }
        }
    }
    return result;
}

// LDS state of one 256-pixel tile: next unit of work and per-pixel sums in
// 2^-32 fixed point (integer sums do not depend on the order of the adds).
// Per-pixel fixed-point sums of a launch whose tiles are split into several
// work items: rgbn[4 pix + k] = red, green, blue (k < 3) and hits | escapes
// << 32 (k = 3); depth[pix] for the AOV.  rgbn == nullptr: every tile is one
// work item and writes its pixels itself.
struct PtSums {
    unsigned long long* rgbn;
    unsigned long long* depth;
};

struct TileShared {
    long long rgb[kBlock][3];
    long long depth[kBlock];
    unsigned int hits[kBlock], escapes[kBlock];
    uint32_t ring[8 * kBlock];   // random words ahead, two Philox blocks per lane
    unsigned int next;
};

__device__ __forceinline__ long long to_fixed(float v) { return __float2ll_rn(v * 4294967296.0f); }

// Bound by VALU issue (a wave instruction every four cycles of a SIMD, 90 % and
// more of the time) with a third of the lanes active: what counts is the number
// of instructions of a turn and the lanes that share them, not bytes.  512^3
// frame (1024^2, 16 samples) 12.2 -> 5.4 ms in this kernel, 994x676x1225 full HD
// with 64 samples 36 -> 15.5 ms, against a descent of the tree per lookup, Philox
// at each draw and a way out of the turn at each event.
// Delta-tracking path tracer (Section 4) over samples [s0, s1) of one tile of
// 256 pixels.  The work item's 256 (s1 - s0) paths (unit u = sample u / 256
// of tile pixel u % 256) are shared by the workgroup: every lane starts on one
// unit and takes the next one from an LDS counter when its path ends, so lanes
// on empty pixels or on short paths keep working.  Within a path the loop is flat: every iteration
// moves the lane to its next tentative collision and handles whatever event
// it reached (collision, escape, end of a shadow ray, start of a new path).
// The arithmetic and the random draws of each path are those of a recursive
// implementation: key (seed_lo ^ pixel, seed_hi), counter (block, sample,
// stream << 16 | bounce, frame).  Stream 0 of bounce b is path segment b:
// two draws for its direction (pixel jitter for b = 0, isotropic scattering
// otherwise), then its free flights and accept tests; stream 1 of bounce b is
// the shadow ray from collision b.  Results depend only on the pixel, not on
// the lane, tile shape or launch.
template <class Acc, bool AOV, bool ENV>
__device__ __forceinline__ void pt_tile(Acc& acc, int nx, int ny, int nz, const CameraK& cam,
                                        const MediumK& m, const PtArgs& g,
                                        const float* __restrict__ maj, const uint32_t* cbits,
                                        int bx, int by, TileShared& ts, const float4* tf_lds,
                                        float* __restrict__ image,
                                        float* __restrict__ aov, uint32_t& nsamp, uint32_t& ncell,
                                        uint32_t& nseg, uint32_t s0, uint32_t s1, PtSums sums)
{
    const int tid = threadIdx.x;
    // the four waves sit side by side in one band of 64 / tw rows: wave w covers
    // columns [x0 + w tw, x0 + (w + 1) tw), so the tile is 4 tw x 64 / tw pixels
    // (256 x 1 at tw = 64: neighbouring waves trace neighbouring rays)
    const int tl = g.twl;   // log2 tw
    const int x0 = bx << (tl + 2), y0 = by << (6 - tl);
    ts.rgb[tid][0] = ts.rgb[tid][1] = ts.rgb[tid][2] = 0;
    ts.depth[tid] = 0;
    ts.hits[tid] = ts.escapes[tid] = 0;
    if (tid == 0) ts.next = (s0 + 1) * kBlock;
    __syncthreads();
    const uint32_t total = kBlock * s1;
    const float inv4pi = 0.0795774715459476679f;
    uint32_t u = s0 * kBlock + (uint32_t)tid;
    uint32_t k0 = 0;
    float L0 = 0.0f, L1 = 0.0f, L2 = 0.0f, b0 = 1.0f, b1 = 1.0f, b2 = 1.0f;
    float t0p = 0.0f, pdepth = 1.0f;
    bool phit = false;
    int b = 0;
    enum { kFlying, kCamera, kShadow, kScatter };
    int begin = kCamera;      // the segment to begin, kFlying inside one
    bool shadow = false;
    Stream rng;
    rng.ring = ts.ring + tid;
    Flight f;
    while (u < total) {
        bool dead = false;   // the path ends here without a flight
        if (begin == kCamera) {
            const int q = (int)(u & (kBlock - 1)), l = q & 63;
            const int px = x0 + ((q >> 6) << tl) + (l & ((1 << tl) - 1)), py = y0 + (l >> tl);
            dead = px >= cam.width || py >= cam.height;   // no pixel here
            k0 = g.seed_lo ^ ((uint32_t)py * (uint32_t)cam.width + (uint32_t)px);
            rng.start(0u, 0u);
            b = 0;
            L0 = L1 = L2 = 0.0f;
            b0 = b1 = b2 = 1.0f;
        }
        // random words of this turn: at most four are taken below
        if (rng.made - rng.d < 4u) rng.fill(k0, g.seed_hi, u >> 8, g.frame);
        if (begin != kFlying) {
            float o[3] = {f.o[0], f.o[1], f.o[2]}, d[3];
            if (begin == kCamera) {
                const int q = (int)(u & (kBlock - 1)), l = q & 63;
                const int px = x0 + ((q >> 6) << tl) + (l & ((1 << tl) - 1)), py = y0 + (l >> tl);
                const float jx = rng.next(), jy = rng.next();
                camera_ray(cam, (float)px + jx, (float)py + jy, o, d);
            } else if (begin == kShadow) {
                d[0] = m.light[0];
                d[1] = m.light[1];
                d[2] = m.light[2];
            } else {
                // segment b: isotropic scattering from the collision point
                // (the shadow ray's origin) with the first two draws of its
                // stream; with Russian roulette one survival draw comes first
                // (from bounce 2 on: survive with q = min(1, max throughput),
                // survivors carry throughput / q)
                if (g.rr) {
                    const float ur = rng.next();
                    const float qs = b >= 2 ? fminf(fmaxf(fmaxf(b0, b1), b2), 1.0f) : 1.0f;
                    if (ur < qs) {
                        b0 /= qs;
                        b1 /= qs;
                        b2 /= qs;
                    } else {
                        dead = true;
                    }
                }
                const float u1 = rng.next(), u2 = rng.next();
                const float z = 1.0f - 2.0f * u1;
                const float r = sqrtf(fmaxf(0.0f, 1.0f - z * z));
                const float phi = 6.28318530717958647692f * u2;
                d[0] = r * __cosf(phi);
                d[1] = r * __sinf(phi);
                d[2] = z;
            }
            float t0;
            flight_begin(f, g, nx, ny, nz, o, d, t0);
            if (AOV && begin == kCamera) t0p = t0;
            if (!dead) ++nseg;
            begin = kFlying;
        }
        // No way out of the middle of a turn from here on: the path's state
        // stays in place under flags.  A turn takes at most walk + 1 draws in
        // flight (walk outside a cell) and one for the accept test.
        f.ok = f.ok && !dead;
        const int left = (int)(rng.made - rng.d) - (f.incell ? 2 : 1);
        const int tentative = flight_advance(f, maj, cbits, g, rng, min(kWalkCells, left), ncell);
        // the density at the tentative collision is taken here, after the walk
        // loop, so that the lanes of a wave that reached one in different
        // steps of the walk sample in one pass
        bool hit = false, path_done = dead;
        float sv = 0.0f;
        if (tentative == 1) {
            sv = trilinear(acc, fmaf(f.t, f.d[0], f.o[0]), fmaf(f.t, f.d[1], f.o[1]), fmaf(f.t, f.d[2], f.o[2]));
            ++nsamp;
            hit = rng.next() * f.mu < m.ds * tf_alpha_at(tf_lds, m, sv);   // else a null collision: keep tracking
        }
        if (!dead && (hit || tentative == 0)) {
            if (!shadow) {
                if (b == 0) {
                    phit = hit;
                    if (AOV) pdepth = hit ? (f.t - t0p) / (f.t1 - t0p) : 1.0f;
                }
                if (hit) {
                    // real collision: weight by albedo and colour, then the
                    // shadow ray towards the light from the collision point
                    const float4 c = tf_eval_at(tf_lds, m, sv);
                    b0 *= m.albedo * c.x;
                    b1 *= m.albedo * c.y;
                    b2 *= m.albedo * c.z;
#pragma unroll
                    for (int a = 0; a < 3; ++a) f.o[a] = fmaf(f.t, f.d[a], f.o[a]);
                    rng.start((uint32_t)b, 1u);
                    begin = kShadow;
                    shadow = true;
                } else {
                    float e0, e1, e2;
                    if (ENV) {   // the map's lookup only where a map is bound
                        escape_radiance(m, f.d, e0, e1, e2);
                    } else {
                        e0 = m.ambient[0];
                        e1 = m.ambient[1];
                        e2 = m.ambient[2];
                    }
                    L0 = fmaf(b0, e0, L0);
                    L1 = fmaf(b1, e1, L1);
                    L2 = fmaf(b2, e2, L2);
                    path_done = true;
                }
            } else {
                if (!hit) {
                    L0 = fmaf(b0 * inv4pi, m.light_E[0], L0);
                    L1 = fmaf(b1 * inv4pi, m.light_E[1], L1);
                    L2 = fmaf(b2 * inv4pi, m.light_E[2], L2);
                }
                shadow = false;
                if (b + 1 == g.max_bounces) {
                    path_done = true;
                } else {
                    ++b;
                    rng.start((uint32_t)b, 0u);
                    begin = kScatter;
                }
            }
        }
        if (path_done) {
            const int q = (int)(u & (kBlock - 1));
            atomicAdd(reinterpret_cast<unsigned long long*>(&ts.rgb[q][0]), (unsigned long long)to_fixed(L0));
            atomicAdd(reinterpret_cast<unsigned long long*>(&ts.rgb[q][1]), (unsigned long long)to_fixed(L1));
            atomicAdd(reinterpret_cast<unsigned long long*>(&ts.rgb[q][2]), (unsigned long long)to_fixed(L2));
            if (AOV) atomicAdd(reinterpret_cast<unsigned long long*>(&ts.depth[q]),
                               (unsigned long long)to_fixed(pdepth));
            atomicAdd(phit ? &ts.hits[q] : &ts.escapes[q], 1u);
            u = atomicAdd(&ts.next, 1u);
            begin = kCamera;
        }
    }
    __syncthreads();
    {
        const int w = tid >> 6, l = tid & 63;
        const int qx = x0 + (w << tl) + (l & ((1 << tl) - 1)), qy = y0 + (l >> tl);
        if (qx < cam.width && qy < cam.height) {
            const uint32_t pix = (uint32_t)qy * (uint32_t)cam.width + (uint32_t)qx;
            if (sums.rgbn) {
                // integer sums: the total does not depend on the order in
                // which the tile's work items finish
                unsigned long long* a = sums.rgbn + 4 * (size_t)pix;
                atomicAdd(a + 0, (unsigned long long)ts.rgb[tid][0]);
                atomicAdd(a + 1, (unsigned long long)ts.rgb[tid][1]);
                atomicAdd(a + 2, (unsigned long long)ts.rgb[tid][2]);
                atomicAdd(a + 3, (unsigned long long)ts.hits[tid] | ((unsigned long long)ts.escapes[tid] << 32));
                if (AOV) atomicAdd(sums.depth + pix, (unsigned long long)ts.depth[tid]);
            } else {
                const double sc = 1.0 / (4294967296.0 * (double)g.spp);
                const float inv = 1.0f / (float)g.spp;
                reinterpret_cast<float4*>(image)[pix] =
                    make_float4((float)((double)ts.rgb[tid][0] * sc), (float)((double)ts.rgb[tid][1] * sc),
                                (float)((double)ts.rgb[tid][2] * sc), (float)ts.hits[tid] * inv);
                if (AOV)
                    reinterpret_cast<float2*>(aov)[pix] =
                        make_float2((float)((double)ts.depth[tid] * sc), (float)ts.escapes[tid] * inv);
            }
        }
    }
    __syncthreads();
}

// Clears the per-pixel sums of a split launch: n 16-byte words.
__global__ void pt_sums_clear_kernel(uint4* __restrict__ p, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// The image (and AOV) of a split launch from its per-pixel sums, with the
// scaling of the tiles that write their pixels themselves.
__global__ void pt_resolve_kernel(PtSums sums, float* __restrict__ image, float* __restrict__ aov, uint32_t npix,
                                  int spp)
{
    const uint32_t pix = blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= npix) return;
    const unsigned long long* a = sums.rgbn + 4 * (size_t)pix;
    const ulonglong2 rg = *reinterpret_cast<const ulonglong2*>(a);
    const ulonglong2 bn = *reinterpret_cast<const ulonglong2*>(a + 2);
    const double sc = 1.0 / (4294967296.0 * (double)spp);
    const float inv = 1.0f / (float)spp;
    reinterpret_cast<float4*>(image)[pix] =
        make_float4((float)((double)(long long)rg.x * sc), (float)((double)(long long)rg.y * sc),
                    (float)((double)(long long)bn.x * sc), (float)(unsigned int)(bn.y & 0xFFFFFFFFull) * inv);
    if (aov)
        reinterpret_cast<float2*>(aov)[pix] =
            make_float2((float)((double)(long long)sums.depth[pix] * sc), (float)(unsigned int)(bn.y >> 32) * inv);
}

// ---------------------------------------------------------------- cost order
// Optional order of the tiles in the work queue: most expensive first, so
// that the longest work items do not start last.  The estimate of a tile is
// the majorant optical depth of four camera rays through it (one through the
// middle of each wave tile, 32 midpoint steps across the volume's box),
// binned on a log scale (four bins per octave of 1 + depth, 64 bins); a
// counting sort over the bins gives the order.  Ties within a bin are taken
// in whatever order the atomics give: the image does not depend on the order.
constexpr int kCostBins = 64;

// Sixteen lanes per tile, eight steps of one ray each (a thread per tile: 82 us
// for 8100 tiles, 32 workgroups of 128 loads one after the other).
constexpr uint32_t kCostLanes = 16;

__global__ __launch_bounds__(kBlock) void pt_tile_cost_kernel(CameraK cam, PtArgs g, int nx, int ny, int nz,
                                                              const float* __restrict__ maj, uint32_t tiles_x,
                                                              uint32_t tiles, uint32_t* __restrict__ key)
{
    const uint32_t t = blockIdx.x * (kBlock / kCostLanes) + threadIdx.x / kCostLanes;
    const int part = (int)(threadIdx.x % kCostLanes), w = part & 3, th = 64 / g.tw;
    if (t >= tiles) return;   // all lanes of a tile alike
    const float x0 = (float)((t % tiles_x) * 4u * (uint32_t)g.tw), y0 = (float)((t / tiles_x) * (uint32_t)th);
    float tau = 0.0f;
    float o[3], d[3], id[3], t0, t1;
    camera_ray(cam, x0 + ((float)w + 0.5f) * (float)g.tw, y0 + 0.5f * (float)th, o, d);
#pragma unroll
    for (int a = 0; a < 3; ++a) id[a] = 1.0f / d[a];
    if (box_clip(nx, ny, nz, o, d, id, t0, t1)) {
        const float dt = (t1 - t0) * (1.0f / 32.0f);
        float mu[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float s = fmaf((float)(4 * q + (part >> 2)) + 0.5f, dt, t0);
            const int cx = min(max((int)floorf((fmaf(s, d[0], o[0]) + 0.5f) * g.invC), 0), g.gx - 1);
            const int cy = min(max((int)floorf((fmaf(s, d[1], o[1]) + 0.5f) * g.invC), 0), g.gy - 1);
            const int cz = min(max((int)floorf((fmaf(s, d[2], o[2]) + 0.5f) * g.invC), 0), g.gz - 1);
            mu[q] = maj[cx + g.gx * (cy + g.gy * cz)];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) tau = fmaf(mu[q], dt, tau);
    }
#pragma unroll
    for (int q = 1; q < (int)kCostLanes; q *= 2) tau += __shfl_xor(tau, q);
    if (part) return;
    // fminf / fmaxf also map an infinite or NaN depth into the bin range
    const int k = (int)fmaxf(fminf(log2f(1.0f + fmaxf(tau, 0.0f)) * 4.0f, (float)(kCostBins - 1)), 0.0f);
    key[t] = (uint32_t)k;
}

// Places of the tiles in the queue, from the most expensive bin down: a counting
// sort by one workgroup, its counters in LDS (a global atomic per tile on the
// few bins in use took 80 us for 8100 tiles, twice).
__global__ __launch_bounds__(1024) void pt_cost_order_kernel(const uint32_t* __restrict__ key,
                                                             uint32_t* __restrict__ order, uint32_t tiles)
{
    static_assert(kCostBins == 64, "a lane per bin");
    __shared__ uint32_t bin[kCostBins];
    if (threadIdx.x < kCostBins) bin[threadIdx.x] = 0u;
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < tiles; t += blockDim.x) atomicAdd(&bin[key[t]], 1u);
    __syncthreads();
    if (threadIdx.x < kCostBins) {
        // first place of a bin: the tiles of the bins above it
        const uint32_t n = bin[threadIdx.x];
        uint32_t above = n;
#pragma unroll
        for (int q = 1; q < kCostBins; q *= 2) {
            const uint32_t up = __shfl_down(above, q);
            above += (int)threadIdx.x + q < kCostBins ? up : 0u;
        }
        bin[threadIdx.x] = above - n;
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < tiles; t += blockDim.x) order[atomicAdd(&bin[key[t]], 1u)] = t;
}

template <class Acc, class View, bool COUNT, bool AOV, bool ENV>
__global__ __launch_bounds__(kBlock, kPtBlocksPerCu<Acc>) void pt_kernel(View view, CameraK cam, MediumK m, PtArgs g,
                                                    const float* __restrict__ maj,
                                                    const uint32_t* __restrict__ coarse,
                                                    float* __restrict__ image,
                                                    float* __restrict__ aov,
                                                    unsigned long long* counter,
                                                    uint32_t* queue, PtSums sums,
                                                    const uint32_t* __restrict__ order)
{
    extern __shared__ uint32_t cbits[];
    __shared__ TileShared ts;
    for (int i = threadIdx.x; i < g.cwords; i += kBlock) cbits[i] = coarse[i];
    // the TF control points in LDS: every tentative collision reads two of them
    __shared__ float4 tf_lds[64];
    for (int i = threadIdx.x; i < m.tf_n; i += kBlock) tf_lds[i] = m.tf[i];
    __syncthreads();
    Acc acc{view};
    acc.reset();
    uint32_t nsamp = 0, ncell = 0, nseg = 0;
    // persistent workgroups take work items (tile, chunk of g.chunk samples)
    // from a queue, the tiles in raster order or in the given order, so a
    // workgroup that drew cheap items goes on to the next one at once, and
    // the paths of one expensive tile are spread over g.chunks workgroups
    __shared__ uint32_t s_item;
    const uint32_t tiles_x = (uint32_t)((cam.width + 4 * g.tw - 1) / (4 * g.tw));
    const uint32_t tiles = tiles_x * (uint32_t)((cam.height + 64 / g.tw - 1) / (64 / g.tw));
    const uint32_t items = tiles * g.chunks;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(queue, 1u);
        __syncthreads();
        const uint32_t it = s_item;   // pt_tile's barriers order this read before the next write
        if (it >= items) break;
        const uint32_t rank = it / g.chunks, s0 = (it % g.chunks) * g.chunk;
        const uint32_t t = order ? order[rank] : rank;
        pt_tile<Acc, AOV, ENV>(acc, view.nx, view.ny, view.nz, cam, m, g, maj, cbits, (int)(t % tiles_x),
                               (int)(t / tiles_x), ts, tf_lds, image, aov, nsamp, ncell, nseg, s0,
                               min(s0 + g.chunk, (uint32_t)g.spp), sums);
    }
    if (COUNT) {
        block_count(nsamp, counter);
        block_count(ncell, counter + 1);
        block_count(nseg, counter + 3);
    }
}

// ---------------------------------------------------------------- batched PT
// Many volumes in one persistent launch: workgroups pull (volume, work item)
// entries from an atomic counter over a list ordered by estimated cost
// (largest first) and render each item with the per-pixel code of pt_kernel,
// so every image is bit-identical to its own launch.  A volume's items are
// its tiles, or with g.chunks > 1 each tile's chunks of g.chunk samples
// (item = tile * g.chunks + chunk), which add into the volume's pixel sums.
struct BatchDesc {
    VdbView view;
    IndexView index;   // when the batch reads its volumes through their region indexes
    CameraK cam;
    MediumK med;
    PtArgs g;
    const float* maj;
    const uint32_t* coarse;
    float* image;
    PtSums sums;   // per-pixel integer sums when g.chunks > 1, else null
    int tiles_x;
};

__global__ void zero_u32(uint32_t* p)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0u;
}

template <class Acc, bool ENV>
__global__ __launch_bounds__(kBlock, kPtBlocksPerCu<Acc>) void pt_batch_kernel(const BatchDesc* __restrict__ descs,
                                                          const uint32_t* __restrict__ items,
                                                          uint32_t n_items, uint32_t* counter)
{
    extern __shared__ uint32_t cbits[];
    __shared__ uint32_t s_item;
    __shared__ TileShared ts;
    __shared__ float4 tf_lds[64];
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = atomicAdd(counter, 1u);
        __syncthreads();
        const uint32_t it = __builtin_amdgcn_readfirstlane(s_item);
        if (it >= n_items) break;
        const uint32_t code = __builtin_amdgcn_readfirstlane(items[it]);
        const BatchDesc* D = descs + (code >> 20);
        const PtArgs g = D->g;
        const uint32_t sub = code & 0xFFFFFu;
        const uint32_t tile = sub / g.chunks, s0 = (sub % g.chunks) * g.chunk;
        const CameraK cam = D->cam;
        for (int i = threadIdx.x; i < g.cwords; i += kBlock) cbits[i] = D->coarse[i];
        for (int i = threadIdx.x; i < D->med.tf_n; i += kBlock) tf_lds[i] = D->med.tf[i];
        __syncthreads();
        Acc acc;
        if constexpr (std::is_same_v<Acc, VdbAcc>) acc.v = D->view;
        else acc.v = D->index;
        acc.reset();
        uint32_t ns = 0, nc = 0, nsg = 0;
        pt_tile<Acc, false, ENV>(acc, D->view.nx, D->view.ny, D->view.nz, cam, D->med, g, D->maj, cbits,
                                 (int)(tile % (uint32_t)D->tiles_x), (int)(tile / (uint32_t)D->tiles_x), ts, tf_lds,
                                 D->image, nullptr, ns, nc, nsg, s0, min(s0 + g.chunk, (uint32_t)g.spp), D->sums);
    }
}

}  // namespace vdbc
