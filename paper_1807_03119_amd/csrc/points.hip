// Surface-point mode: the filter evaluated only at a list of voxels.  In the
// paper the filter runs at the first surface intersection point of each ray
// inside the renderer (Section "Our Method"; Results, Performance), so the
// work is a sparse gather rather than a dense stencil.
//
// Sixteen lanes per point (sixty-four in a short list, see launch_points_r), four
// neighbouring points of the list per wavefront (lane % 4, so that points beside
// each other, which share most of their rows, read the same cache lines in one
// instruction).  The nine clusters cover the
// (4r+1)^3 block around the point (coordinates clamped into the volume); the
// lanes split its (4r+1)^2 x-rows.  A row is read as the r * sizeof(T)
// + 1 aligned words that hold its 4r+1 voxels, for every alignment of a voxel,
// and shifted into place; rows that leave the volume in x, and uint16 volumes
// at an odd address, are read voxel by voxel.
// MEAN9 needs two weighted sums of a row, S = sum_rows c(dy) c(dz) sum_x c(dx) v
// + sum_{|dy|,|dz| <= r} sum_{|dx| <= r} v with c = 1, and 2 at 0: integer dot
// products of the packed words with constant weights.  MINVAR9 sums each row
// (and its squares) over the left, right and centre ranges of the clusters,
// which go to the corner clusters whose y- and z-ranges hold the row and, when
// |dy|, |dz| <= r, to the centre cluster.  The lanes' sums are combined with
// cross-lane shuffles; one lane applies the rule, rounding and gate.
//
// What bounds it: the rows' cache-line requests (169 rows a point at r = 3).
// One wavefront per point with 13 two-byte loads a row took 925 us for the
// 262144 rays of a 512^3 uint16 volume (r = 3, MEAN9); this takes 179 (MINVAR9
// 969 and 222).  Scattered points are bound by their cache misses (2^20 of 512 x
// 512 x 256 uint16, r = 1..4: 454 -> 473, 1516 -> 1558, 3960 -> 3470, 12480 -> 6160).
//
// The first-hit pass produces that point list for rays parallel to z: per
// pixel (x, y), the first voxel of the column, in the ray's direction, whose
// value reaches the threshold (the surface, Otsu's T in the paper).  One lane
// per ray, 64 neighbouring x per wavefront, so every slice step of a
// wavefront reads one contiguous row segment; each step issues kHitStep
// independent slice loads before testing them, to keep enough reads in
// flight for HBM.  A lane stops at its hit (its loads are masked off from
// then on) and the wavefront at its deepest hit, so the bytes read are the
// columns up to their hits.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "lnf.h"
#include "lnf_ctx.h"
#include "lnf_internal.h"

namespace lnf {
namespace {

constexpr int kPointThreads = 256;

// Sum over the LANES lanes of a point (the upper lane bits).
template <int LANES, typename V>
__device__ __forceinline__ V point_sum(V v)
{
#pragma unroll
    for (int off = 64 / LANES; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The weights of word a of a row's packed voxels: MEAN9's c(dx) (BOX: 1 for
// |dx| <= r), 0 past the row.
template <int R, typename T, bool BOX>
constexpr uint32_t row_weights(int a)
{
    constexpr int kPer = 4 / (int)sizeof(T);
    uint32_t w = 0;
    for (int b = 0; b < kPer; ++b) {
        const int dx = a * kPer + b - 2 * R;
        uint32_t c = dx > 2 * R ? 0u : dx == 0 ? 2u : 1u;
        if (BOX) c = dx >= -R && dx <= R ? 1u : 0u;
        w |= c << (8 * (int)sizeof(T) * b);
    }
    return w;
}

template <int R, typename T, int RULE, int LANES>
__global__ __launch_bounds__(kPointThreads) void filter_points_kernel(
    const T* __restrict__ in, Geom g, const int32_t* __restrict__ xyz, int64_t n, uint32_t gate,
    uint32_t* __restrict__ out)
{
    constexpr int M = 2 * R + 1, NB = M * M * M;
    constexpr int W = 4 * R + 1, NROW = W * W;  // side and x-rows of the nine clusters' block
    constexpr int ND = R * (int)sizeof(T) + 1;  // aligned words that hold a row
    constexpr int kPer = 4 / (int)sizeof(T);
    constexpr bool VAR = RULE == LNF_MINVAR9;
    // squares: uint32 holds a cluster's for uint8 (729 * 255^2), fp64 for uint16
    using Q = std::conditional_t<sizeof(T) == 1, uint32_t, double>;
    constexpr int kWave = 64 / LANES;  // points of a wavefront
    const int lane = threadIdx.x & 63, sub = lane / kWave;
    const int64_t pi = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * (kPointThreads / LANES) +
                       (threadIdx.x >> 6) * kWave + lane % kWave;
    const int64_t p = pi < n ? pi : n - 1;  // lanes past the list redo its last point
    int px = xyz[3 * p], py = xyz[3 * p + 1], pz = xyz[3 * p + 2];
    const bool inside = px >= 0 && py >= 0 && pz >= 0 && px < g.nx && py < g.ny && pz < g.nz;
    if (!inside) px = py = pz = 0;
    const size_t nx = g.nx, plane = (size_t)g.nx * g.ny;
    // rows inside the volume in x; a uint16 row that starts at an odd byte could
    // end a byte past its words
    const bool whole = px >= 2 * R && px + 2 * R < g.nx &&
                       reinterpret_cast<uintptr_t>(in) % sizeof(T) == 0;

    uint32_t s[9];
    Q q[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        s[k] = 0;
        q[k] = 0;
    }
    int dy = sub % W - 2 * R, dz = sub / W - 2 * R;
    // points outside the volume read nothing
    for (int row = inside ? sub : NROW; row < NROW; row += LANES) {
        const int y = clampi(py + dy, 0, g.ny - 1), z = clampi(pz + dz, 0, g.nz - 1);
        const T* rp = in + (size_t)z * plane + (size_t)y * nx;
        uint32_t w[ND];  // packed voxels from px - 2R on
        if (whole) {
            const uintptr_t at = reinterpret_cast<uintptr_t>(rp + (px - 2 * R));
            const uint32_t* wp = reinterpret_cast<const uint32_t*>(at & ~(uintptr_t)3);
#pragma unroll
            for (int a = 0; a < ND; ++a) w[a] = wp[a];
#pragma unroll
            for (int a = 0; a < ND; ++a)
                w[a] = __builtin_amdgcn_alignbyte(a + 1 < ND ? w[a + 1] : 0u, w[a], (uint32_t)at);
        } else {
#pragma unroll
            for (int a = 0; a < ND; ++a) {
                w[a] = 0;
#pragma unroll
                for (int b = 0; b < kPer; ++b)
                    if (a * kPer + b < W)
                        w[a] |= (uint32_t)rp[clampi(px - 2 * R + a * kPer + b, 0, g.nx - 1)]
                                << (8 * (int)sizeof(T) * b);
            }
        }
        const bool inc = dy >= -R && dy <= R && dz >= -R && dz <= R;
        if constexpr (!VAR) {
            uint32_t c = 0, box = 0;
#pragma unroll
            for (int a = 0; a < ND; ++a) {
                if constexpr (sizeof(T) == 2) {
                    using u16x2 = unsigned short __attribute__((ext_vector_type(2)));
                    const u16x2 v = __builtin_bit_cast(u16x2, w[a]);
                    c = __builtin_amdgcn_udot2(v, __builtin_bit_cast(u16x2, row_weights<R, T, false>(a)), c, false);
                    box = __builtin_amdgcn_udot2(v, __builtin_bit_cast(u16x2, row_weights<R, T, true>(a)), box, false);
                } else {
                    c = __builtin_amdgcn_udot4(w[a], row_weights<R, T, false>(a), c, false);
                    box = __builtin_amdgcn_udot4(w[a], row_weights<R, T, true>(a), box, false);
                }
            }
            s[0] += (c << ((dy == 0) + (dz == 0))) + (inc ? box : 0u);
        } else {
            // sums over [0, R), [R, 2R), 2R, (2R, 3R], (3R, 4R]: the three
            // ranges are made of them
            uint32_t t[5] = {0, 0, 0, 0, 0};
            Q u[5] = {0, 0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const uint32_t v = (w[i / kPer] >> (8 * (int)sizeof(T) * (i % kPer))) &
                                   ((1u << (8 * (int)sizeof(T))) - 1u);
                const int k = i < R ? 0 : i < 2 * R ? 1 : i == 2 * R ? 2 : i <= 3 * R ? 3 : 4;
                t[k] += v;
                u[k] += (Q)(v * v);  // exact: below 2^32
            }
            const uint32_t centre = t[1] + t[2] + t[3];
            const Q qc = u[1] + u[2] + u[3];
            const uint32_t side[2] = {t[0] + t[1] + t[2], t[2] + t[3] + t[4]};
            const Q qside[2] = {u[0] + u[1] + u[2], u[2] + u[3] + u[4]};
            s[0] += inc ? centre : 0u;
            q[0] += inc ? qc : (Q)0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {  // cluster j + 1: x, y, z side by bits 0, 1, 2
                const bool in_yz = ((j & 2) ? dy >= 0 : dy <= 0) && ((j & 4) ? dz >= 0 : dz <= 0);
                s[j + 1] += in_yz ? side[j & 1] : 0u;
                q[j + 1] += in_yz ? qside[j & 1] : (Q)0;
            }
        }
        // the row LANES further on
        dy += LANES % W;
        dz += LANES / W;
        if (dy > 2 * R) {
            dy -= W;
            dz += 1;
        }
    }
    uint32_t o;
    if constexpr (!VAR) {
        o = round_div_odd(point_sum<LANES>(s[0]), 1.0 / (9.0 * NB));
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            s[k] = point_sum<LANES>(s[k]);
            q[k] = point_sum<LANES>(q[k]);
        }
        uint32_t best_s = s[0];
        double best_v = __builtin_fma((double)NB, (double)q[0], -(double)s[0] * (double)s[0]);
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            const double v = __builtin_fma((double)NB, (double)q[k], -(double)s[k] * (double)s[k]);
            if (v < best_v) {
                best_v = v;
                best_s = s[k];
            }
        }
        o = round_div_odd(best_s, 1.0 / NB);
    }
    if (sub != 0 || pi >= n) return;
    if (o < gate) o = 0;
    out[p] = inside ? o : 0xffffffffu;  // point outside the volume
}

// slices loaded per step of a ray (512^3 uint16, mean depth 49: 43 us with 8, 37 with 16)
constexpr int kHitStep = 16;
constexpr int kHitRows = 4;     // wavefronts (pixel rows) per workgroup

template <typename T, bool BACK>
__global__ __launch_bounds__(64 * kHitRows) void first_hit_kernel(const T* __restrict__ in,
                                                                  Geom g, uint32_t thr,
                                                                  int tiles_x,
                                                                  int32_t* __restrict__ xyz)
{
    const int bx = blockIdx.x % tiles_x, by = blockIdx.x / tiles_x;
    const int x = bx * 64 + (threadIdx.x & 63);
    const int y = by * kHitRows + (threadIdx.x >> 6);
    if (x >= g.nx || y >= g.ny) return;
    const size_t plane = (size_t)g.nx * g.ny;
    const T* col = in + (size_t)y * g.nx + x;
    int hit = -1;  // steps from the ray's first slice
    for (int s0 = 0; s0 < g.nz; s0 += kHitStep) {
        uint32_t v[kHitStep];
#pragma unroll
        for (int k = 0; k < kHitStep; ++k) {
            const int s = s0 + k;
            const int z = BACK ? g.nz - 1 - s : s;
            v[k] = s < g.nz ? (uint32_t)col[(size_t)z * plane] : 0u;
        }
#pragma unroll
        for (int k = kHitStep - 1; k >= 0; --k)  // the first qualifying step wins
            if (s0 + k < g.nz && v[k] >= thr) hit = s0 + k;
        if (hit >= 0) break;
    }
    int32_t* o = xyz + 3 * ((size_t)y * g.nx + x);
    o[0] = x;
    o[1] = y;
    o[2] = hit < 0 ? -1 : (BACK ? g.nz - 1 - hit : hit);
}

template <typename T>
hipError_t launch_first_hit(const void* vol, Geom g, uint32_t thr, int direction, int32_t* xyz,
                            hipStream_t s)
{
    const int tiles_x = (g.nx + 63) / 64;
    const long long blocks = (long long)tiles_x * ((g.ny + kHitRows - 1) / kHitRows);
    const dim3 grid((unsigned)blocks), block(64 * kHitRows);
    const T* in = static_cast<const T*>(vol);
    if (direction > 0)
        hipLaunchKernelGGL((first_hit_kernel<T, false>), grid, block, 0, s, in, g, thr, tiles_x,
                           xyz);
    else
        hipLaunchKernelGGL((first_hit_kernel<T, true>), grid, block, 0, s, in, g, thr, tiles_x,
                           xyz);
    return hipGetLastError();
}

template <int R, typename T, int LANES>
hipError_t launch_points_lanes(int rule, const void* vol, Geom g, const int32_t* xyz, int64_t n,
                               uint32_t gate, uint32_t* out, hipStream_t s)
{
    constexpr int kGroup = kPointThreads / LANES;
    const dim3 grid((unsigned)((n + kGroup - 1) / kGroup)), block(kPointThreads);
    const T* in = static_cast<const T*>(vol);
    if (rule == LNF_MEAN9)
        hipLaunchKernelGGL((filter_points_kernel<R, T, LNF_MEAN9, LANES>), grid, block, 0, s, in, g,
                           xyz, n, gate, out);
    else
        hipLaunchKernelGGL((filter_points_kernel<R, T, LNF_MINVAR9, LANES>), grid, block, 0, s, in, g,
                           xyz, n, gate, out);
    return hipGetLastError();
}

// Sixteen lanes a point, but a wavefront for lists of up to two points a SIMD from
// r = 2: they leave the chip idle, and a point's rows are one chain for its lanes
// (1024 scattered points of uint16, sixteen lanes against sixty-four: r = 2 4.9 and
// 3.3 us, r = 4 21.2 and 9.3; 4096 rays' hits side by side, r = 4: 22.1 and 35.5).
template <int R, typename T>
hipError_t launch_points_r(int rule, const void* vol, Geom g, const int32_t* xyz, int64_t n,
                           uint32_t gate, uint32_t* out, hipStream_t s)
{
    if (R >= 2 && n <= 8 * device_cus()) return launch_points_lanes<R, T, 64>(rule, vol, g, xyz, n, gate, out, s);
    return launch_points_lanes<R, T, 16>(rule, vol, g, xyz, n, gate, out, s);
}

template <typename T>
hipError_t launch_points(int rule, int r, const void* vol, Geom g, const int32_t* xyz, int64_t n,
                         uint32_t gate, uint32_t* out, hipStream_t s)
{
    switch (r) {
    case 1: return launch_points_r<1, T>(rule, vol, g, xyz, n, gate, out, s);
    case 2: return launch_points_r<2, T>(rule, vol, g, xyz, n, gate, out, s);
    case 3: return launch_points_r<3, T>(rule, vol, g, xyz, n, gate, out, s);
    default: return launch_points_r<4, T>(rule, vol, g, xyz, n, gate, out, s);
    }
}

}  // namespace
}  // namespace lnf

using namespace lnf;

namespace {

// Checks shared by the first-hit entry points: the volume and a hit list of
// nx * ny entries on the context's device.
int check_first_hit(lnf_handle h, const void* vol, const int64_t dims[3], int dtype,
                    int direction, const int32_t* xyz, Geom* g)
{
    if (!h || !vol || !dims || !xyz) return LNF_EINVAL;
    if (dtype != LNF_U8 && dtype != LNF_U16) return LNF_EINVAL;
    if (direction != 1 && direction != -1) return LNF_EINVAL;
    for (int i = 0; i < 3; ++i)
        if (dims[i] < 1 || dims[i] > INT32_MAX) return LNF_EINVAL;
    if (dims[0] * dims[1] > INT32_MAX) return LNF_EINVAL;
    *g = Geom{(int)dims[0], (int)dims[1], (int)dims[2]};
    const size_t bytes = (size_t)dims[0] * dims[1] * dims[2] * (dtype == LNF_U8 ? 1 : 2);
    int rc;
    if ((rc = check_device_range(vol, bytes, h->device))) return rc;
    return check_device_range(xyz, (size_t)dims[0] * dims[1] * 3 * sizeof(int32_t), h->device);
}

}  // namespace

extern "C" int lnf_first_hit(lnf_handle h, const void* vol, const int64_t dims[3], int dtype,
                             uint32_t threshold, int direction, int32_t* xyz, hipStream_t stream)
{
    if (!h) return LNF_EINVAL;
    DeviceGuard dg(h->device);
    if (!dg.ok()) return LNF_EHIP;
    Geom g;
    const int rc = check_first_hit(h, vol, dims, dtype, direction, xyz, &g);
    if (rc) return rc;
    const hipError_t e = dtype == LNF_U8
                             ? launch_first_hit<uint8_t>(vol, g, threshold, direction, xyz, stream)
                             : launch_first_hit<uint16_t>(vol, g, threshold, direction, xyz, stream);
    return e == hipSuccess ? LNF_OK : LNF_EHIP;
}

extern "C" int lnf_filter_surface(lnf_handle h, const void* vol, const int64_t dims[3], int dtype,
                                  int radius, uint32_t threshold, int direction, int32_t* xyz,
                                  uint32_t* out, hipStream_t stream)
{
    if (!h || !out) return LNF_EINVAL;
    if (h->geom) return LNF_EINVAL;  // default cluster geometry only, as lnf_filter_points
    if (radius < 1 || radius > LNF_RADIUS_MAX) return LNF_EINVAL;
    DeviceGuard dg(h->device);
    if (!dg.ok()) return LNF_EHIP;
    Geom g;
    int rc = check_first_hit(h, vol, dims, dtype, direction, xyz, &g);
    if (rc) return rc;
    const int64_t n = dims[0] * dims[1];
    if ((rc = check_device_range(out, (size_t)n * sizeof(uint32_t), h->device))) return rc;
    if ((rc = lnf_first_hit(h, vol, dims, dtype, threshold, direction, xyz, stream))) return rc;
    return lnf_filter_points(h, vol, dims, dtype, radius, xyz, n, out, stream);
}

extern "C" int lnf_filter_points(lnf_handle h, const void* vol, const int64_t dims[3], int dtype,
                                 int radius, const int32_t* xyz, int64_t n, uint32_t* out,
                                 hipStream_t stream)
{
    if (!h || !vol || !dims || n < 0 || (n > 0 && (!xyz || !out))) return LNF_EINVAL;
    if (h->geom) return LNF_EINVAL;  // default cluster geometry only
    if (dtype != LNF_U8 && dtype != LNF_U16) return LNF_EINVAL;
    if (radius < 1 || radius > LNF_RADIUS_MAX) return LNF_EINVAL;
    for (int i = 0; i < 3; ++i)
        if (dims[i] < 1 || dims[i] > INT32_MAX) return LNF_EINVAL;
    if (dims[0] * dims[1] > INT32_MAX) return LNF_EINVAL;
    if (n > (int64_t)INT32_MAX * 4) return LNF_EINVAL;
    if (n == 0) return LNF_OK;
    const Geom g{(int)dims[0], (int)dims[1], (int)dims[2]};
    const size_t bytes = (size_t)dims[0] * dims[1] * dims[2] * (dtype == LNF_U8 ? 1 : 2);
    DeviceGuard dg(h->device);
    if (!dg.ok()) return LNF_EHIP;
    int rc;
    if ((rc = check_device_range(vol, bytes, h->device))) return rc;
    if ((rc = check_device_range(xyz, (size_t)n * 3 * sizeof(int32_t), h->device))) return rc;
    if ((rc = check_device_range(out, (size_t)n * sizeof(uint32_t), h->device))) return rc;
    const hipError_t e =
        dtype == LNF_U8
            ? launch_points<uint8_t>(h->rule, radius, vol, g, xyz, n, h->gate, out, stream)
            : launch_points<uint16_t>(h->rule, radius, vol, g, xyz, n, h->gate, out, stream);
    return e == hipSuccess ? LNF_OK : LNF_EHIP;
}
