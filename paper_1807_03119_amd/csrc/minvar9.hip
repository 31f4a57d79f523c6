// MINVAR9 single-volume kernel: a thin wrapper around the tile body of
// plane_tile.h (least-variance selection among the nine clusters).
#include "device_common.h"
#include "lnf_internal.h"
#include "plane_tile.h"

namespace lnf {
namespace {

template <int R, typename T, bool GATE, bool WT>
__global__ __launch_bounds__((MV9Shape<R, WT>::THREADS))
__attribute__((amdgpu_waves_per_eu(MV9Shape<R, WT>::WAVES))) void minvar9_planes(
    const T* __restrict__ in, T* __restrict__ out, Geom g, int zs, int tiles_x, int tiles_y,
    int total, uint32_t gate, double dn, double invn, const uint32_t* __restrict__ gate_dev)
{
    if (GATE && gate_dev) gate = *gate_dev;  // a threshold found on the device
    using S = MV9Shape<R, WT>;
    __shared__ __align__(16) MV9Lds<R, T, WT> sm;
    const int tile = xcd_tile(blockIdx.x, total);
    const int bx = tile % tiles_x;
    const int rest = tile / tiles_x;
    const int by = rest % tiles_y;
    const int bz = rest / tiles_y;
    const int z0 = bz * zs;
    minvar9_tile<R, T, GATE, WT>(sm, in, out, g, bx * S::TX, by * S::TY, z0, min(z0 + zs, g.nz),
                                 gate, dn, invn, (int)threadIdx.x);
}

template <int R, typename T, bool WT>
hipError_t launch_planes(const void* in, void* out, Geom g, uint32_t gate, int zs, hipStream_t s,
                         TileCfg* plan, const uint32_t* gate_dev)
{
    using S = MV9Shape<R, WT>;
    const int tiles_x = (g.nx + S::TX - 1) / S::TX, tiles_y = (g.ny + S::TY - 1) / S::TY;
    if (zs <= 0)
        zs = default_zs(tiles_x * tiles_y, g.nz,
                        resident_groups((const void*)minvar9_planes<R, T, false, WT>, S::THREADS));
    if (plan) {
        plan->zs = zs;
        return hipSuccess;
    }
    const int nzs = (g.nz + zs - 1) / zs;
    const int total = tiles_x * tiles_y * nzs;
    const int n = (2 * R + 1) * (2 * R + 1) * (2 * R + 1);
    const T* pin = static_cast<const T*>(in);
    T* pout = static_cast<T*>(out);
    if (gate || gate_dev)
        hipLaunchKernelGGL((minvar9_planes<R, T, true, WT>), dim3(total), dim3(S::THREADS), 0, s,
                           pin, pout, g, zs, tiles_x, tiles_y, total, gate, (double)n, 1.0 / n, gate_dev);
    else
        hipLaunchKernelGGL((minvar9_planes<R, T, false, WT>), dim3(total), dim3(S::THREADS), 0, s,
                           pin, pout, g, zs, tiles_x, tiles_y, total, gate, (double)n, 1.0 / n, gate_dev);
    return hipGetLastError();
}

template <int R, typename T>
hipError_t launch_variant(int variant, const void* in, void* out, Geom g, uint32_t gate, int zs,
                          hipStream_t s, TileCfg* plan, const uint32_t* gate_dev)
{
    if (variant == 1) return launch_planes<R, T, true>(in, out, g, gate, zs, s, plan, gate_dev);
    return launch_planes<R, T, false>(in, out, g, gate, zs, s, plan, gate_dev);
}

// Estimated time of a launch, in rounds of the workgroups that the CUs hold at
// once x slices: a round that is not full still takes 0.4 of a full one, and a
// strip 8 slices more than its depth.  `round`: a full round of this tile, of
// the narrow tile's.
template <int R, typename T, bool WT>
double planes_cost(Geom g, double round)
{
    using S = MV9Shape<R, WT>;
    const int tiles = ((g.nx + S::TX - 1) / S::TX) * ((g.ny + S::TY - 1) / S::TY);
    const int resident = resident_groups((const void*)minvar9_planes<R, T, false, WT>, S::THREADS);
    const int zs = default_zs(tiles, g.nz, resident), cus = device_cus(), per_cu = resident / cus;
    const long long groups = (long long)tiles * ((g.nz + zs - 1) / zs);
    const long long n = (groups + cus - 1) / cus, rest = n % per_cu;
    return ((double)(n / per_cu) + (rest ? 0.4 + 0.6 * (double)rest / per_cu : 0.0)) * (zs + 8) * round;
}

// The tile with the least estimated time.  A full round of wide tiles (2 to 4 on a
// CU) takes 0.92 to 1.06 of one of narrow tiles (4 to 7), for the same outputs
// from r = 2, so what decides is how well either fills its rounds and the rows: of
// 740 random volumes the choice is on average within 0.2 % of the faster tile
// (0.5 % of those above 9 * 10^7 voxels); wide from 256 x 256 on was 2 to 4 % off
// (uint8 r = 2, 391 x 585 x 251: 171 and 210 us, 716 x 370 x 31 41 and 49; r = 3,
// 512^3: 362 and 353).
template <typename T>
int faster_variant(int r, Geom g)
{
    switch (r) {
    case 1: return planes_cost<1, T, true>(g, sizeof(T) == 1 ? 1.04 : 1.06) < planes_cost<1, T, false>(g, 1.0);
    case 2: return planes_cost<2, T, true>(g, 0.96) < planes_cost<2, T, false>(g, 1.0);
    case 3: return planes_cost<3, T, true>(g, 0.92) < planes_cost<3, T, false>(g, 1.0);
    default: return 0;  // one shape
    }
}

template <typename T>
hipError_t dispatch_r(const void* in, void* out, int r, Geom g, uint32_t gate, TileCfg cfg,
                      hipStream_t s, TileCfg* plan, const uint32_t* gate_dev)
{
    const int v = cfg.variant >= 0 ? cfg.variant : faster_variant<T>(r, g);
    if (plan) plan->variant = v;
    switch (r) {
    case 1: return launch_variant<1, T>(v, in, out, g, gate, cfg.zs, s, plan, gate_dev);
    case 2: return launch_variant<2, T>(v, in, out, g, gate, cfg.zs, s, plan, gate_dev);
    case 3: return launch_variant<3, T>(v, in, out, g, gate, cfg.zs, s, plan, gate_dev);
    case 4: return launch_variant<4, T>(v, in, out, g, gate, cfg.zs, s, plan, gate_dev);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// 0: 32 x 16 outputs, 256 threads; 1: 64 x 16 outputs, 512 threads (up to
// r = 3; the same tile as 0 at r = 4)
int minvar9_variants() { return 2; }

// In the launch of a batch the narrow tile is the faster up to r = 2 (60 random
// classes of 1 to 24 volumes: the wide one 3 to 28 % slower, 10 % on average);
// at r = 3 they are within a few percent, the wide one ahead where volumes are
// large (24 of 256 to 400, uint16: 3350 and 3184 us).
int minvar9_batch_variant(int r, Geom g) { return r == 3 && g.nx >= 256 && g.ny >= 256 ? 1 : 0; }

void minvar9_tile_shape(int variant, int r, int* tx, int* ty)
{
    const bool w = variant == 1;
    switch (r) {
    case 1: *tx = w ? MV9Shape<1, true>::TX : MV9Shape<1>::TX; *ty = MV9Shape<1>::TY; return;
    case 2: *tx = w ? MV9Shape<2, true>::TX : MV9Shape<2>::TX; *ty = MV9Shape<2>::TY; return;
    case 3: *tx = w ? MV9Shape<3, true>::TX : MV9Shape<3>::TX; *ty = MV9Shape<3>::TY; return;
    default: *tx = MV9Shape<4>::TX; *ty = MV9Shape<4>::TY; return;
    }
}

hipError_t launch_minvar9(const void* in, void* out, int dtype, int r, Geom g, uint32_t gate,
                          TileCfg cfg, hipStream_t s, TileCfg* plan, const uint32_t* gate_dev)
{
    if (dtype == LNF_U8) return dispatch_r<uint8_t>(in, out, r, g, gate, cfg, s, plan, gate_dev);
    return dispatch_r<uint16_t>(in, out, r, g, gate, cfg, s, plan, gate_dev);
}

}  // namespace lnf
