// MEAN9: every voxel becomes the rounded mean of its nine cluster means
// (paper, Section "Our Method", eqs. 2-3 and the nine-cluster figure).
//
// The nine clusters have equal size n = (2r+1)^3, so the mean of means is
// S / (9n) with S the sum over all nine clusters.  S is a convolution of the
// clamp-extended volume E with a kernel that splits into two separable parts:
//   S = box_x box_y box_z E  +  c_x c_y c_z E,
//   box = ones on [-r, r]   (the centre cluster S_0),
//   c   = ones on [-2r, 2r] plus one more at 0  (per axis, the two diagonal
//         clusters at -r and +r overlap on the centre voxel; the product over
//         the three axes enumerates the eight diagonal clusters).
// The kernel evaluates the x- and y-axis as products with banded matrices on
// the matrix cores, in exact arithmetic, and slides a z-window through a
// register ring while each wavefront streams down its z-strip (mean9_tile.h).
#include <algorithm>
#include <vector>

#include "device_common.h"
#include "lnf_internal.h"
#include "mean9_tile.h"

namespace lnf {
namespace {

// Single-volume wrapper around the streaming tile body of mean9_tile.h.  BOX:
// the paper's mean filter (eq. 4), the box term of the same tile.
template <int R, int TY, typename T, bool GATE, int TXW, bool BOX>
__global__ __launch_bounds__((M9Geo<R, TY, TXW, T>::THREADS))
__attribute__((amdgpu_waves_per_eu((m9_waves<R, TY, T>())))) void mean9_stream(
    const T* __restrict__ in, T* __restrict__ out, Geom g, int zs, int tiles_x, int tiles_y,
    int total, uint32_t gate, double inv_div, int words, const uint32_t* __restrict__ gate_dev)
{
    if (GATE && gate_dev) gate = *gate_dev;  // a threshold found on the device
    __shared__ __align__(16) M9Smem<R, TY, TXW, T> sm;
    const int tile = xcd_tile(blockIdx.x, total);
    const int bx = tile % tiles_x;
    const int rest = tile / tiles_x;
    const int by = rest % tiles_y;
    const int bz = rest / tiles_y;
    const int z0 = bz * zs;
    mean9_tile<R, TY, T, GATE, TXW, BOX>(sm, words != 0, in, out, g, bx * TXW, by * TY, z0,
                                         min(z0 + zs, g.nz), gate, inv_div, (int)threadIdx.x);
}

template <int R, typename T, bool GATE>
hipError_t launch_box(const T* in, T* out, Geom g, uint32_t gate, hipStream_t s)
{
    constexpr int threads = M9Geo<R, 16, 64, T>::THREADS;
    const auto kern = mean9_stream<R, 16, T, GATE, 64, true>;
    const int tiles_x = (g.nx + 63) / 64, tiles_y = (g.ny + 15) / 16;
    const int zs = default_zs(tiles_x * tiles_y, g.nz, resident_groups((const void*)kern, threads));
    const int total = tiles_x * tiles_y * ((g.nz + zs - 1) / zs);
    const int n = (2 * R + 1) * (2 * R + 1) * (2 * R + 1);
    const int words = mean9_words_ok(in, out, g.nx, sizeof(T) == 1 ? LNF_U8 : LNF_U16) ? 1 : 0;
    hipLaunchKernelGGL(kern, dim3(total), dim3(threads), 0, s, in, out, g, zs, tiles_x, tiles_y,
                       total, gate, 1.0 / n, words, (const uint32_t*)nullptr);
    return hipGetLastError();
}

template <typename T>
hipError_t dispatch_box(int r, const void* in, void* out, Geom g, uint32_t gate, hipStream_t s)
{
    const T* pin = static_cast<const T*>(in);
    T* pout = static_cast<T*>(out);
    switch (r) {
    case 1: return gate ? launch_box<1, T, true>(pin, pout, g, gate, s) : launch_box<1, T, false>(pin, pout, g, gate, s);
    case 2: return gate ? launch_box<2, T, true>(pin, pout, g, gate, s) : launch_box<2, T, false>(pin, pout, g, gate, s);
    case 3: return gate ? launch_box<3, T, true>(pin, pout, g, gate, s) : launch_box<3, T, false>(pin, pout, g, gate, s);
    case 4: return gate ? launch_box<4, T, true>(pin, pout, g, gate, s) : launch_box<4, T, false>(pin, pout, g, gate, s);
    default: return hipErrorInvalidValue;
    }
}

struct Variant {
    int tx, ty, threads;
};
// output tiles of the compiled shapes
constexpr Variant kVariants[] = {{64, 16, 256}, {128, 32, 512}, {32, 16, 128}, {128, 16, 512}};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

// The default tile is the variant and strip depth with the least estimated
// time: for each round of resident workgroups, iterations of a strip x time of
// an iteration.  Iterations come in whole blocks of 2r+2 and include the 4r
// slices of z-halo, the two of the pipeline.  at[n - 1] is the measured time of
// an iteration (10.5 ns) with n workgroups on a CU, for n up to what the
// registers let be resident; within 5 % the same for r = 1, 2, 3 and for the
// shapes measured (128 x 256 x 200 to 256 x 256 x 150).  It steps where a SIMD
// gets one wavefront more: the narrow tiles, whose workgroups are two
// wavefronts, run four to a CU in little more than the time of one.
// Kept for rows that are staged and stored as whole words (mean9_words_ok) and
// for others, which are shifted as they are read and stored.
struct TileCost {
    int at[6];  // 0: not resident
};
constexpr TileCost kCostU16[2][kNumVariants] = {
    {{{44, 61, 84, 111, 136}}, {{100}}, {{37, 51, 54, 59, 78, 85}}, {{67, 134}}},
    {{{34, 48, 69, 92, 113}}, {{77}}, {{28, 41, 42, 47, 65, 70}}, {{46, 98}}}};
constexpr TileCost kCostU8[2][kNumVariants] = {
    {{{29, 38, 52, 65, 82}}, {{61}}, {{26, 33, 34, 36, 50, 61}}, {{44, 76}}},
    {{{22, 28, 40, 51, 66}}, {{40}}, {{19, 24, 26, 28, 38, 48}}, {{30, 53}}}};
// At r = 4 the rings take more registers, so fewer workgroups are resident.
constexpr int kResidentU16R4[kNumVariants] = {2, 1, 4, 1}, kResidentU8R4[kNumVariants] = {3, 1, 6, 1};

// whether rows start at whole words, given volumes that do
int row_words(int dtype, int nx) { return nx % (dtype == LNF_U8 ? 4 : 2) == 0; }

TileCost cost_of(int dtype, int variant, int r, Geom g)
{
    const int words = row_words(dtype, g.nx);
    TileCost c = dtype == LNF_U8 ? kCostU8[words][variant] : kCostU16[words][variant];
    if (r == 4)
        for (int n = dtype == LNF_U8 ? kResidentU8R4[variant] : kResidentU16R4[variant]; n < 6; ++n) c.at[n] = 0;
    return c;
}

int resident_of(const TileCost& c)
{
    int n = 1;
    while (n < 6 && c.at[n]) ++n;
    return n;
}

// What the halos cost once the volume does not stay in the caches: percent of
// the time above, by variant.  A row of a narrow tile is part of a 128-byte
// line that its neighbours fetch again.  Between 64 MB and 256 MB (input and
// output) that shows for the 32-wide tile (320^3 uint8, r = 3: 64 x 16 25.6 us,
// 32 x 16 29.2), beyond it is memory that bounds the narrow tiles (512^3 uint16,
// r = 3: 128 x 32 129 us, 128 x 16 148, 64 x 16 172, 32 x 16 250).
constexpr int kMidU16[kNumVariants] = {100, 100, 120, 100}, kMidU8[kNumVariants] = {100, 100, 140, 100};
constexpr int kLarge[kNumVariants] = {125, 100, 190, 112};

int traffic_percent(int dtype, int variant, double voxels)
{
    const double bytes = voxels * (dtype == LNF_U8 ? 2 : 4);
    if (bytes > 268435456.0) return kLarge[variant];
    if (bytes > 67108864.0) return dtype == LNF_U8 ? kMidU8[variant] : kMidU16[variant];
    return 100;
}

long long tile_groups(int variant, int zs, Geom g)
{
    const Variant v = kVariants[variant];
    return (long long)((g.nx + v.tx - 1) / v.tx) * ((g.ny + v.ty - 1) / v.ty) * ((g.nz + zs - 1) / zs);
}

int tile_iterations(int zs, int r)
{
    const int d = 2 * r + 2;
    return (zs + 4 * r + 2 + d - 1) / d * d;
}

// Whether `variant` is one to consider when `want` is asked for.
bool tile_eligible(int variant, int want, int dtype, int r)
{
    if (want >= 0 && want < kNumVariants) return variant == want;
    return !(variant == 1 && r == 4 && dtype == LNF_U16);
}

// variant < 0 and zs <= 0 ask for the default.
TileCfg resolve_tile(TileCfg want, int dtype, int r, Geom g)
{
    TileCfg best = want;
    double best_cost = -1;
    const int cus = device_cus(), most = std::max(1, g.nz / 4);  // strips of 4 slices at least
    for (int v = 0; v < kNumVariants; ++v) {
        if (!tile_eligible(v, want.variant, dtype, r)) continue;
        const TileCost c = cost_of(dtype, v, r, g);
        const int resident = resident_of(c), percent = traffic_percent(dtype, v, (double)g.nx * g.ny * g.nz);
        const int cols = (int)std::min<long long>(tile_groups(v, g.nz, g), 1 << 24);
        // strip counts that fill whole rounds: one round of 1 .. resident
        // workgroups per CU, or up to four full ones
        for (int i = 1; i < resident + 4; ++i) {
            const int per_cu = std::min(i, resident), rounds = i - per_cu + 1;
            int nzs = want.zs > 0 ? (g.nz + want.zs - 1) / want.zs
                                  : std::min(most, std::max(1, cus * per_cu * rounds / cols));
            const int zs = want.zs > 0 ? want.zs : (g.nz + nzs - 1) / nzs;
            nzs = (g.nz + zs - 1) / zs;
            const int groups = (int)std::min<long long>((long long)cols * nzs, 1 << 30);
            const int n = (groups + cus - 1) / cus;  // workgroups of a CU
            const int time = n / resident * c.at[resident - 1] + (n % resident ? c.at[n % resident - 1] : 0);
            // a further round starts with its weights and first slices: 3 iterations
            const double cost =
                ((double)time * tile_iterations(zs, r) + (n - 1) / resident * 3 * c.at[resident - 1]) * percent;
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = TileCfg{v, zs};
            }
        }
    }
    return best;
}

template <int R, typename T, bool GATE, int TY, int TXW>
hipError_t launch_stream(const T* in, T* out, Geom g, uint32_t gate, int zs, hipStream_t s,
                         const uint32_t* gate_dev)
{
    constexpr int threads = M9Geo<R, TY, TXW, T>::THREADS;
    const auto kern = mean9_stream<R, TY, T, GATE, TXW, false>;
    const int tiles_x = (g.nx + TXW - 1) / TXW, tiles_y = (g.ny + TY - 1) / TY;
    const int nzs = (g.nz + zs - 1) / zs;
    const int total = tiles_x * tiles_y * nzs;
    const int n = (2 * R + 1) * (2 * R + 1) * (2 * R + 1);
    const int words = mean9_words_ok(in, out, g.nx, sizeof(T) == 1 ? LNF_U8 : LNF_U16) ? 1 : 0;
    hipLaunchKernelGGL(kern, dim3(total), dim3(threads), 0, s, in, out, g, zs, tiles_x, tiles_y,
                       total, gate, 1.0 / (9.0 * n), words, gate_dev);
    return hipGetLastError();
}

template <int R, typename T, bool GATE>
hipError_t launch_variant(int variant, const void* in, void* out, Geom g, uint32_t gate, int zs,
                          hipStream_t s, const uint32_t* gate_dev)
{
    const T* pin = static_cast<const T*>(in);
    T* pout = static_cast<T*>(out);
    switch (variant) {
    case 0: return launch_stream<R, T, GATE, 16, 64>(pin, pout, g, gate, zs, s, gate_dev);
    case 1: return launch_stream<R, T, GATE, 32, 128>(pin, pout, g, gate, zs, s, gate_dev);
    case 2: return launch_stream<R, T, GATE, 16, 32>(pin, pout, g, gate, zs, s, gate_dev);
    default: return launch_stream<R, T, GATE, 16, 128>(pin, pout, g, gate, zs, s, gate_dev);
    }
}

template <int R, typename T>
hipError_t launch_r(int variant, const void* in, void* out, Geom g, uint32_t gate, int zs,
                    hipStream_t s, const uint32_t* gate_dev)
{
    if (gate || gate_dev)
        return launch_variant<R, T, true>(variant, in, out, g, gate, zs, s, gate_dev);
    return launch_variant<R, T, false>(variant, in, out, g, gate, zs, s, nullptr);
}

template <typename T>
hipError_t dispatch_r(const void* in, void* out, int r, Geom g, uint32_t gate, TileCfg cfg,
                      hipStream_t s, TileCfg* plan, const uint32_t* gate_dev)
{
    if (r < 1 || r > LNF_RADIUS_MAX) return hipErrorInvalidValue;
    cfg = resolve_tile(cfg, sizeof(T) == 1 ? LNF_U8 : LNF_U16, r, g);
    if (plan) {
        *plan = cfg;
        return hipSuccess;
    }
    const int v = cfg.variant;
    switch (r) {
    case 1: return launch_r<1, T>(v, in, out, g, gate, cfg.zs, s, gate_dev);
    case 2: return launch_r<2, T>(v, in, out, g, gate, cfg.zs, s, gate_dev);
    case 3: return launch_r<3, T>(v, in, out, g, gate, cfg.zs, s, gate_dev);
    default: return launch_r<4, T>(v, in, out, g, gate, cfg.zs, s, gate_dev);
    }
}

}  // namespace

int mean9_variants() { return kNumVariants; }

// The tile and strip depth of a batch class: work spread over the CUs and a
// tail of the longest strip.  Each volume pushes the others out of the caches,
// which costs the narrow tiles more than alone (64 volumes of 64^3 to 384^3:
// 857 us with these times of an iteration, 1049 us with those of single calls,
// which prefer 32 x 16): {with one workgroup on a CU, more for each further
// one, resident}.
struct BatchCost {
    int one, more, resident;
};
constexpr BatchCost kBatchU16[2][kNumVariants] = {{{38, 22, 3}, {104, 0, 1}, {36, 12, 6}, {64, 0, 1}},
                                                  {{36, 20, 3}, {84, 0, 1}, {33, 12, 6}, {50, 0, 1}}};
constexpr BatchCost kBatchU8[2][kNumVariants] = {{{30, 10, 4}, {62, 0, 1}, {28, 8, 8}, {44, 20, 2}},
                                                 {{28, 9, 4}, {48, 0, 1}, {26, 8, 8}, {36, 20, 2}}};

TileCfg mean9_class_tile(int variant, int dtype, int r, const std::vector<Geom>& g)
{
    constexpr int kDepths[] = {16, 24, 32, 48, 64, 96, 128, 192};
    TileCfg best{0, 16};
    float best_cost = -1.f;
    const float cus = (float)device_cus();
    for (int v = 0; v < kNumVariants; ++v) {
        if (!tile_eligible(v, variant, dtype, r)) continue;
        float work[8] = {}, longest[8] = {};
        for (const Geom& q : g) {
            const int words = row_words(dtype, q.nx);
            const BatchCost c = dtype == LNF_U8 ? kBatchU8[words][v] : kBatchU16[words][v];
            const int resident = r == 4 ? (dtype == LNF_U8 ? kResidentU8R4 : kResidentU16R4)[v] : c.resident;
            const float tau = (float)(c.one + (resident - 1) * c.more);
            const float cols = (float)tile_groups(v, q.nz, q) * tau / resident;
            for (int i = 0; i < 8; ++i) {
                const int nzs = (q.nz + kDepths[i] - 1) / kDepths[i];
                const float iters = (float)tile_iterations((q.nz + nzs - 1) / nzs, r);
                work[i] += cols * nzs * iters;
                longest[i] = std::max(longest[i], tau * iters);
            }
        }
        for (int i = 0; i < 8; ++i) {
            const float cost = work[i] / cus + longest[i];
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = TileCfg{v, kDepths[i]};
            }
        }
    }
    return best;
}

void mean9_tile_shape(int variant, int* tx, int* ty)
{
    const Variant v = kVariants[(variant >= 0 && variant < kNumVariants) ? variant : 0];
    *tx = v.tx;
    *ty = v.ty;
}

hipError_t launch_box_mean(const void* in, void* out, int dtype, int r, Geom g, uint32_t gate,
                           hipStream_t s)
{
    if (dtype == LNF_U8) return dispatch_box<uint8_t>(r, in, out, g, gate, s);
    return dispatch_box<uint16_t>(r, in, out, g, gate, s);
}

hipError_t launch_mean9(const void* in, void* out, int dtype, int r, Geom g, uint32_t gate,
                        TileCfg cfg, hipStream_t s, TileCfg* plan, const uint32_t* gate_dev)
{
    if (dtype == LNF_U8) return dispatch_r<uint8_t>(in, out, r, g, gate, cfg, s, plan, gate_dev);
    return dispatch_r<uint16_t>(in, out, r, g, gate, cfg, s, plan, gate_dev);
}

}  // namespace lnf
