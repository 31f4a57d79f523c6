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
#include <cmath>
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

// Strip depth of the mean filter, of those that fill whole blocks of 2r+2
// iterations (a strip takes its slices, the 2r of halo and the two of the
// pipeline): least (iterations + 4) x the time of the rounds that the CUs take,
// 1 + n for n workgroups on a CU.  On ten volumes of 101 x 133 x 75 to 512 x 512 x 128,
// both types, r = 1..3, within 0.7 % of the best of twenty depths on average;
// strips of 16 slices at least, at the general cost, 11 % (203 x 301 x 99 uint16 r
// = 1, odd rows: 17.3 -> 14.4 us; 101 x 133 x 75 r = 2: 12.9 -> 8.1).
int box_depth(int tiles, int nz, int r, int resident)
{
    const int cus = device_cus(), d = 2 * r + 2;
    int best = nz;
    long long best_cost = -1;
    for (long long k = ((long long)nz + 2 * d - 1) / d; k >= 2; k -= 1 + k / 64) {  // every one up to 64 blocks
        const int zs = (int)std::min<long long>(nz, (k - 1) * d);
        const long long n = ((long long)tiles * (((long long)nz + zs - 1) / zs) + cus - 1) / cus;
        const long long full = n / resident, rest = n % resident;
        const long long cost = (full * (1 + resident) + (rest ? 1 + rest : 0)) * (k * d + 4);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = zs;
        }
    }
    return best;
}

template <int R, typename T, bool GATE>
hipError_t launch_box(const T* in, T* out, Geom g, uint32_t gate, hipStream_t s)
{
    constexpr int threads = M9Geo<R, 16, 64, T>::THREADS;
    const auto kern = mean9_stream<R, 16, T, GATE, 64, true>;
    const int tiles_x = (g.nx + 63) / 64, tiles_y = (g.ny + 15) / 16;
    const int zs = box_depth(tiles_x * tiles_y, g.nz, R, resident_groups((const void*)kern, threads) / device_cus());
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

constexpr int kMostResident = 10;  // most workgroups of a tile kernel on a CU

struct Variant {
    int tx, ty;
};
// output tiles of the compiled shapes
constexpr Variant kVariants[] = {{64, 16}, {128, 32}, {32, 16}, {128, 16}};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

// The default tile is the variant and strip depth with the least estimated
// time: for each round of the workgroups that the CUs hold at once (as many as a
// row of the table has entries: the kernels' occupancy), iterations of a strip,
// and 6 for its start, x time of an iteration.  Iterations come in
// whole blocks of 2r+2 and include the 4r slices of z-halo, the two of the
// pipeline.  at[n - 1] is the time of an iteration, in ns, with n workgroups on a
// CU: medians over 450 random volumes (sides 48..800, 2^26 voxels at most, every
// variant at up to 20 depths, the GPU kept busy), less 4 us for a launch.  It
// steps where a SIMD gets one wavefront more: the narrow tiles, whose workgroups
// are two wavefronts, run four to a CU in little more than the time of two.
// Kept for rows that are staged and stored as whole words (mean9_words_ok) and
// for others, which are shifted as they are read and stored.
// On 250 other volumes the choice takes 1.3 % more than the best of the
// times measured on average, 4 % more in nine of ten; on 70 of 2^26 to 2^28
// voxels 1 %.
struct TileCost {
    int at[kMostResident];  // 0: never resident
};
// [r - 1][whole words][variant]
constexpr TileCost kCostU16[LNF_RADIUS_MAX][2][kNumVariants] = {
    {{{{393, 512, 670, 842}}, {{854}}, {{358, 467, 470, 506, 658, 800, 807, 842}}, {{579, 960}}},
     {{{299, 395, 534, 673}}, {{673}}, {{279, 379, 379, 406, 537, 664, 677, 704}}, {{397, 662}}}},
    {{{{398, 527, 705}}, {{849}}, {{350, 450, 468, 489, 660, 688}}, {{545}}},
     {{{326, 423, 582}}, {{671}}, {{280, 379, 385, 408, 557, 575}}, {{397}}}},
    {{{{402, 545, 735}}, {{876}}, {{349, 461, 474, 521, 685, 708}}, {{594}}},
     {{{328, 433, 598}}, {{685}}, {{281, 381, 381, 413, 567, 605}}, {{438}}}},
    {{{{447, 605}}, {{1684}}, {{370, 516, 530, 576}}, {{666}}},
     {{{352, 494}}, {{1179}}, {{310, 452, 454, 496}}, {{489}}}}};
constexpr TileCost kCostU8[LNF_RADIUS_MAX][2][kNumVariants] = {
    {{{{279, 340, 431, 537, 641}}, {{515, 839}}, {{251, 298, 307, 314, 416, 501, 509, 530, 615, 645}}, {{383, 622}}},
     {{{225, 261, 348, 434, 521}}, {{351, 591}}, {{187, 232, 235, 243, 334, 404, 411, 432, 507, 537}}, {{271, 424}}}},
    {{{{276, 338, 433, 535}}, {{509}}, {{250, 303, 309, 318, 413, 511, 512, 534}}, {{390, 622}}},
     {{{220, 256, 343, 435}}, {{370}}, {{188, 230, 233, 249, 330, 401, 405, 428}}, {{276, 434}}}},
    {{{{280, 331, 443, 549}}, {{530}}, {{257, 310, 317, 337, 436, 526, 541, 570}}, {{411, 657}}},
     {{{219, 256, 343, 439}}, {{364}}, {{197, 240, 258, 309, 399, 435, 493, 547}}, {{268, 434}}}},
    {{{{297, 377, 502}}, {{643}}, {{271, 340, 352, 370, 491, 511}}, {{434}}},
     {{{247, 297, 403}}, {{429}}, {{221, 270, 276, 307, 414, 432}}, {{288}}}}};

// whether rows start at whole words, given volumes that do
int row_words(int dtype, int nx) { return nx % (dtype == LNF_U8 ? 4 : 2) == 0; }

const TileCost& cost_of(int dtype, int variant, int r, Geom g)
{
    return (dtype == LNF_U8 ? kCostU8 : kCostU16)[r - 1][row_words(dtype, g.nx)][variant];
}

// Workgroups of the variant's kernel that a CU holds at once.
int resident_of(const TileCost& c)
{
    int n = 1;
    while (n < kMostResident && c.at[n]) ++n;
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
// 128 x 32 at r = 4 on uint16 only then: 18 ring values of 8 outputs do not fit
// the registers (120 spills; an output takes 1.2 to 1.5 times that of 128 x 16).
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
        const TileCost& c = cost_of(dtype, v, r, g);
        const int resident = resident_of(c);
        const int percent = traffic_percent(dtype, v, (double)g.nx * g.ny * g.nz);
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
            const double time = (double)(n / resident) * c.at[resident - 1] + (n % resident ? c.at[n % resident - 1] : 0);
            const double cost = time * (tile_iterations(zs, r) + 6) * percent;
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = TileCfg{v, zs};
            }
            if (want.zs > 0 || nzs >= most) break;  // no other depth follows
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

// The tile and strip depth of a batch class, by estimated time.  Strips: with no
// more workgroups than the CUs hold, the longest strip at the time of an
// iteration with that many; else all strips spread over the CUs, and a tail of
// three quarters of the longest strip alone (3 iterations for the start of
// each).  Memory: kTraffic input sizes at 4.6 GB/ms for what a tile shape fetches
// beside its outputs, half of it below 2^27 voxels.  The estimate is the root of
// the two squares, since neither hides the other.  In a batch the 128-wide tiles
// take 8 % longer than the tables above, the 32-wide 5 %.
// From 240 random batches of one class (2 to 24 volumes with sides of 32 to
// 520), every variant at eight depths: of those above 60 us the choice
// takes 4.5 % more than the best of the times on average (with times fitted to
// one batch of 64 volumes, 10 %).
constexpr float kTraffic[kNumVariants] = {2.4f, 1.6f, 4.f, 1.6f}, kInBatch[kNumVariants] = {1.f, 1.08f, 1.05f, 1.08f};

TileCfg mean9_class_tile(int variant, int dtype, int r, const std::vector<Geom>& g)
{
    constexpr int kDepths[] = {16, 24, 32, 48, 64, 96, 128, 192}, kN = 8;
    // strips and iterations of a strip by volume and depth, the same for every
    // variant; the longest strip by depth, for rows that are whole words or not
    std::vector<float> strips(g.size() * kN), iters(g.size() * kN);
    float most[2][kN] = {};
    double voxels = 0;
    for (size_t q = 0; q < g.size(); ++q) {
        voxels += (double)g[q].nx * g[q].ny * g[q].nz;
        for (int i = 0; i < kN; ++i) {
            const int nzs = (g[q].nz + kDepths[i] - 1) / kDepths[i];
            strips[q * kN + i] = (float)nzs;
            iters[q * kN + i] = (float)(tile_iterations((g[q].nz + nzs - 1) / nzs, r) + 3);
            float& m = most[row_words(dtype, g[q].nx)][i];
            m = std::max(m, iters[q * kN + i]);
        }
    }
    TileCfg best{0, 16};
    float best_cost = -1.f;
    const float cus = (float)device_cus();
    const double passes = voxels * (dtype == LNF_U8 ? 1 : 2) / 4600.0 * (voxels < 134217728.0 ? 0.5 : 1.0);
    for (int v = 0; v < kNumVariants; ++v) {
        if (!tile_eligible(v, variant, dtype, r)) continue;
        const TileCost* const c = (dtype == LNF_U8 ? kCostU8 : kCostU16)[r - 1][0] + v;
        const TileCost* const cw = (dtype == LNF_U8 ? kCostU8 : kCostU16)[r - 1][1] + v;
        const int resident = resident_of(*c);
        float groups[kN] = {}, work[kN] = {};
        for (size_t q = 0; q < g.size(); ++q) {
            const float cols = (float)tile_groups(v, g[q].nz, g[q]);
            const float tau = cols * (float)(row_words(dtype, g[q].nx) ? cw : c)->at[resident - 1] / (float)resident;
            for (int i = 0; i < kN; ++i) {
                groups[i] += cols * strips[q * kN + i];
                work[i] += tau * strips[q * kN + i] * iters[q * kN + i];
            }
        }
        for (int i = 0; i < kN; ++i) {
            const int n = std::max(1, (int)std::min((groups[i] + cus - 1.f) / cus, (float)resident));
            const float longest = std::max(most[0][i] * (float)c->at[n - 1], most[1][i] * (float)cw->at[n - 1]);
            const float alone = std::max(most[0][i] * (float)c->at[0], most[1][i] * (float)cw->at[0]);
            const bool rounds = groups[i] > cus * (float)resident;
            const float time = rounds ? std::max(work[i] / cus + 0.75f * alone, longest) : longest;
            const float cost = std::hypot(time * kInBatch[v], (float)passes * kTraffic[v]);
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
