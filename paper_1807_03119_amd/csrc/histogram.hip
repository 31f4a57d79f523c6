// Grey-level histogram of a volume and Otsu's data threshold (paper, Section
// "Our Method", eq. 1), and the paper's automatic pipeline: threshold, then
// the nine-cluster filter gated at that threshold.
//
// Histogram kernels privatise the bins in LDS and flush them with global
// atomics once per workgroup:
//   - uint8: 256 uint32 counters per workgroup;
//   - uint16: 65536 bins as two 16-bit counters per LDS word (128 KiB of the
//     160 KiB LDS, one 1024-thread workgroup per CU).  A workgroup takes chunks
//     of fewer than 65536 voxels, so neither half of a word can carry into the
//     other, and between chunks moves the counts to registers, 64 bins a
//     thread: global memory sees one flush per CU, not one per chunk.  The next
//     chunk's loads are in flight meanwhile.
// The output histogram is cleared by a fill kernel (no memset node), so the
// sequence can be captured in a graph.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>

#include "device_common.h"
#include "lnf.h"
#include "lnf_ctx.h"
#include "lnf_internal.h"

namespace lnf {
namespace {

constexpr int kThreads = 256;
constexpr int kThreads16 = 1024;  // uint16: one 128 KiB workgroup per CU, 16 waves
// 16-byte vectors of a uint16 chunk: 8 per thread, and with up to 14 voxels
// outside the vectors fewer than 65536 voxels
constexpr int kVecs16 = 8189;

__global__ __launch_bounds__(kThreads) void fill_u64(unsigned long long* p, int n)
{
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) p[i] = 0;
}

__global__ __launch_bounds__(kThreads) void hist_u8(const uint8_t* __restrict__ in, size_t n,
                                                     size_t chunk, unsigned long long* hist)
{
    __shared__ uint32_t bins[256];
    bins[threadIdx.x] = 0;
    __syncthreads();
    const size_t begin = (size_t)blockIdx.x * chunk;
    const size_t end = begin + chunk < n ? begin + chunk : n;
    for (size_t i = begin + threadIdx.x; i < end; i += kThreads) atomicAdd(&bins[in[i]], 1u);
    __syncthreads();
    const uint32_t c = bins[threadIdx.x];
    if (c) atomicAdd(&hist[threadIdx.x], (unsigned long long)c);
}

// Chunk c of a workgroup is vectors [(c * gridDim + block) * cv, ... + cv) past
// the first 16-byte boundary, cv <= kVecs16; block 0's first chunk also takes
// the voxels before that boundary and after the last vector.  One flush for all
// chunks, a bin a lane (512 adjacent bytes an atomic instruction; both bins of a
// word by one lane meet 1 KiB): 512^3 of 12 bits 117 us with a flush per chunk,
// 71 with one, 59 with adjacent lanes; 2^25 voxels of 16 bits 570, 324 and 123.
__global__ __launch_bounds__(kThreads16) void hist_u16(const uint16_t* __restrict__ in, size_t n,
                                                        unsigned long long* hist, int cv, int chunks)
{
    constexpr int kLoads = 4, kWords = 32768 / kThreads16;
    __shared__ __align__(16) uint32_t pairs[32768];  // bin 2i in the low half, bin 2i+1 in the high half
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kWords; ++k) pairs[tid + k * kThreads16] = 0;
    const size_t head = std::min<size_t>(n, (16 - reinterpret_cast<uintptr_t>(in) % 16) % 16 / 2);
    const size_t nv = (n - head) / 8;
    const uint4* p = reinterpret_cast<const uint4*>(in + head);
    auto add = [&](uint32_t v) { atomicAdd(&pairs[v >> 1], (v & 1) ? 65536u : 1u); };
    uint32_t lo[kWords] = {}, hi[kWords] = {};
    uint4 v[kLoads];
    bool ok[kLoads];
    // vector i of this thread in half h & 1 of chunk h / 2: none past the chunk
    // or the volume
    auto load = [&](int h, int i) {
        const int c = h >> 1, e = tid + ((h & 1) * kLoads + i) * kThreads16;
        const size_t at = ((size_t)c * gridDim.x + blockIdx.x) * cv + e;
        ok[i] = e < cv && at < nv && c < chunks;
        v[i] = uint4{0, 0, 0, 0};
        if (ok[i]) v[i] = p[at];
    };
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(0, i);
    __syncthreads();
    if (blockIdx.x == 0) {
        const size_t rest = n - head - nv * 8;
        if ((size_t)tid < head) add(in[tid]);
        if ((size_t)tid < rest) add(in[head + nv * 8 + tid]);
    }
    for (int c = 0; c < chunks; ++c) {
#pragma unroll 1
        for (int h = 2 * c; h < 2 * c + 2; ++h)
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const uint4 w = v[i];
                const bool mine = ok[i];
                load(h + 1, i);
                if (mine) {
                    add(w.x & 0xffffu);
                    add(w.x >> 16);
                    add(w.y & 0xffffu);
                    add(w.y >> 16);
                    add(w.z & 0xffffu);
                    add(w.z >> 16);
                    add(w.w & 0xffffu);
                    add(w.w >> 16);
                }
            }
        barrier_lds();
        if (chunks == 1) {
            // the only chunk: straight from LDS, a bin a lane, so that an atomic
            // instruction meets 512 adjacent bytes; 512 empty bins are passed over
            // at once, and each workgroup starts at another part of the bins
            const int lane = tid & 63;
#pragma unroll 2
            for (int k = 0; k < kWords / 4; ++k) {
                const int q = tid - lane + (int)((k + blockIdx.x) % (kWords / 4)) * kThreads16;
                const uint4 w4 = reinterpret_cast<const uint4*>(pairs)[q + lane];
                if (!__any((w4.x | w4.y | w4.z | w4.w) != 0)) continue;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int i = 8 * q + 64 * j + lane;
                    const uint32_t w = pairs[i >> 1], count = (i & 1) ? w >> 16 : w & 0xffffu;
                    if (count) atomicAdd(&hist[i], (unsigned long long)count);
                }
            }
            return;
        }
        int t = tid;  // opaque: the addresses are formed here, not kept over the loop
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int k = 0; k < kWords; ++k) {
            if (k % 8 == 0) asm volatile("" ::: "memory");  // eight words in registers at a time
            const uint32_t w = pairs[t + k * kThreads16];
            pairs[t + k * kThreads16] = 0;
            lo[k] += w & 0xffffu;
            hi[k] += w >> 16;
        }
        barrier_lds();
    }
    // as above, a bin a lane: the wavefront's words hold two bins each, which go
    // to neighbouring lanes (selection by mask: the counts stay 32-bit registers)
    const int lane = tid & 63, base = 2 * (tid - lane) + lane;
    const bool odd = lane & 1;
#pragma unroll
    for (int k = 0; k < kWords; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t l = __shfl(lo[k], 32 * h + (lane >> 1), 64), u = __shfl(hi[k], 32 * h + (lane >> 1), 64);
            const uint32_t c = odd ? u : l;
            if (c) atomicAdd(&hist[base + 64 * h + 2 * k * kThreads16], (unsigned long long)c);
        }
}

// ---- Otsu's threshold and 2 sigma of a histogram, on the device -------------
// One workgroup.  The levels come in chunks of 64, one per lane; wave w takes
// chunks w, w + 16, ... so that the occupied levels, wherever they lie, are
// spread over the waves.  Chunk totals are scanned over the workgroup, then
// each occupied chunk is scanned over its lanes.  Counts and weighted sums are
// exact in uint64 (a volume on the device has fewer than 2^40 voxels).  The
// criterion is evaluated in fp64, good to 2^-50, and the thresholds within
// 2^-40 of its maximum are compared exactly (320-bit products), so the result
// is the host function's for every histogram.
constexpr int kSelThreads = 1024, kSelWaves = kSelThreads / 64, kSelChunks = 1024;

struct Split {
    uint64_t n0, s0;  // class 0 (levels below the threshold): count and weighted sum
    int t;            // the threshold, -1: none
};

using u128 = unsigned __int128;

// num[a]/den[a] > num[b]/den[b] with num = (N s0 - n0 S)^2, den = n0 (N - n0)
__device__ bool split_better(const Split& a, const Split& b, uint64_t N, uint64_t S)
{
    auto dist = [&](const Split& x) -> u128 {
        const u128 p = (u128)N * x.s0, q = (u128)x.n0 * S;
        return p >= q ? p - q : q - p;
    };
    // d^2 * e (d < 2^104, e < 2^80) in five 64-bit limbs
    auto product = [&](u128 d, u128 e, uint64_t(&out)[5]) {
        const uint64_t d0 = (uint64_t)d, d1 = (uint64_t)(d >> 64);
        const u128 p00 = (u128)d0 * d0, p01 = (u128)d0 * d1, p11 = (u128)d1 * d1;
        uint64_t sq[4];
        sq[0] = (uint64_t)p00;
        u128 c = (p00 >> 64) + (u128)(uint64_t)p01 * 2;
        sq[1] = (uint64_t)c;
        c = (c >> 64) + (u128)(uint64_t)(p01 >> 64) * 2 + (uint64_t)p11;
        sq[2] = (uint64_t)c;
        sq[3] = (uint64_t)((c >> 64) + (p11 >> 64));
        const uint64_t e0 = (uint64_t)e, e1 = (uint64_t)(e >> 64);
        uint64_t r[5] = {0, 0, 0, 0, 0};
        u128 carry = 0;
        for (int i = 0; i < 4; ++i) {
            carry += (u128)sq[i] * e0;
            r[i] = (uint64_t)carry;
            carry >>= 64;
        }
        r[4] = (uint64_t)carry;
        carry = 0;
        for (int i = 0; i < 4; ++i) {
            carry += (u128)sq[i] * e1 + r[i + 1];
            r[i + 1] = (uint64_t)carry;
            carry >>= 64;
        }
        for (int i = 0; i < 5; ++i) out[i] = r[i];
    };
    uint64_t x[5], y[5];
    product(dist(a), (u128)b.n0 * (N - b.n0), x);
    product(dist(b), (u128)a.n0 * (N - a.n0), y);
    for (int i = 4; i >= 0; --i)
        if (x[i] != y[i]) return x[i] > y[i];
    return false;
}

template <typename V>
__device__ V wave_scan(V v, int lane)  // inclusive
{
    for (int off = 1; off < 64; off <<= 1) {
        const V u = __shfl_up(v, off, 64);
        if (lane >= off) v += u;
    }
    return v;
}

template <typename V>
__device__ V wave_total(V v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__global__ __launch_bounds__(kSelThreads) void select_scalar(
    const unsigned long long* __restrict__ hist, int levels, int sigma, uint32_t* dev,
    uint32_t* host)
{
    __shared__ uint64_t cn[kSelChunks], cs[kSelChunks];  // chunk totals, then what precedes them
    __shared__ double cmax[kSelChunks];                  // best criterion of a chunk
    __shared__ uint64_t wn[kSelWaves], ws[kSelWaves];
    __shared__ double wmax[kSelWaves];
    __shared__ Split wbest[kSelWaves];
    __shared__ int first_level;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunks = levels / 64;  // 4 or 1024
    cn[tid] = cs[tid] = 0;
    cmax[tid] = -1.0;
    if (tid == 0) first_level = levels;
    __syncthreads();
    uint64_t q2 = 0;  // sigma: this lane's sum of c v^2 (below 2^64: fewer than 2^32 voxels)
    for (int j0 = wave; j0 < chunks; j0 += 8 * kSelWaves) {
        uint64_t c[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = j0 + i * kSelWaves;
            c[i] = j < chunks ? hist[j * 64 + lane] : 0;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = j0 + i * kSelWaves, v = j * 64 + lane;
            if (!__any(c[i] != 0)) continue;
            if (c[i]) atomicMin(&first_level, v);
            if (sigma) q2 += c[i] * (uint64_t)((uint32_t)v * (uint32_t)v);
            const uint64_t n = wave_total(c[i]), s = wave_total(c[i] * (uint64_t)v);
            if (lane == 0) {
                cn[j] = n;
                cs[j] = s;
            }
        }
    }
    __syncthreads();
    // what precedes chunk tid, and the totals
    const uint64_t n_own = cn[tid], s_own = cs[tid];
    const uint64_t n_in = wave_scan(n_own, lane), s_in = wave_scan(s_own, lane);
    if (lane == 63) {
        wn[wave] = n_in;
        ws[wave] = s_in;
    }
    __syncthreads();
    uint64_t N = 0, S = 0, nb = 0, sb = 0;
    for (int w = 0; w < kSelWaves; ++w) {
        if (w == wave) {
            nb = N;
            sb = S;
        }
        N += wn[w];
        S += ws[w];
    }
    cn[tid] = nb + n_in - n_own;
    cs[tid] = sb + s_in - s_own;
    if (sigma) {
        // floor(2 sigma) = the largest w with w^2 N^2 <= 4 (N Q - S^2): the
        // quotient's floor and its root's are the same integer
        __shared__ uint64_t wq[kSelWaves];
        const uint64_t q = wave_total(q2);
        if (lane == 0) wq[wave] = q;
        __syncthreads();
        if (tid == 0) {
            uint64_t Q = 0;
            for (int w = 0; w < kSelWaves; ++w) Q += wq[w];
            const u128 num = 4 * ((u128)N * Q - (u128)S * S), n2 = (u128)N * N;
            // the fp64 root is off by less than 2^-32: at most one step (products
            // below 2^100).  Eighteen 128-bit comparisons of one thread took 4 us.
            const auto real = [](u128 v) { return (double)(uint64_t)(v >> 64) * 18446744073709551616.0 + (double)(uint64_t)v; };
            uint32_t w = (uint32_t)__builtin_sqrt(real(num) / real(n2));
            if (n2 * ((uint64_t)w * w) > num) --w;
            if (n2 * ((uint64_t)(w + 1) * (w + 1)) <= num) ++w;
            *dev = w;
            *host = w;
        }
        return;
    }
    __syncthreads();
    // criterion of every threshold that ends at an occupied level
    auto split_of = [&](int j, uint64_t c) -> Split {
        const int v = j * 64 + lane;
        const Split x{cn[j] + wave_scan(c, lane), cs[j] + wave_scan(c * (uint64_t)v, lane), v + 1};
        return (c == 0 || x.n0 == N) ? Split{0, 0, -1} : x;
    };
    auto criterion = [&](const Split& x) -> double {
        if (x.t < 0) return -1.0;
        const u128 p = (u128)N * x.s0, q = (u128)x.n0 * S, d = p >= q ? p - q : q - p;
        const double df = (double)(uint64_t)(d >> 64) * 18446744073709551616.0 + (double)(uint64_t)d;
        return df / ((double)x.n0 * (double)(N - x.n0)) * df;
    };
    double best = -1.0;
    for (int j = wave; j < chunks; j += kSelWaves) {
        const uint64_t c = hist[j * 64 + lane];
        if (!__any(c != 0)) continue;
        double v = criterion(split_of(j, c));
        for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
        if (lane == 0) cmax[j] = v;
        best = fmax(best, v);
    }
    if (lane == 0) wmax[wave] = best;
    __syncthreads();
    for (int w = 0; w < kSelWaves; ++w) best = fmax(best, wmax[w]);
    const double near = best * (1.0 - 0x1p-40);
    // exact comparison of the near ones, lowest threshold first
    Split mine{0, 0, -1};
    if (best >= 0.0) {
        for (int j = wave; j < chunks; j += kSelWaves) {
            if (cmax[j] < near) continue;  // the same for the whole wave
            const Split x = split_of(j, hist[j * 64 + lane]);
            if (criterion(x) >= near && (mine.t < 0 || split_better(x, mine, N, S))) mine = x;
        }
    }
    // over the lanes: better, or equal and lower
    auto take = [&](Split& a, const Split& b) {
        if (b.t < 0) return;
        if (a.t < 0 || split_better(b, a, N, S) || (!split_better(a, b, N, S) && b.t < a.t)) a = b;
    };
    if (__any(mine.t >= 0)) {
        for (int off = 32; off > 0; off >>= 1) {
            Split o;
            o.n0 = __shfl_xor(mine.n0, off, 64);
            o.s0 = __shfl_xor(mine.s0, off, 64);
            o.t = __shfl_xor(mine.t, off, 64);
            take(mine, o);
        }
    }
    if (lane == 0) wbest[wave] = mine;
    __syncthreads();
    if (tid == 0) {
        Split all{0, 0, -1};
        for (int w = 0; w < kSelWaves; ++w) take(all, wbest[w]);
        // fewer than two levels present: the present one, 0 for none
        const uint32_t t = all.t >= 0 ? (uint32_t)all.t : first_level < levels ? (uint32_t)first_level : 0u;
        *dev = t;
        *host = t;
    }
}

// ---- exact Otsu on the host ------------------------------------------------
// Fixed-width unsigned integers of 12 x 64 bits (least significant limb
// first): wide enough for every product below with counts up to 2^64.
struct Big {
    static constexpr int L = 12;
    uint64_t w[L] = {};
};

Big big(unsigned __int128 v)
{
    Big r;
    r.w[0] = (uint64_t)v;
    r.w[1] = (uint64_t)(v >> 64);
    return r;
}

Big mul(const Big& a, const Big& b)
{
    Big r;
    for (int i = 0; i < Big::L; ++i) {
        if (!a.w[i]) continue;
        unsigned __int128 carry = 0;
        for (int j = 0; i + j < Big::L; ++j) {
            const unsigned __int128 cur = (unsigned __int128)a.w[i] * b.w[j] + r.w[i + j] + carry;
            r.w[i + j] = (uint64_t)cur;
            carry = cur >> 64;
        }
    }
    return r;
}

int cmp(const Big& a, const Big& b)
{
    for (int i = Big::L - 1; i >= 0; --i)
        if (a.w[i] != b.w[i]) return a.w[i] < b.w[i] ? -1 : 1;
    return 0;
}

Big sub(const Big& a, const Big& b)  // a >= b
{
    Big r;
    unsigned __int128 borrow = 0;
    for (int i = 0; i < Big::L; ++i) {
        const unsigned __int128 x = (unsigned __int128)a.w[i] - b.w[i] - borrow;
        r.w[i] = (uint64_t)x;
        borrow = (x >> 64) ? 1 : 0;
    }
    return r;
}

}  // namespace

// T maximising the between-class variance (N*s0 - n0*S)^2 / (n0*n1), which is
// the T minimising eq. 1's within-class variance (their sum is the constant
// total variance).  Class 0 is v < T; lowest T among maxima; with fewer than
// two levels present, T = the present level (0 for an empty histogram).
// Exact for any counts: N < 2^64, S < 2^80, every product below < 2^640.
uint32_t otsu_from_hist(const uint64_t* hist, int levels)
{
    unsigned __int128 N = 0, S = 0;
    for (int v = 0; v < levels; ++v) {
        N += hist[v];
        S += (unsigned __int128)hist[v] * (unsigned)v;
    }
    const Big bN = big(N), bS = big(S);
    unsigned __int128 n0 = 0, s0 = 0;
    int best_t = -1;
    Big best_num, best_den;
    for (int t = 1; t < levels; ++t) {
        // an empty level t-1 leaves both classes, so the criterion, as they
        // were at t-1: a tie, which the lower threshold keeps
        if (!hist[t - 1]) continue;
        n0 += hist[t - 1];
        s0 += (unsigned __int128)hist[t - 1] * (unsigned)(t - 1);
        const unsigned __int128 n1 = N - n0;
        if (n0 == 0 || n1 == 0) continue;
        const Big a = mul(bN, big(s0)), b = mul(big(n0), bS);
        const Big d = cmp(a, b) >= 0 ? sub(a, b) : sub(b, a);
        const Big num = mul(d, d);
        const Big den = mul(big(n0), big(n1));
        if (best_t < 0 || cmp(mul(num, best_den), mul(best_num, den)) > 0) {
            best_t = t;
            best_num = num;
            best_den = den;
        }
    }
    if (best_t >= 0) return (uint32_t)best_t;
    for (int v = 0; v < levels; ++v)
        if (hist[v]) return (uint32_t)v;
    return 0;
}

hipError_t launch_histogram(const void* vol, size_t n, int dtype, uint64_t* hist, hipStream_t s)
{
    const int levels = dtype == LNF_U8 ? 256 : 65536;
    auto* h = reinterpret_cast<unsigned long long*>(hist);
    hipLaunchKernelGGL(fill_u64, dim3((levels + kThreads - 1) / kThreads), dim3(kThreads), 0, s, h,
                       levels);
    if (n == 0) return hipGetLastError();
    if (dtype == LNF_U8) {
        const size_t groups = std::min<size_t>(4096, (n + 65535) / 65536);
        const size_t chunk = (n + groups - 1) / groups;
        hipLaunchKernelGGL(hist_u8, dim3((unsigned)groups), dim3(kThreads), 0, s,
                           static_cast<const uint8_t*>(vol), n, chunk, h);
    } else {
        // At most one workgroup per CU.  A chunk takes about 6.5 us; what a
        // further workgroup's flush adds depends on the occupied levels, 0.03 us
        // for 4096 of them, 0.5 us for all: 9 sqrt(chunks), and up to 128
        // workgroups one chunk each, lies between the two (2^23 voxels in 48, 128
        // and 192 workgroups: 25, 18 and 13 us, and 46, 81 and 89).  Short volumes
        // are spread over more than they have chunks for, as far as their few
        // voxels bound the flush (2^15 voxels of all levels in 1 and 64
        // workgroups: 14 and 10 us; 2^18 in 4 and 16: 21 and 14, of 4096 levels 17
        // and 7).  A workgroup's counts stay below 2^32.
        const size_t nv = n / 8, full = nv / kVecs16 + 1;
        const size_t best = std::max<size_t>(128, (size_t)(9.0 * std::sqrt((double)full)));
        const size_t spread = std::min<size_t>(n <= 131072 ? 64 : 16, nv / 32 + 1);
        const size_t groups = std::max(std::min({(size_t)device_cus(), std::max(full, spread), best}), nv >> 28);
        const size_t chunks = std::max<size_t>(1, (nv + groups * kVecs16 - 1) / (groups * kVecs16));
        const int cv = (int)((nv + groups * chunks - 1) / (groups * chunks));
        hipLaunchKernelGGL(hist_u16, dim3((unsigned)groups), dim3(kThreads16), 0, s,
                           static_cast<const uint16_t*>(vol), n, h, cv, (int)chunks);
    }
    return hipGetLastError();
}

}  // namespace lnf

namespace lnf {

void otsu_scratch_free(lnf_ctx* h)
{
    for (ScalarSlot& s : h->scalar) {
        if (s.done) {
            if (s.pending) (void)hipEventSynchronize(s.done);
            (void)hipEventDestroy(s.done);
        }
        if (s.ready) (void)hipEventDestroy(s.ready);
        s = ScalarSlot{};
    }
    if (h->otsu_dev) (void)hipFree(h->otsu_dev);
    if (h->otsu_host) (void)hipHostFree(h->otsu_host);
    h->otsu_dev = nullptr;
    h->otsu_host = nullptr;
}

int otsu_scratch(lnf_ctx* h)
{
    if (h->otsu_dev) return LNF_OK;
    // the slots' values lie behind the 65536 counters, a cache line each
    constexpr size_t kLine = 16, kWords = 65536 + kScalarSlots * kLine;
    bool ok = hipMalloc((void**)&h->otsu_dev, kWords * sizeof(uint64_t)) == hipSuccess &&
              hipHostMalloc((void**)&h->otsu_host, kWords * sizeof(uint64_t), hipHostMallocDefault) == hipSuccess;
    for (int i = 0; ok && i < kScalarSlots; ++i) {
        ScalarSlot& s = h->scalar[i];
        s.dev = reinterpret_cast<uint32_t*>(h->otsu_dev + 65536 + i * kLine);
        s.host = reinterpret_cast<uint32_t*>(h->otsu_host + 65536 + i * kLine);
        ok = hipEventCreateWithFlags(&s.ready, hipEventDisableTiming) == hipSuccess &&
             hipEventCreateWithFlags(&s.done, hipEventDisableTiming) == hipSuccess;
    }
    if (!ok) {
        (void)hipGetLastError();
        otsu_scratch_free(h);
        return LNF_ENOMEM;
    }
    return LNF_OK;
}

int launch_scalar(lnf_ctx* h, const void* vol, size_t n, int dtype, bool sigma, hipStream_t stream,
                  ScalarSlot** slot)
{
    // the value is waited for, which a capture cannot do
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return LNF_EHIP;
    if (int rc = otsu_scratch(h)) return rc;
    ScalarSlot& s = h->scalar[h->next_scalar];
    h->next_scalar = (h->next_scalar + 1) % kScalarSlots;
    if (s.pending && hipEventSynchronize(s.done) != hipSuccess) return LNF_EHIP;
    s.pending = false;
    const int levels = dtype == LNF_U8 ? 256 : 65536;
    if (launch_histogram(vol, n, dtype, h->otsu_dev, stream) != hipSuccess) return LNF_EHIP;
    hipLaunchKernelGGL(select_scalar, dim3(1), dim3(kSelThreads), 0, stream,
                       reinterpret_cast<const unsigned long long*>(h->otsu_dev), levels, sigma ? 1 : 0, s.dev, s.host);
    if (hipGetLastError() != hipSuccess || hipEventRecord(s.ready, stream) != hipSuccess) return LNF_EHIP;
    *slot = &s;
    return LNF_OK;
}

int finish_scalar(ScalarSlot* s, hipStream_t stream, uint32_t* value)
{
    // the caller may give the histogram scratch to another stream after this
    if (hipEventRecord(s->done, stream) != hipSuccess) return LNF_EHIP;
    s->pending = true;
    if (hipEventSynchronize(s->ready) != hipSuccess) return LNF_EHIP;
    *value = *static_cast<volatile uint32_t*>(s->host);
    return LNF_OK;
}

}  // namespace lnf

using namespace lnf;

extern "C" int lnf_histogram(lnf_handle h, const void* vol, const int64_t dims[3], int dtype,
                             uint64_t* hist, hipStream_t stream)
{
    if (!h || !vol || !hist || !dims || (dtype != LNF_U8 && dtype != LNF_U16)) return LNF_EINVAL;
    for (int i = 0; i < 3; ++i)
        if (dims[i] < 1 || dims[i] > INT32_MAX) return LNF_EINVAL;
    const size_t n = (size_t)dims[0] * (size_t)dims[1] * (size_t)dims[2];
    const size_t bytes = n * (dtype == LNF_U8 ? 1 : 2);
    const size_t hbytes = (dtype == LNF_U8 ? 256 : 65536) * sizeof(uint64_t);
    const uintptr_t a = (uintptr_t)vol, b = (uintptr_t)hist;
    if (a < b + hbytes && b < a + bytes) return LNF_EINVAL;
    DeviceGuard dg(h->device);
    if (!dg.ok()) return LNF_EHIP;
    int rc;
    if ((rc = check_device_range(vol, bytes, h->device))) return rc;
    if ((rc = check_device_range(hist, hbytes, h->device))) return rc;
    return launch_histogram(vol, n, dtype, hist, stream) == hipSuccess ? LNF_OK : LNF_EHIP;
}

extern "C" int lnf_otsu_threshold(const uint64_t* hist, int levels, uint32_t* T)
{
    if (!hist || !T || levels < 1 || levels > 65536) return LNF_EINVAL;
    *T = otsu_from_hist(hist, levels);
    return LNF_OK;
}

extern "C" int lnf_filter_otsu(lnf_handle h, const void* vol, const int64_t dims[3], int dtype,
                               int radius, void* out, hipStream_t stream, uint32_t* T)
{
    Geom g;
    size_t bytes = 0;
    int rc = check_volume_args(h, vol, dims, dtype, radius, out, &g, &bytes);
    if (rc) return rc;
    DeviceGuard dg(h->device);
    if (!dg.ok()) return LNF_EHIP;
    if ((rc = check_device_range(vol, bytes, h->device))) return rc;
    if ((rc = check_device_range(out, bytes, h->device))) return rc;
    std::lock_guard<std::mutex> lk(h->otsu_mu);
    // the threshold stays on the device for the filter behind it; the host
    // waits for its copy while the filter runs
    ScalarSlot* slot = nullptr;
    if ((rc = launch_scalar(h, vol, (size_t)g.nx * g.ny * g.nz, dtype, false, stream, &slot))) return rc;
    const hipError_t e = launch_rule(h->rule, h->geom, vol, out, dtype, radius, g, 0,
                                     ctx_tile(h, h->rule, dtype, radius, g), stream, nullptr, slot->dev);
    uint32_t t = 0;
    if ((rc = finish_scalar(slot, stream, &t))) return rc;
    if (e != hipSuccess) return LNF_EHIP;
    if (T) *T = t;
    return LNF_OK;
}
