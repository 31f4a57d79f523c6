// Streaming MEAN9 tile body: one workgroup filters a TXW x TY column of output
// voxels over the z-range [z0, z1).  Shared by the single-volume kernel, the
// mean filter and the batch kernel.
//
// Arithmetic (paper, Section "Our Method", eqs. 2-3): the sum S over the nine
// clusters is box_x box_y box_z E + c_x c_y c_z E, with box = ones on [-r, r]
// and c = box shifted by -r plus box shifted by +r (the two diagonal clusters
// of an axis).  Per input slice s the x- and y-passes give the plane sums
//   P(s) = box_y box_x E(s),   Q(s) = c_y c_x E(s)
// at each output column, and along z
//   S(z) = sum_{t=z..z+2r} G(t),   G(t) = P(t-r) + Q(t) + Q(t-2r).
//
// The x- and y-passes are products with banded matrices, and run on the matrix
// cores.  One wavefront computes 16 columns x 16*NO rows of outputs; TXW / 16
// of them, side by side, share the staged rows of a slice.
//   1. staging.  The 32 columns [x-8, x+24) around a 16-column block hold its
//      window for every r <= 4, as do 32 rows.  The rows of a slice go to LDS
//      in 16-byte chunks, by LDS DMA (buffer_load ... lds, 16 bytes per lane)
//      PF slices ahead; rows are clamped by their address.  In x the chunks
//      just run on past the row: what is outside the volume has no weight, and
//      the range check of the buffer resource ends the slice.
//   2. digits.  f16 holds integers up to 2048 exactly and the products
//      accumulate in fp32, exact below 2^24.  A voxel is split into bytes
//      (uint16: low and high): one byte permute forms two f16 1024 + byte, and
//      the accumulator of the x-pass starts at -1152 * (sum of the weights),
//      so that the sums are those of byte - 128.  Window sums of a digit are
//      at most 128 (4r+2), 1792 at r = 3; at r = 4 the c-sum would reach 2304,
//      so it is kept as its two boxes.
//   3. x-pass: D1[row][col] = sum_k raw[row][k] Wx[k][col], 16x16x32 products
//      whose A operand is one 16-byte LDS read per lane (row = lane % 16,
//      chunk lane / 16).  The weights of samples outside the volume are folded
//      onto the face voxel that they clamp to.
//   4. y-pass: a lane of D1 holds four consecutive rows of one column, so the
//      D1 of two row blocks are, converted to f16, the A operand of the
//      transposed product D2[col][row] = sum_k D1[k][col] Wy[k][row] with k in
//      the order that the registers have: no exchange between the passes.
//      uint16: the high digit's weights are 256-fold and chained onto the low
//      digit's sum; |D2| <= 324 * 32896 < 2^24.
//   5. z-pass in registers: V(t) = P(t) + Q(t-r), G(t) = Q(t) + V(t-r), a
//      running box of G over 2r+1 slices: 4r+2 values per output, in rings
//      indexed statically by the unrolled loop (uint32 arithmetic modulo 2^32
//      for uint16; uint8 sums stay below 2^24 and are kept in fp32).
//   6. out = round(S / 9n), gate.  A lane holds four consecutive columns of one
//      row, so the outputs pass through LDS and are stored, one slice later,
//      with 16 adjacent lanes to a row.
// One LDS barrier a slice: iteration k computes slice k, starts the staging of
// slice k+PF and stores the outputs of iteration k-1.
// Everything is exact: the same bytes as the definition for every input.
#pragma once

#include <type_traits>

#include "device_common.h"
#include "lnf_internal.h"

namespace lnf {

using half4_t = _Float16 __attribute__((ext_vector_type(4)));
using half8_t = _Float16 __attribute__((ext_vector_type(8)));
using f32x4_t = float __attribute__((ext_vector_type(4)));
using u32x4_t = uint32_t __attribute__((ext_vector_type(4)));

// Tile geometry: TXW / 16 wavefronts side by side, NO = TY / 16 row blocks each.
template <int R, int TY, int TXW, typename T>
struct M9Geo {
    static constexpr int THREADS = TXW / 16 * 64;
    static constexpr int NO = TY / 16;         // 16-row output blocks
    static constexpr int NR = NO + 1;          // 16-row raw blocks
    static constexpr int LY = TY + 4 * R;      // staged rows
    static constexpr int CV = 16 / sizeof(T);  // voxels of a chunk
    // Staged chunks per row: one left of the tile, and past it 8 columns and
    // the word that an unaligned row is shifted by; odd, so that eight rows of a
    // 16-byte read start in eight different groups of four banks.
    static constexpr int NC = ((TXW + CV + 8) / CV + 1) | 1;
    static constexpr int NCH = LY * NC;        // chunks per slice
    static constexpr int NLOAD = (NCH + THREADS - 1) / THREADS;
    static constexpr int D = 2 * R + 2;        // ring period and unroll (even)
    // raw slices in LDS: a divisor of the unroll, so that a slice's buffer is static
    static constexpr int NRB = R == 4 ? 5 : R == 2 ? 3 : 4;
    static constexpr int PF = NRB - 1;         // slices staged ahead
    static_assert(TXW % 16 == 0 && TY % 16 == 0 && R <= 4 && D % NRB == 0, "tile shape");
};

// Waves per SIMD the tile kernels are compiled for: as many as the registers
// allow without spills (none but the 128 x 32 tile of uint16 at r = 4, with 120:
// not a default, see mean9.hip).
template <int R, int TY, typename T>
constexpr int m9_waves()
{
    if (TY == 32) return 2;
    return sizeof(T) == 1 ? (R <= 3 ? 4 : 3) : (R <= 3 ? 3 : 2);
}

template <int R, int TY, int TXW, typename T>
struct M9Smem {
    using G = M9Geo<R, TY, TXW, T>;
    u32x4_t raw[G::NRB][G::NLOAD * G::THREADS];
    T outs[2][TY][TXW + 16];  // pitch: of the sixteen rows written at once eight (uint8: all) fall in different banks
};

// WORDS: every row of both volumes starts at a 32-bit word (mean9_words_ok) and
// the tile has at least four columns in the volume, so rows are staged as they
// are and four outputs of a row stored at once; where two columns are left at
// the end of a uint16 row, the last four outputs overlap those before them.
// Otherwise a row is staged from the aligned word that holds its first byte on
// and shifted as it is read; its outputs leave as described at kPieces.  One
// iteration of a 32 x 16 tile of uint16, four on a CU, takes 0.49 us with words
// and 0.62 without: 0.1 of it the shift, the rest the stores.
// inv_div: 1/(9n), or 1/n with BOX (the box term alone: the mean filter).
template <int R, int TY, typename T, bool GATE, int TXW, bool BOX, bool WORDS>
__device__ __forceinline__ void mean9_body(M9Smem<R, TY, TXW, T>& sm, const T* __restrict__ in,
                                           T* __restrict__ out, Geom g, int x0, int y0, int z0,
                                           int z1, uint32_t gate, double inv_div, int tid)
{
    using S = M9Geo<R, TY, TXW, T>;
    constexpr int NO = S::NO, NR = S::NR, D = S::D, NC = S::NC, NLOAD = S::NLOAD, CV = S::CV;
    constexpr int kT = S::THREADS, NRB = S::NRB, PF = S::PF;
    constexpr int DIG = sizeof(T);               // digits (bytes) per voxel
    constexpr bool SPLIT = !BOX && R == 4;       // c-sum as its two boxes
    constexpr int NQ = BOX ? 1 : SPLIT ? 3 : 2;  // x-pass quantities: P, then Q (or its halves)
    constexpr int LAG = BOX ? 2 * R : 4 * R;     // input slices before the first output
    constexpr int ZH = BOX ? R : 2 * R;          // z-halo of the strip
    constexpr float kBias = sizeof(T) == 1 ? 128.f : 32896.f;
    constexpr bool FP = sizeof(T) == 1;          // z-sums in fp32
    using Z = std::conditional_t<FP, float, uint32_t>;

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 15, gq = (tid >> 4) & 3;
    const int nx = g.nx, ny = g.ny;
    const size_t plane = (size_t)nx * ny;
    const uint32_t pbytes = (uint32_t)(plane * sizeof(T));

    // ---- staging: slot tid + i * kT of a buffer holds chunk slot % NC of row
    // slot / NC; lanes past the tile repeat the last slot's.  off: its byte
    // offset from the first staged voxel of the slice (row ys, column xs); only
    // chunks outside the volume start before that, and they are moved to it.
    // Addresses count from the tile's first voxel and end behind its last row,
    // so that they, the drop offset below included, fit 32 bits for planes of
    // up to 4 GiB.
    const int xl = x0 - CV;  // first staged column
    const int xs = max(xl, 0), ys = max(y0 - 2 * R, 0);
    const int yn = min(y0 - 2 * R + S::LY, ny) - ys;  // staged rows inside the volume
    const size_t sorigin = (size_t)ys * nx + xs;
    const uint32_t sbytes = (uint32_t)(min((int64_t)(plane - sorigin), (int64_t)(yn - 1) * nx + NC * CV) * (int)sizeof(T));
    uint32_t off[NLOAD];
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
        const int e = min(tid + i * kT, S::NCH - 1);
        const int row = e / NC, c = e - row * NC;
        const int64_t at = (int64_t)(clampi(y0 - 2 * R + row, 0, ny - 1) - ys) * nx + xl - xs + CV * c;
        off[i] = (uint32_t)(max(at, (int64_t)0) * (int)sizeof(T));
    }
    // the next slice to load, clamped into the volume
    int zl = z0 - ZH;
    const T* lp = in + (size_t)clampi(zl, 0, g.nz - 1) * plane + sorigin;
    auto stage = [&](int buf) {  // the next slice into buffer buf
        const uint32_t lead = WORDS ? 0u : (uint32_t)(reinterpret_cast<uintptr_t>(lp) & 3);
        const rsrc_t rs = make_rsrc(reinterpret_cast<const char*>(lp) - lead, WORDS ? sbytes : (sbytes + lead + 3) & ~3u);
#pragma unroll
        for (int i = 0; i < NLOAD; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (lds_void_t*)&sm.raw[buf][i * kT + wave * 64], 16,
                WORDS ? off[i] : (off[i] + lead) & ~3u, 0, 0, 0);
        lp += (zl >= 0 && zl < g.nz - 1) ? plane : 0;
        ++zl;
    };

    // ---- x-pass weights of output column x0 + 16 wave + l: how often its
    // window samples column x0 - 8 + 16 wave + 8 gq + j, the voxel of k-slot
    // (gq, j); clamped samples count at the faces, columns outside nothing
    half8_t wx[NQ];
    {
        const int xc = x0 + 16 * wave + l;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int c = x0 - 8 + 16 * wave + 8 * gq + j;
            const bool mine = c >= 0 && c < nx;
            auto box = [&](int ctr) {
                const int hi = c >= nx - 1 ? 2 * R + 1 : clampi(c - (ctr - R) + 1, 0, 2 * R + 1);
                const int lo = c <= 0 ? 0 : clampi(c - (ctr - R), 0, 2 * R + 1);
                return mine ? hi - lo : 0;
            };
            wx[0][j] = (_Float16)(float)box(xc);
            if constexpr (SPLIT) {
                wx[1][j] = (_Float16)(float)box(xc - R);
                wx[2][j] = (_Float16)(float)box(xc + R);
            } else if constexpr (!BOX) {
                wx[1][j] = (_Float16)(float)(box(xc - R) + box(xc + R));
            }
        }
    }
    // ---- y-pass weights of output row l of a block over the 32 raw rows from
    // 8 above the block; k-slot (gq, j) is row 4 gq + j of the upper raw block
    // for j < 4, row 4 gq + j - 4 of the lower one from there
    half8_t wyp[DIG], wyq[DIG];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int d = (j < 4 ? 4 * gq + j : 16 + 4 * gq + j - 4) - 8 - l;
        const int p = (d >= -R && d <= R) ? 1 : 0;
        const int q = ((d >= -2 * R && d <= 0) ? 1 : 0) + ((d >= 0 && d <= 2 * R) ? 1 : 0);
#pragma unroll
        for (int t = 0; t < DIG; ++t) {
            wyp[t][j] = (_Float16)(float)(t ? 256 * p : p);
            wyq[t][j] = (_Float16)(float)(t ? 256 * q : q);
        }
    }
    // ---- A operands: raw row block rt holds rows y0 - 8 + 16 rt + l, staged
    // from y0 - 2R on; rows outside have no weight and read a staged one
    int aoff[NR];       // byte offset in a buffer
    uint32_t arow[NR];  // byte offset of the staged row, as off (modulo 4)
#pragma unroll
    for (int rt = 0; rt < NR; ++rt) {
        const int row = clampi(16 * rt + l - 8 + 2 * R, 0, S::LY - 1);
        aoff[rt] = row * NC * 16 + (CV - 8 + 8 * (2 * wave + gq)) * (int)sizeof(T);
        arow[rt] = ((uint32_t)(clampi(y0 - 2 * R + row, 0, ny - 1) - ys) * (uint32_t)nx + (uint32_t)(xl - xs)) * (uint32_t)sizeof(T);
    }
    // the slice read, clamped as staged, and its bytes past an aligned word
    int zr = z0 - ZH;
    uint32_t rlead = (uint32_t)(reinterpret_cast<uintptr_t>(lp) & 3);
    using words_t = uint32_t __attribute__((ext_vector_type(2 * sizeof(T))));
    auto read_raw = [&](int buf, int rt) -> words_t {
        const char* p = reinterpret_cast<const char*>(sm.raw[buf]) + aoff[rt];
        words_t w = *reinterpret_cast<const words_t*>(p);
        if constexpr (!WORDS) {
            constexpr int kN = 2 * sizeof(T);
            const uint32_t more = *reinterpret_cast<const uint32_t*>(p + 4 * kN), by = arow[rt] + rlead;
#pragma unroll
            for (int a = 0; a < kN; ++a)
                w[a] = __builtin_amdgcn_alignbyte(a + 1 < kN ? w[a + 1] : more, w[a], by);
        }
        return w;
    };
    auto operand = [&](const words_t& w, int t) -> half8_t {  // 1024 + byte t of 8 voxels
        u32x4_t d;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            if constexpr (sizeof(T) == 2)
                d[a] = __builtin_amdgcn_perm(0x64646464u, w[a], t ? 0x04030401u : 0x04020400u);
            else
                d[a] = __builtin_amdgcn_perm(0x64646464u, w[a / 2], (a & 1) ? 0x04030402u : 0x04010400u);
        }
        return __builtin_bit_cast(half8_t, d);
    };

    constexpr float kP = -1152.f * (2 * R + 1), kQ = SPLIT ? kP : 2.f * kP;
    const f32x4_t cp = {kP, kP, kP, kP}, cq = {kQ, kQ, kQ, kQ}, zero = {0.f, 0.f, 0.f, 0.f};

    // ---- outputs as stored.  WORDS: 4 columns per thread, TXW / 4 adjacent
    // threads to a row.  Otherwise tiles 128 wide store the whole 8-byte pieces
    // of a row from its first aligned word on (shifted out of the LDS words that
    // hold them), and what is left at its two ends voxel by voxel, sixteen
    // threads to a row (511 x 512 x 512 uint16, r = 3, 128 x 32 tiles: 175 -> 156
    // us against voxel by voxel); narrower tiles, whose rows have more ends,
    // store voxel by voxel (64 x 16: 200 us against 228).
    // Outputs outside the volume get an offset past the tile's end (the bytes from
    // a tile's first voxel to its last stay 16 below 4 GiB: of its last row it has
    // 256 bytes at most, of a plane below 4 GiB all of it), and slices that
    // are not the strip's an empty buffer resource: either is dropped by the
    // range check, so every iteration issues the same memory operations and
    // its waits can leave the younger ones in flight.
    constexpr int kDrop = (int)0xfffffff0u;
    constexpr bool kPieces = !WORDS && TXW >= 128;
    constexpr int kLanes = WORDS ? TXW / 4 : kPieces ? TXW * (int)sizeof(T) / 8 : TXW;  // threads per row
    constexpr int kRows = kT / kLanes, kBody = (TY + kRows - 1) / kRows;
    constexpr int kEdge = kPieces ? (TY * 16 + kT - 1) / kT : 0;
    constexpr int kStores = kBody + kEdge;
    const int sj = tid % kLanes, srow = tid / kLanes;
    const int cols = min(TXW, nx - x0);  // columns of the tile inside the volume
    const uint32_t rowb = (uint32_t)nx * (uint32_t)sizeof(T);
    const uint32_t sbase = (uint32_t)srow * rowb, ebase = (uint32_t)(tid / 16) * rowb;
    const uint32_t tbytes = (uint32_t)(((int64_t)(min(TY, ny - y0) - 1) * nx + cols) * (int)sizeof(T));
    T* wp = out + (size_t)z0 * plane + (size_t)y0 * nx + x0;
    // held: what a thread stores, read from LDS before the y-pass and stored
    // behind it, so that the read's latency is covered (the same tiles: 23.1 ->
    // 22.1 us; 511 x 512 x 512, r = 3, 128 x 32: 152 -> 149)
    using u32x2 = uint32_t __attribute__((ext_vector_type(2)));
    using body_t = std::conditional_t<kPieces || (WORDS && sizeof(T) == 2), u32x2, std::conditional_t<WORDS, uint32_t, T>>;
    body_t held[kBody];
    T ends[kEdge ? kEdge : 1];
    // bytes of the row at `at` before its first aligned word; the voxel of a
    // row's ends that this thread stores, in bytes from the row's start
    auto head_of = [](uint32_t at) { return (int)(-at & 3u); };
    auto end_pos = [&](int head) {
        const int eb = (tid & 15) * (int)sizeof(T);
        return eb < head ? eb : (max(cols * (int)sizeof(T) - head, 0) & ~7) + eb;
    };
    const int scol = WORDS ? min(4 * sj, max(cols - 4, 0)) : sj;
    // the offsets stored to (not kPieces), formed once: 32 x 16 tiles, 203 x 201 x
    // 201 uint16, r = 1: 22.2 -> 21.4 us
    uint32_t so[kBody];
#pragma unroll
    for (int i = 0; i < kBody; ++i) {
        constexpr int kPer = WORDS ? 4 : 1;
        so[i] = (kPer * sj < cols && y0 + srow + i * kRows < ny)
                    ? sbase + (uint32_t)(i * kRows) * rowb + (uint32_t)scol * (uint32_t)sizeof(T)
                    : (uint32_t)kDrop;
    }
    auto read_out = [&](int buf) {
        const uint32_t lead = (uint32_t)(reinterpret_cast<uintptr_t>(wp) & 3);
#pragma unroll
        for (int i = 0; i < kBody; ++i) {
            const int row = srow + i * kRows;
            if constexpr (WORDS) {
                using at4_t = body_t __attribute__((aligned(4)));
                held[i] = *reinterpret_cast<const at4_t*>(&sm.outs[buf][row][scol]);
            } else if constexpr (kPieces) {
                const int head = head_of(sbase + (uint32_t)(i * kRows) * rowb + lead);
                const uint32_t* p = reinterpret_cast<const uint32_t*>(&sm.outs[buf][row % TY][0]) + 2 * sj;
                const u32x2 d = *reinterpret_cast<const u32x2*>(p);
                held[i] = u32x2{__builtin_amdgcn_alignbyte(d[1], d[0], head), __builtin_amdgcn_alignbyte(p[2], d[1], head)};
            } else {
                held[i] = sm.outs[buf][row][sj];
            }
        }
#pragma unroll
        for (int i = 0; i < kEdge; ++i) {
            const int row = tid / 16 + i * (kT / 16);
            const int pos = end_pos(head_of(ebase + (uint32_t)(i * (kT / 16)) * rowb + lead));
            ends[i] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(&sm.outs[buf][row % TY][0]) +
                                                  min(pos, TXW * (int)sizeof(T)));
        }
    };
    auto store_out = [&](int zo) {
        const bool live = zo >= z0 && zo < z1;
        // rows that start anywhere share cache lines with the tiles beside
        // them: kept in L2 until those are whole, not streamed past it
        // (64 x 16 tiles, 511 x 512 x 512 uint16, r = 3: 245 -> 200 us)
        const uint32_t lead = kPieces ? (uint32_t)(reinterpret_cast<uintptr_t>(wp) & 3) : 0u;
        const rsrc_t wr = make_rsrc(reinterpret_cast<const char*>(wp) - lead, live ? tbytes + lead : 0u);
#pragma unroll
        for (int i = 0; i < kBody; ++i) {
            const int row = srow + i * kRows;
            const uint32_t at = sbase + (uint32_t)(i * kRows) * rowb + lead;
            if constexpr (WORDS) {
                if constexpr (sizeof(T) == 2)
                    __builtin_amdgcn_raw_buffer_store_b64(held[i], wr, so[i], 0, kStoreNT);
                else
                    __builtin_amdgcn_raw_buffer_store_b32(held[i], wr, so[i], 0, kStoreNT);
            } else if constexpr (kPieces) {
                const int from = head_of(at) + 8 * sj;
                const bool ok = row < TY && y0 + row < ny && from + 8 <= cols * (int)sizeof(T);
                __builtin_amdgcn_raw_buffer_store_b64(held[i], wr, ok ? at + from : (uint32_t)kDrop, 0, 0);
            } else {
                buffer_store<T, 0>(held[i], wr, so[i], 0u);
            }
        }
#pragma unroll
        for (int i = 0; i < kEdge; ++i) {
            const int row = tid / 16 + i * (kT / 16);
            const uint32_t at = ebase + (uint32_t)(i * (kT / 16)) * rowb + lead;
            const int pos = end_pos(head_of(at));
            const bool ok = row < TY && y0 + row < ny && pos < cols * (int)sizeof(T);
            buffer_store<T, 0>(ends[i], wr, ok ? at + pos : (uint32_t)kDrop, 0u);
        }
        wp += live ? plane : 0;
    };

    // rings: Q and V hold r slices, G 2r+1 (P of the mean filter in G)
    Z qr[D][NO][4], vr[D][NO][4], gr[D][NO][4], acc[NO][4];
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[o][i] = 0;
#pragma unroll
            for (int u = 0; u < D; ++u) qr[u][o][i] = vr[u][o][i] = gr[u][o][i] = 0;
        }

    const int ns = (z1 - z0) + LAG;  // input slices z0 - ZH .. z1 - 1 + ZH
    // vector-memory operations younger than a slice's staging when it is waited for
    constexpr int kWait = (PF - 1) * (NLOAD + kStores) + kStores;
    // each slice before dropped stores: the operations of an iteration
    read_out(0);
#pragma unroll
    for (int p = 0; p < PF; ++p) {
        stage(p);
        store_out(-1);
    }
    wait_vmem_le<kWait>();
    barrier_lds();
    half4_t d1[DIG][NQ][NR];  // x-pass of the previous iteration's slice
#pragma unroll
    for (int t = 0; t < DIG; ++t)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int rt = 0; rt < NR; ++rt) d1[t][q][rt] = half4_t{0, 0, 0, 0};
    // whole blocks of D slices (no exit inside the unrolled block); the slices
    // past the end are clamped and store nothing
    for (int kb = 0; kb <= ns + 1; kb += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k = kb + u;
            const int us = (u + D - 1) % D;  // ring slot of slice k-1
            const int buf = u & 1;  // == k & 1 because D is even
            // outputs of iteration k-1
            const int zo = z0 + k - 2 - LAG;
            read_out(buf ^ 1);
            stage((u + PF) % NRB);  // slice k+PF; the buffer held slice k-1
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                auto col = [&](int t, int q) {
                    return __builtin_shufflevector(d1[t][q][o], d1[t][q][o + 1], 0, 1, 2, 3, 4, 5, 6, 7);
                };
                f32x4_t sp = zero, sq = zero;
#pragma unroll
                for (int t = 0; t < DIG; ++t) {
                    sp = __builtin_amdgcn_mfma_f32_16x16x32_f16(col(t, 0), wyp[t], sp, 0, 0, 0);
                    if constexpr (!BOX) {
                        sq = __builtin_amdgcn_mfma_f32_16x16x32_f16(col(t, 1), wyq[t], sq, 0, 0, 0);
                        if constexpr (SPLIT)
                            sq = __builtin_amdgcn_mfma_f32_16x16x32_f16(col(t, NQ - 1), wyq[t], sq, 0, 0, 0);
                    }
                }
                uint32_t v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Z p = FP ? (Z)sp[i] : (Z)(int)sp[i];
                    Z gn = p;
                    if constexpr (!BOX) {
                        const Z q = FP ? (Z)sq[i] : (Z)(int)sq[i];
                        // slot (u - R) mod D: r slices ago
                        gn = q + vr[(us + D - R) % D][o][i];
                        vr[us][o][i] = p + qr[(us + D - R) % D][o][i];
                        qr[us][o][i] = q;
                    }
                    // slot (u + 1) mod D holds G of 2r+1 slices ago
                    acc[o][i] += gn - gr[(us + 1) % D][o][i];
                    gr[us][o][i] = gn;
                    if constexpr (FP) {
                        // S' = S - 128 * 9n with |S' / 9n| <= 128: the fp32
                        // product is off by at most 2^-16, less than the
                        // 1/(18n) >= 7.6e-5 to the nearest half
                        const float t = __builtin_fmaf((float)acc[o][i], (float)inv_div, 12582912.f + kBias);
                        v[i] = __builtin_bit_cast(uint32_t, t) - 0x4B400000u;
                    } else {
                        // as round_div_odd, with the bias put back
                        const double t = __builtin_fma((double)(int)acc[o][i], inv_div, 4503599627370496.0 + (double)kBias);
                        v[i] = (uint32_t)__builtin_bit_cast(uint64_t, t);
                    }
                    if (GATE && v[i] < gate) v[i] = 0;
                }
                // row l of the block, columns 16 wave + 4 gq ..
                using out_t = uint32_t __attribute__((ext_vector_type(sizeof(T))));
                out_t w;
                if constexpr (sizeof(T) == 2) {
                    w[0] = v[0] | (v[1] << 16);
                    w[1] = v[2] | (v[3] << 16);
                } else {
                    w[0] = v[0] | (v[1] << 8) | (v[2] << 16) | (v[3] << 24);
                }
                *reinterpret_cast<out_t*>(&sm.outs[buf][16 * o + l][16 * wave + 4 * gq]) = w;
            }
            store_out(zo);
            // x-pass of every raw block, rounded to f16 (exact)
#pragma unroll
            for (int rt = 0; rt < NR; ++rt) {
                const words_t w = read_raw(u % NRB, rt);
#pragma unroll
                for (int t = 0; t < DIG; ++t) {
                    const half8_t a = operand(w, t);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const f32x4_t s = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            a, wx[q], q ? cq : cp, 0, 0, 0);
                        const auto lo = __builtin_amdgcn_cvt_pkrtz(s[0], s[1]);
                        const auto hi = __builtin_amdgcn_cvt_pkrtz(s[2], s[3]);
                        d1[t][q][rt] = half4_t{(_Float16)lo[0], (_Float16)lo[1], (_Float16)hi[0], (_Float16)hi[1]};
                    }
                }
            }
            if constexpr (!WORDS) {
                rlead = (rlead + ((zr >= 0 && zr < g.nz - 1) ? pbytes : 0u)) & 3u;
                ++zr;
            }
            wait_vmem_le<kWait>();  // slice k+1 has landed
            barrier_lds();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // drain the staging of the slices past the end before the LDS is reused
    wait_vmem();
    barrier_lds();
}

// One tile.  words: see WORDS.  tid: threadIdx.x (see tile_tid for loops over
// several tiles).
template <int R, int TY, typename T, bool GATE, int TXW = 64, bool BOX = false>
__device__ __forceinline__ void mean9_tile(M9Smem<R, TY, TXW, T>& sm, bool words,
                                           const T* __restrict__ in, T* __restrict__ out, Geom g,
                                           int x0, int y0, int z0, int z1, uint32_t gate,
                                           double inv_div, int tid)
{
    if (words && g.nx - x0 >= 4)
        mean9_body<R, TY, T, GATE, TXW, BOX, true>(sm, in, out, g, x0, y0, z0, z1, gate, inv_div, tid);
    else
        mean9_body<R, TY, T, GATE, TXW, BOX, false>(sm, in, out, g, x0, y0, z0, z1, gate, inv_div, tid);
}

}  // namespace lnf
