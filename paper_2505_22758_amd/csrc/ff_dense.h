// Projections of the wide pass: a dense contraction on the matrix cores, v_mfma_f32_16x16x32_bf16
// multiplying the inputs of 16 sequences (A operand) by 16 weight rows (B operand) over 32 columns.
//
// The paper keeps its row-partitioned matrix-vector scheme up to batch 4 (Section 5.2, larger batch
// sizes) and leaves more sequences open.  Here
//   * a WORKGROUP owns a contiguous range of rows (N / workgroups, in groups of four) and works on it
//     in panels of up to kPanelTiles tiles of 16 rows; its eight waves split K, each multiplying every
//     eighth block of columns for ALL tiles of the panel.  Every input element is therefore
//     needed by exactly one wave of the workgroup, which loads it straight from the global image
//     (ff_wide.h: written in operand order, 1 KB per load, the workgroups of an XCD share it in
//     their L2) into registers and reuses it for every tile: nothing is staged through LDS;
//   * weights are stored tile by tile in operand order (PMat): a load is one contiguous kilobyte, lane
//     (r = lane % 16, g = lane / 16) getting 16 bytes of weight row r.  From row-major weights (64 bytes
//     of each of 16 rows per load) the same loop streams at 3.8 TB/s, from tiles at 6.6 (8B gate/up).
//     The accumulators of lane (r, g) hold row r for sequences 4 g .. 4 g + 3, so what belongs to a
//     weight row (int4 scales and zeros) belongs to the lane that loaded the row;
//   * a wave keeps D iterations of weights (and of the inputs they meet) in flight in a register ring,
//     refilled tile by tile behind its products, unconditionally (where code paths that issued different
//     numbers of loads meet, the compiler waits for all);
//   * the waves' partial tiles meet in LDS, wave t adds and finishes tile t.
// Two waves per SIMD: the eight waves' rings hold up to 112 KB per compute unit in flight, and one
// wave's conversions overlap the other's matrix-core work.
//
// Inputs are bf16 head + bf16 remainder (17 significant bits).  NC = 16: heads and remainders are
// separate operands, 16 sequences per tile.  NC = 8: rows 0..7 of the operand are the heads and rows
// 8..15 the remainders of 8 sequences, i.e. one multiplication and half the input bytes per k-step;
// the two halves of the result are added when the waves' partial tiles meet.  NC = 1: one sequence,
// whose inputs keep the 24 bits of fp32 (as on the vector ALU): head, remainder and third part are rows 0, 1, 2.
#pragma once
#include "ff_kernels.h"

namespace ff {

constexpr int kWideWaves = 8;
constexpr int kWideThreads = kWideWaves * 64;
constexpr int kPanelTiles = 7;                               // tiles of one panel: one per wave when the partial tiles are added
constexpr int kWideRedBytes = kWideWaves * kPanelTiles * 1024;   // LDS: the waves' partial tiles
constexpr int kWideSzBytes = 64 * 1024;                      // LDS: int4 scales and zeros of the panel(s)
typedef __bf16 mfma_bf8 __attribute__((ext_vector_type(8)));

// Per weight format: 16-byte loads per tile and iteration, k-steps (32 columns) and columns per iteration.
template <int WD> constexpr int kWLoads = WD == W_BF16 ? 2 : 1;
template <int WD> constexpr int kWSteps = WD == W_INT4 ? 4 : 2;
template <int WD> constexpr int kWCols = 32 * kWSteps<WD>;
template <int NC> constexpr int kXOps = NC == 16 ? 2 : 1;   // input operands per k-step
// Ring depth in iterations: about 14 weight loads (14 KB) per wave in flight, i.e. 112 KB per compute unit, as far
// as the registers and six iterations go (panels of one tile: int8 6 loads, int4 5, at 16 sequences 3).  Twice as many measured slower everywhere (8B bf16 x 2, x 8, 70B x 16, us a pass: 14 loads 1541,
// 1729, 5396; 28 loads 1693, 1914, 5735; 8 loads 1563, 1775, 5464): requests that wait for the memory pipe block the
// younger wave of a SIMD, which then finishes alone, and stand in front of the next hand-over.  (One sequence, 8B bf16, eight
// layers, us per step: 8, 10, 14, 20, 28 loads 766, 762, 749, 775, 763.)
template <int WD, int NC, int T> constexpr int kWDepth = [] {
    const int want = (14 + T * kWLoads<WD> - 1) / (T * kWLoads<WD>);
    const int regs = 4 * (T * kWLoads<WD> + kWSteps<WD> * kXOps<NC>), fit = (WD == W_INT4 ? 112 : 144) / regs;
    const int d = want < fit ? want : fit;
    return d < 1 ? 1 : d > 6 ? 6 : d;
}();

// Tiles of a panel: as few panels as possible, of equal size (by the workgroup that has most rows).
__host__ inline int panel_tiles(int n, int n_ctas) {
    const int tiles = (4 * (((n + 3) / 4 + n_ctas - 1) / n_ctas) + 15) / 16, np = (tiles + kPanelTiles - 1) / kPanelTiles;
    return (tiles + np - 1) / np;
}

// Rows [r0, r1) of a projection that this workgroup computes: whole groups of four (PMat::cta_rows).
struct RowRange { int r0, r1; };
__device__ __forceinline__ RowRange wide_rows(int n, const UDiv& n_ctas) {
    const u32 ngroups = (u32)(n + 3) / 4;
    return RowRange{4 * (int)n_ctas.div(ngroups * blockIdx.x), min(4 * (int)n_ctas.div(ngroups * (blockIdx.x + 1)), n)};
}

// One panel's weights as a wave sees them (tiled layout): load j of tile t is 64 bytes times the tile's rows, contiguous.
template <int T>
struct PanelSrc {
    __amdgpu_buffer_rsrc_t base;   // from the panel's first row on
    u32 tile[T], step[T];          // tile's first byte, bytes per load (uniform)
    u32 lane_off[T];               // lane (r, g): unit g of row r (rows past the end repeat the last one)
    static constexpr u32 kNowhere = 0x7FFFFFF0u;   // an offset behind every panel's descriptor: answered with zeros, without an access
    // Size of the descriptor over `rows` rows.  (Cut off below kNowhere: a panel is far smaller, int4 matrices may reach 8 GB.)
    __host__ __device__ __forceinline__ static u32 extent(int rows, u32 row_bytes) {
        const size_t left = (size_t)rows * row_bytes;
        return left < kNowhere ? (u32)left : kNowhere;
    }
    __device__ __forceinline__ static PanelSrc make(const PMat& M, int p0, int r1, int lane) {
        PanelSrc S;
        const u32 rowb = (u32)M.row_bytes();
        S.base = __builtin_amdgcn_make_buffer_rsrc((void*)(M.w + (size_t)p0 * rowb), 0, (int)extent(M.n - p0, rowb), 0x00020000);
#pragma unroll
        for (int t = 0; t < T; t++) {
            const bool some = p0 + 16 * t < r1;               // a tile past the workgroup's rows repeats the first one
            const int nt = min(r1 - (some ? p0 + 16 * t : p0), 16);
            S.tile[t] = some ? (u32)(16 * t) * rowb : 0u;
            S.step[t] = (u32)nt * 64u;
            S.lane_off[t] = (u32)((lane >> 4) * nt + min(lane & 15, nt - 1)) * 16u;
        }
        return S;
    }
};

// A projection's input image as a wave reads it: lanes of sequences beyond the batch repeat the last one
// (rows of the operand do not mix, theirs are never looked at).
struct PanelImg {
    __amdgpu_buffer_rsrc_t base;
    int step;        // bytes per k-step
    int lane_off;
    template <int WD, int NC>
    __device__ __forceinline__ static PanelImg make(const uint8_t* img, int K, int batch, int lane) {
        const int r = lane & 15, g = lane >> 4, step = wide_step_bytes(NC, batch);
        const int steps = (K + kWCols<WD> - 1) / kWCols<WD> * kWSteps<WD>;
        const int piece = NC == 1 ? 4 * g + min(r, 2) : NC == 8 ? (2 * g + (r >> 3)) * batch + min(r & 7, batch - 1) : g * batch + min(r, batch - 1);
        return PanelImg{__builtin_amdgcn_make_buffer_rsrc((void*)img, 0, steps * step, 0x00020000), step, piece * 16};
    }
};

template <int WD, int NC, int T>
struct PanelRing {
    static constexpr int D = kWDepth<WD, NC, T>, DX = D < 2 ? 2 : D, L = kWLoads<WD>, NP = kXOps<NC>, NB = kWSteps<WD> * NP;
    u32x4 w[D][T][L];
    u32x4 x[DX][NB];
    static constexpr u32 kNowhere = PanelSrc<T>::kNowhere;
    // Weights of iteration it (zeros unless `real`).
    __device__ __forceinline__ void load_w(const PanelSrc<T>& S, int slot, int it, bool real) {
#pragma unroll
        for (int t = 0; t < T; t++) load_wt(S, slot, it, t, real);
    }
    __device__ __forceinline__ void load_wt(const PanelSrc<T>& S, int slot, int it, int t, bool real) {
#pragma unroll
        for (int l = 0; l < L; l++)
                w[slot][t][l] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(S.base, real ? S.lane_off[t] : kNowhere, S.tile[t] + (u32)(it * L + l) * S.step[t], 2))   /* streaming */;
    }
    // Inputs of iteration it.  (Buffer loads: base and iteration are scalar operands, the lane's offset one register.)
    __device__ __forceinline__ void load_x(const PanelImg& I, int slot, int it, bool real) {
#pragma unroll
        for (int k = 0; k < kWSteps<WD>; k++)
#pragma unroll
            for (int h = 0; h < NP; h++)
                x[slot][k * NP + h] =
                    __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(I.base, real ? I.lane_off : (int)kNowhere, (it * kWSteps<WD> + k) * I.step + h * (I.step >> 1), 0));
    }
};

__device__ __forceinline__ mfma_f4 mfma16(const u32x4& a, const u32x4& b, const mfma_f4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mfma_bf8, a), __builtin_bit_cast(mfma_bf8, b), c, 0, 0, 0);
}
// Eight int8 codes as bf16 (exact): sign-extending byte conversions, upper halves of two floats packed.
__device__ __forceinline__ u32x4 i8_to_bf16(u32 wa, u32 wb) {
    auto pack = [](float lo, float hi) { return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u); };
    return u32x4{pack((float)(int)(int8_t)wa, (float)(int)(int8_t)(wa >> 8)), pack((float)(int)(int8_t)(wa >> 16), (float)((int)wa >> 24)),
                 pack((float)(int)(int8_t)wb, (float)(int)(int8_t)(wb >> 8)), pack((float)(int)(int8_t)(wb >> 16), (float)((int)wb >> 24))};
}
// Eight int4 codes n (tiled order) as the bf16 numbers 16 + n (0x4180 | n << 3), in column order.
// (With 128 + n what is subtracted again is six times as large: relative error of the logits against 64 bits, one layer,
// 16 sequences: 2.5e-5 with 128 + n, 7.2e-6 with 16 + n, bf16 weights 6.1e-6; 8B x 16, eight layers 681 / 679 us per step.)
constexpr float kI4Offset = 16.f;
__device__ __forceinline__ u32x4 i4_to_bf16(u32 w, u32 mask = 0x00780078u, u32 offs = 0x41804180u) {
    return u32x4{(w & mask) | offs, ((w >> 4) & mask) | offs, ((w >> 8) & mask) | offs, (__builtin_amdgcn_alignbit(w, w, 12) & mask) | offs};
}

// acc[t] += (inputs of iteration it) x (weights of tile t).
// int8: a lane's 16 codes are two k-steps; the row scales multiply the finished sums.
// int4 group-128: an iteration is one group; with the codes n as 16 + n the four k-steps yield
// d = sum (16 + n) x, and with X = sum x of the group (the same instruction with a weight operand of ones)
//     sum s (n - z) x  =  s (d - (16 + z) X).
typedef __attribute__((address_space(3))) f16_t lds_f16;
// Where a wave finds a panel's int4 scales and zeros.
struct PanelSz {
    const lds_f16* lds;          // scales of the panel's rows, as they lie in memory, [row][group]
    int zeros;                   // elements from a scale to its zero
    int ng;                      // groups of a row
};
template <int WD, int NC, int T, class Refill>
__device__ __forceinline__ void panel_multiply(const PanelRing<WD, NC, T>& R, int slot, int xslot, int it, const PanelSz& sz, int lane, mfma_f4 (&acc)[T], Refill&& refill) {
    constexpr int NP = kXOps<NC>;
    mfma_f4 X = {0.f, 0.f, 0.f, 0.f};
    const lds_f16* szp = nullptr;
    int ng = 0;
    if constexpr (WD == W_INT4) {
        const u32x4 ones{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
        for (int i = 0; i < 4 * NP; i++) X = mfma16(R.x[xslot][i], ones, X);
        ng = sz.ng;
        szp = sz.lds + ((lane & 15) * ng + it);
    }
#pragma unroll
    for (int t = 0; t < T; t++) {
        if constexpr (WD == W_BF16) {
#pragma unroll
            for (int k = 0; k < 2; k++)
#pragma unroll
                for (int h = 0; h < NP; h++) acc[t] = mfma16(R.x[xslot][k * NP + h], R.w[slot][t][k], acc[t]);
        } else if constexpr (WD == W_INT8) {
            const u32x4 w = R.w[slot][t][0];
            const u32x4 b0 = i8_to_bf16(w.x, w.y), b1 = i8_to_bf16(w.z, w.w);
#pragma unroll
            for (int h = 0; h < NP; h++) acc[t] = mfma16(R.x[xslot][h], b0, acc[t]);
#pragma unroll
            for (int h = 0; h < NP; h++) acc[t] = mfma16(R.x[xslot][NP + h], b1, acc[t]);
        } else {
            const u32x4 w = R.w[slot][t][0];
            const u32 ww[4] = {w.x, w.y, w.z, w.w};
            mfma_f4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const u32x4 b = i4_to_bf16(ww[q]);
#pragma unroll
                for (int h = 0; h < NP; h++) d = mfma16(R.x[xslot][q * NP + h], b, d);
            }
            const f16_t sv = szp[16 * t * ng], zv = szp[16 * t * ng + sz.zeros];
            const float s = f16_to_f(sv), zp = kI4Offset + f16_to_f(zv);
#pragma unroll
            for (int i = 0; i < 4; i++) acc[t][i] = fmaf(s, fmaf(-zp, X[i], d[i]), acc[t][i]);
        }
        refill(t);
    }
}

// int4: scales and zeros of a panel's rows go into LDS as the slabs that they are in memory, a kilobyte per load, shared out over the waves.  The loads are
// inline assembly (no register outputs); a wave waits for its own by the number of loads made behind them, and for the others' at the barrier in front of the
// products.  (Through registers and transposed into words of scale and zero they held the wave up between the requests for a projection's first tiles and
// the wait for its input, 1 to 3 us: 8B, eight layers, us per step, int4 x 4 498 -> 486, x 16 694 -> 675.)
constexpr int kSzHalf = kWideSzBytes / 2;   // of a panel: one being multiplied, one on its way
// A slab begins at 16 bytes' alignment in memory, up to this many elements in front of the first row's scales (p0 is a multiple of four), and ends at it:
// inside the matrix's region, whose ends are aligned to more.
__device__ __forceinline__ int panel_skew(int p0, int k) { return (p0 * (k / 128)) & 4; }
__host__ __device__ __forceinline__ int panel_zeros(int k, int T) { return (16 * T * (k / 128) * 2 + 8 + 1023) / 1024 * 512; }   // element of the zeros' slab
__device__ __forceinline__ void panel_scales_send(const PMat& M, int p0, int nrows, int T, u32 lds, int wave, int lane) {
    const int ng = M.k / 128, skew = panel_skew(p0, M.k), bytes = ((nrows * ng + skew) * 2 + 15) & ~15, chunks = (bytes + 1023) >> 10;
    const size_t e = (size_t)p0 * ng - skew;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(M.s + e), 0, bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc((void*)(M.z + e), 0, bytes, 0x00020000);
    const u32 z = lds + 2u * (u32)panel_zeros(M.k, T);
    for (int c = wave; c < chunks; c += kWideWaves) {
        const u32 o = (u32)c << 10;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds\n\t"
                     "s_mov_b32 m0, %5\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %4, %3 offen lds"
                     ::"s"(__builtin_amdgcn_readfirstlane(lds + o)), "v"((u32)lane * 16u), "s"(rs), "s"(o), "s"(rz), "s"(__builtin_amdgcn_readfirstlane(z + o)) : "memory", "m0");
    }
}
// Rows too long for that (one or two tiles, more than 1023 or 511 groups): a wave brings the scales of its own next kSzFar iterations into its share of
// the space.  (Read from memory within the loop over tiles, on a branch for such rows, every tile waited for all of the ring where the branch ended, whatever the length of
// its rows.  Us per step with / without it: 8B int4, eight layers, one sequence on a model for eight 438 / 426, x 4 460 / 447, x 16 655 / 645; 70B, four layers, one 517 /
// 457, x 4 532 / 476, x 16 669 / 647.  That the 16 rows of a read meet in two to eight banks, rows of 32 to 224 groups, costs less than changing the places of a row's
// pieces on their way does, 8B x 4 446, x 16 647, or about as much, 70B x 4 470, x 16 643.)
constexpr int kSzFar = 60;   // a multiple of every ring depth
struct PanelSzFar { const f16_t *s, *z; int ng, rows; };   // of the panel's first row; groups of a row, rows
template <int T, class At>
__device__ __forceinline__ void panel_scales_far(const PanelSzFar& far, lds_f16* lds, int lane, At&& at) {   // at: iteration (group) of the i-th
    static_assert(T > 2 || kWideWaves * 2 * 16 * T * kSzFar * 2 <= kWideSzBytes, "scales of a wave's iterations");
#pragma unroll 1
    for (int t = 0; t < T; t++)
#pragma unroll 1
        for (int i = lane >> 4; i < kSzFar; i += 4) {
            const int r = 16 * t + (lane & 15);
            const size_t e = (size_t)max(min(r, far.rows - 1), 0) * far.ng + at(i);
            lds[r * kSzFar + i] = as_global(far.s)[e];
            lds[(16 * T + r) * kSzFar + i] = as_global(far.z)[e];
        }
    settled();
}
template <int LATER> __device__ __forceinline__ void panel_scales_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LATER) : "memory"); }

// A wave's iterations of a panel: every eighth one, so that the workgroup's waves together read contiguous pieces of
// each tile (8B bf16 x 8, int4 x 16, us a pass: 1729, 1591; each wave a contiguous eighth of K: 1730, 1598).
struct WaveIters {
    int n, first;
    __device__ __forceinline__ static WaveIters of(int ni, int wave) {
        const int n = (ni - wave + kWideWaves - 1) / kWideWaves;
        return WaveIters{n, n > 0 ? wave : 0};
    }
    // iteration number i (in the wave's order) as an iteration of the panel; past the end: the last one again
    __device__ __forceinline__ int at(int i) const { return max(min(i, n - 1), 0) * kWideWaves + first; }
};

// The wave's iterations of a panel; the first D slots of weights and DX of inputs have been requested (slots past the end hold repeats).
// int4 up to eight sequences: requests past the end read nothing, so that the loop has no tail of its own to be unrolled, a copy of the long
// product per slot and step (a layer uses three or four panel widths, and the instruction cache holds 64 KB: kernel 272 -> 184 KB, spilled
// registers 56 -> 16, 8B x 4, eight layers, 529 -> 516 us per step).  The others are ahead with the last iterations peeled off the loop (735 /
// 770 bf16 x 2, 534 / 555 int8 x 4, 779 / 811 bf16 x 8, 724 / 737 int4 x 16).
// FAR: rows too long for LDS to hold the panel's scales (far; sz: the space).
template <int WD, int NC, int T, bool FAR = false>
__device__ __forceinline__ void panel_run(const PanelSrc<T>& S, PanelRing<WD, NC, T>& R, const PanelImg& img, const WaveIters& I, const PanelSz& sz_, const PanelSzFar* far, int wave, int lane,
                                          mfma_f4 (&acc)[T]) {
    constexpr int D = PanelRing<WD, NC, T>::D, DX = PanelRing<WD, NC, T>::DX;
    static_assert(DX % D == 0 && kSzFar % DX == 0, "slots");
    lds_f16* own = (lds_f16*)sz_.lds + wave * 2 * 16 * T * kSzFar;
    int i0 = 0;
    auto bring = [&](int i) {
        i0 = i;
        panel_scales_far<T>(*far, own, lane, [&](int k) { return I.at(i + k); });
    };
    auto group = [&](int i) { return FAR ? i - i0 : I.at(i); };
    if constexpr (WD == W_INT4 && (NC <= 8 || FAR)) {
        for (int i = 0; i < I.n; i += DX) {
            if constexpr (FAR) if (i % kSzFar == 0) bring(i);
#pragma unroll
            for (int j = 0; j < DX; j++) {
                if (j > 0 && i + j >= I.n) break;
                const int nw = i + j + D, nx = i + j + DX;
                // a tile's weights are requested again right behind its products
                panel_multiply<WD, NC, T>(R, j % D, j, group(i + j), FAR ? PanelSz{own, 16 * T * kSzFar, kSzFar} : sz_, lane, acc, [&](int t) {
                    __builtin_amdgcn_sched_barrier(0);
                    R.load_wt(S, j % D, I.at(nw), t, nw < I.n);
                    __builtin_amdgcn_sched_barrier(0);
                });
                R.load_x(img, j, I.at(nx), nx < I.n);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        return;
    }
    const auto keep = [](int) {};
    int i = 0;
    for (; i + DX + D <= I.n; i += DX) {
#pragma unroll
        for (int j = 0; j < DX; j++) {
            const int nw = I.at(i + j + D), nx = I.at(i + j + DX);
            // a tile's weights are requested again right behind its products
            panel_multiply<WD, NC, T>(R, j % D, j, I.at(i + j), sz_, lane, acc, [&](int t) {
                __builtin_amdgcn_sched_barrier(0);
                R.load_wt(S, j % D, nw, t, true);
                __builtin_amdgcn_sched_barrier(0);
            });
            R.load_x(img, j, nx, true);   // (past the end: the last one again)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // fewer than DX + D iterations left
#pragma unroll
    for (int j = 0; j < DX + D - 1; j++) {
        if (i + j < I.n) {
            panel_multiply<WD, NC, T>(R, j % D, j % DX, I.at(i + j), sz_, lane, acc, keep);
            __builtin_amdgcn_sched_barrier(0);
            if (i + j + D < I.n) R.load_w(S, j % D, I.at(i + j + D), true);
            if (i + j + DX < I.n) R.load_x(img, j % DX, I.at(i + j + DX), true);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// A wave's partial tiles into LDS: [wave][tile][sequence % 4][lane] (NC = 1: the three parts in place of four sequences).
template <int T, int NC>
__device__ __forceinline__ void panel_put(lds_float* red, const mfma_f4 (&acc)[T], int wave, int lane) {
    if (NC == 1 && lane >= 16) return;
#pragma unroll
    for (int t = 0; t < T; t++)
#pragma unroll
        for (int i = 0; i < (NC == 1 ? 3 : 4); i++) red[((wave * T + t) * 4 + i) * 64 + lane] = acc[t][i];
}
// Rows 4 q .. 4 q + 3 of tile t for sequence n, summed over the waves (and over the parts of the inputs).
template <int NC, int T>
__device__ __forceinline__ f32x4 panel_get(const lds_float* red, int t, int q, int n) {
    typedef __attribute__((address_space(3))) f32x4 lds_f4;
    if constexpr (NC == 1) n = 0;
    const lds_f4* p = (const lds_f4*)(red + ((size_t)t * 4 + (n & 3)) * 64 + (n >> 2) * 16 + 4 * q);
    f32x4 v[kWideWaves];
#pragma unroll
    for (int w = 0; w < kWideWaves; w++) {
        v[w] = p[w * T * 64];
        if constexpr (NC == 8) v[w] += p[w * T * 64 + 8];   // sequence n's remainders: operand row n + 8
        if constexpr (NC == 1) v[w] += p[w * T * 64 + 16] + p[w * T * 64 + 32];   // operand rows 1 and 2
    }
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

}  // namespace ff
