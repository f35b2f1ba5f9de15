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
    __device__ __forceinline__ static PanelSrc make(const PMat& M, int p0, int r1, int lane) {
        PanelSrc S;
        const u32 rowb = (u32)M.row_bytes();
        const size_t left = (size_t)(M.n - p0) * rowb;
        S.base = __builtin_amdgcn_make_buffer_rsrc((void*)(M.w + (size_t)p0 * rowb), 0, (int)(u32)(left < 0xFFFFFFFFu ? left : 0xFFFFFFFFu), 0x00020000);
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
    static constexpr u32 kNowhere = 0x7FFFFFF0u;   // an offset behind every buffer: answered with zeros, without an access
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
// Where a wave finds a panel's int4 scales and zeros.
struct PanelSz {
    const lds_u32* lds;          // (scale | zero << 16) words, [group][16 T rows]; null: too many of them, read in place
    const PMat* M; int p0, r1;
};
template <int WD, int NC, int T, class Refill>
__device__ __forceinline__ void panel_multiply(const PanelRing<WD, NC, T>& R, int slot, int xslot, int it, const PanelSz& sz, int lane, mfma_f4 (&acc)[T], Refill&& refill) {
    constexpr int NP = kXOps<NC>;
    mfma_f4 X = {0.f, 0.f, 0.f, 0.f};
    const lds_u32* szp = nullptr;
    if constexpr (WD == W_INT4) {
        const u32x4 ones{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
        for (int i = 0; i < 4 * NP; i++) X = mfma16(R.x[xslot][i], ones, X);
        szp = sz.lds + (size_t)it * (16 * T) + (lane & 15);
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
            u32 v;
            if (T > 2 || sz.lds) v = szp[16 * t];
            else {   // (only rows much longer than their number: one or two tiles)
                const size_t e = (size_t)max(min(sz.p0 + 16 * t + (lane & 15), sz.r1 - 1), 0) * (sz.M->k / 128) + it;
                v = (u32)as_global(sz.M->s)[e] | ((u32)as_global(sz.M->z)[e] << 16);
            }
            const float s = f16_to_f((f16_t)(v & 0xFFFFu)), zp = kI4Offset + f16_to_f((f16_t)(v >> 16));
#pragma unroll
            for (int i = 0; i < 4; i++) acc[t][i] = fmaf(s, fmaf(-zp, X[i], d[i]), acc[t][i]);
        }
        refill(t);
    }
}

// int4: scales and zeros of a panel's rows, loaded as whole row slabs (contiguous) by the workgroup
// ahead of the weights and dropped into LDS behind their requests.
constexpr int kSzItems = 4;   // (row, four groups) items of one thread held in registers
template <int T>
struct PanelScales {
    u32x2 s[kSzItems], z[kSzItems];
    __device__ __forceinline__ static int items(const PMat& M, int nrows) { return nrows * ((M.k / 128 + 3) / 4); }
    // (item i: four groups of row i / q; only rows of whole items, others go word by word in store)
    __device__ __forceinline__ void load(const PMat& M, int tid, int p0, int nrows, int i0) {
        const int ng = M.k / 128, q = (ng + 3) / 4, n = nrows * q;
        if (ng & 3) return;   // (not whole 8-byte pieces: see store)
#pragma unroll
        for (int u = 0; u < kSzItems; u++) {
            const int i = min(i0 + tid + u * kWideThreads, n - 1);
            const size_t e = (size_t)p0 * ng + (size_t)i * 4;   // whole rows of whole items: contiguous
            s[u] = *as_global((const u32x2*)(M.s + e));
            z[u] = *as_global((const u32x2*)(M.z + e));
        }
    }
    __device__ __forceinline__ void store(const PMat& M, int tid, int p0, int nrows, int i0, lds_u32* sz) const {
        const int ng = M.k / 128, q = (ng + 3) / 4, n = nrows * q;
        if (ng & 3) {   // rows of a group count that is no multiple of four: one word at a time
            if (i0 == 0)
                for (int i = tid; i < nrows * ng; i += kWideThreads) {
                    const size_t e = (size_t)p0 * ng + i;
                    sz[(i % ng) * (16 * T) + i / ng] = (u32)as_global(M.s)[e] | ((u32)as_global(M.z)[e] << 16);
                }
            return;
        }
#pragma unroll
        for (int u = 0; u < kSzItems; u++) {
            const int i = i0 + tid + u * kWideThreads;
            if (i < n) {
                const int r = i / q, g = (i - r * q) * 4;
                lds_u32* p = sz + (size_t)g * (16 * T) + r;
                p[0] = (s[u].x & 0xFFFFu) | (z[u].x << 16);
                p[16 * T] = (s[u].x >> 16) | (z[u].x & 0xFFFF0000u);
                p[2 * 16 * T] = (s[u].y & 0xFFFFu) | (z[u].y << 16);
                p[3 * 16 * T] = (s[u].y >> 16) | (z[u].y & 0xFFFF0000u);
            }
        }
    }
};

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
template <int WD, int NC, int T>
__device__ __forceinline__ void panel_run(const PanelSrc<T>& S, PanelRing<WD, NC, T>& R, const PanelImg& img, const WaveIters& I, const PanelSz& sz, int lane,
                                          mfma_f4 (&acc)[T]) {
    constexpr int D = PanelRing<WD, NC, T>::D, DX = PanelRing<WD, NC, T>::DX;
    static_assert(DX % D == 0, "slots");
    if constexpr (WD == W_INT4 && NC <= 8) {
        for (int i = 0; i < I.n; i += DX) {
#pragma unroll
            for (int j = 0; j < DX; j++) {
                if (j > 0 && i + j >= I.n) break;
                const int nw = i + j + D, nx = i + j + DX;
                // a tile's weights are requested again right behind its products
                panel_multiply<WD, NC, T>(R, j % D, j, I.at(i + j), sz, lane, acc, [&](int t) {
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
            panel_multiply<WD, NC, T>(R, j % D, j, I.at(i + j), sz, lane, acc, [&](int t) {
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
            panel_multiply<WD, NC, T>(R, j % D, j % DX, I.at(i + j), sz, lane, acc, keep);
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
