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
//   * lane (r = lane % 16, g = lane / 16) loads 16 bytes of weight row r per load; the accumulators of
//     lane (r, g) hold row r for sequences 4 g .. 4 g + 3, so what belongs to a weight row (int4
//     scales and zeros) belongs to the lane that loaded the row;
//   * a wave keeps D iterations of weights (and of the inputs they meet) in flight in a register ring
//     whose refills run unconditionally; the last D iterations are peeled off the loop (where code
//     paths that issued different numbers of loads meet, the compiler waits for all of them);
//   * the waves' partial tiles meet in LDS, wave t adds and finishes tile t.
// Two waves per SIMD: the eight waves' rings hold up to 128 KB per compute unit in flight, and one
// wave's conversions overlap the other's matrix-core work.
//
// Inputs are bf16 head + bf16 remainder (17 significant bits).  NC = 16: heads and remainders are
// separate operands, 16 sequences per tile.  NC = 8: rows 0..7 of the operand are the heads and rows
// 8..15 the remainders of 8 sequences, i.e. one multiplication and half the input bytes per k-step;
// the two halves of the result are added when the waves' partial tiles meet.
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
// Ring depth in iterations: what about 144 registers hold, at least two.
template <int WD, int NC, int T> constexpr int kWDepth = [] {
    const int regs = 4 * (T * kWLoads<WD> + kWSteps<WD> * (NC / 8)), d = (WD == W_INT4 && T >= 4 ? 112 : 144) / regs;
    return d < 2 ? 2 : d > 6 ? 6 : d;
}();

// Rows [own0, own1) of a projection that this workgroup computes: whole groups of four.
struct RowRange { int r0, r1; };
__device__ __forceinline__ RowRange wide_rows(int n, const UDiv& n_ctas) {
    const u32 ngroups = (u32)(n + 3) / 4;
    return RowRange{4 * (int)n_ctas.div(ngroups * blockIdx.x), min(4 * (int)n_ctas.div(ngroups * (blockIdx.x + 1)), n)};
}

// One panel's weights as a wave sees them.
template <int WD, int T>
struct PanelSrc {
    const uint8_t* base;   // first row of the panel (uniform)
    u32 row[T];            // byte offset of this lane's row of tile t (rows past the end repeat the last one)
    int units;             // 16-byte units per row
    __device__ __forceinline__ static PanelSrc make(const PMat& M, int p0, int r1, int lane) {
        PanelSrc S;
        const u32 rowb = (u32)M.row_bytes();
        S.base = M.w + (size_t)p0 * rowb;
        S.units = (int)(rowb >> 4);
#pragma unroll
        for (int t = 0; t < T; t++) S.row[t] = (u32)(max(min(p0 + 16 * t + (lane & 15), r1 - 1), p0) - p0) * rowb;
        return S;
    }
};

template <int WD, int NC, int T>
struct PanelRing {
    static constexpr int D = kWDepth<WD, NC, T>, L = kWLoads<WD>, NB = kWSteps<WD> * (NC / 8);
    u32x4 w[D][T][L];
    u32x4 x[D][NB];
    // (Cacheable loads: a load takes 64 bytes of each of 16 rows, and the other half of the 128-byte lines follows in the
    // next load or in the neighbouring wave's.  As streaming loads, 8B bf16 x 8: 2206 instead of 2004 us a pass.)
    // Weights of iteration it (columns past the end of a row repeat its last unit and meet zeros in the image).
    __device__ __forceinline__ void load_w(const PanelSrc<WD, T>& S, int slot, int it, int lane) {
        u32 col[L];
#pragma unroll
        for (int l = 0; l < L; l++) col[l] = (u32)min((it * L + l) * 4 + (lane >> 4), S.units - 1) * 16u;
#pragma unroll
        for (int t = 0; t < T; t++)
#pragma unroll
            for (int l = 0; l < L; l++) w[slot][t][l] = *as_global((const u32x4*)(S.base + (S.row[t] + col[l])));
    }
    // Inputs of iteration it.  (Buffer loads: base and iteration are scalar operands, the lane's offset one register.)
    __device__ __forceinline__ void load_x(__amdgpu_buffer_rsrc_t img, int slot, int it, int lane) {
#pragma unroll
        for (int k = 0; k < kWSteps<WD>; k++)
#pragma unroll
            for (int h = 0; h < NC / 8; h++)
                x[slot][k * (NC / 8) + h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(img, lane * 16 + h * 1024, (it * kWSteps<WD> + k) * kWideStepBytes, 0));
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
// Eight int4 codes n as the bf16 numbers 128 + n (0x4300 | n), in column order.
__device__ __forceinline__ u32x4 i4_to_bf16(u32 w) {
    const u32 e = w & 0x0F0F0F0Fu, o = (w >> 4) & 0x0F0F0F0Fu;   // codes 0,2,4,6 / 1,3,5,7 as bytes
    return u32x4{__builtin_amdgcn_perm(o, e, 0x0c040c00u) | 0x43004300u, __builtin_amdgcn_perm(o, e, 0x0c050c01u) | 0x43004300u,
                 __builtin_amdgcn_perm(o, e, 0x0c060c02u) | 0x43004300u, __builtin_amdgcn_perm(o, e, 0x0c070c03u) | 0x43004300u};
}

// acc[t] += (inputs of iteration it) x (weights of tile t).
// int8: a lane's 16 codes are two k-steps; the row scales multiply the finished sums.
// int4 group-128: an iteration is one group; with the codes n as 128 + n the four k-steps yield
// d = sum (128 + n) x, and with X = sum x of the group (the same instruction with a weight operand of ones)
//     sum s (n - z) x  =  s (d - (128 + z) X).
// sz: this panel's (scale | zero << 16) words in LDS, [group][16 T rows].
template <int WD, int NC, int T>
__device__ __forceinline__ void panel_multiply(const PanelRing<WD, NC, T>& R, int slot, int it, const lds_u32* sz, int lane, mfma_f4 (&acc)[T]) {
    constexpr int NP = NC / 8;
    if constexpr (WD == W_BF16) {
#pragma unroll
        for (int k = 0; k < 2; k++)
#pragma unroll
            for (int h = 0; h < NP; h++)
#pragma unroll
                for (int t = 0; t < T; t++) acc[t] = mfma16(R.x[slot][k * NP + h], R.w[slot][t][k], acc[t]);
    } else if constexpr (WD == W_INT8) {
#pragma unroll
        for (int t = 0; t < T; t++) {
            const u32x4 w = R.w[slot][t][0];
            const u32x4 b0 = i8_to_bf16(w.x, w.y), b1 = i8_to_bf16(w.z, w.w);
#pragma unroll
            for (int h = 0; h < NP; h++) acc[t] = mfma16(R.x[slot][h], b0, acc[t]);
#pragma unroll
            for (int h = 0; h < NP; h++) acc[t] = mfma16(R.x[slot][NP + h], b1, acc[t]);
        }
    } else {
        const u32x4 ones{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
        mfma_f4 X = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4 * NP; i++) X = mfma16(R.x[slot][i], ones, X);
        const lds_u32* szp = sz + (size_t)it * (16 * T) + (lane & 15);
#pragma unroll
        for (int t = 0; t < T; t++) {
            const u32x4 w = R.w[slot][t][0];
            const u32 ww[4] = {w.x, w.y, w.z, w.w};
            mfma_f4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const u32x4 b = i4_to_bf16(ww[q]);
#pragma unroll
                for (int h = 0; h < NP; h++) d = mfma16(R.x[slot][q * NP + h], b, d);
            }
            const u32 v = szp[16 * t];
            const float s = f16_to_f((f16_t)(v & 0xFFFFu)), zp = 128.f + f16_to_f((f16_t)(v >> 16));
#pragma unroll
            for (int i = 0; i < 4; i++) acc[t][i] = fmaf(s, fmaf(-zp, X[i], d[i]), acc[t][i]);
        }
    }
}

// int4: scales and zeros of a panel's rows, loaded as whole row slabs (contiguous) by the workgroup
// ahead of the weights and dropped into LDS behind their requests.
constexpr int kSzItems = 4;   // (row, four groups) items of one thread held in registers
template <int T>
struct PanelScales {
    u32x2 s[kSzItems], z[kSzItems];
    __device__ __forceinline__ static int items(const PMat& M, int nrows) { return nrows * ((M.k / 128 + 3) / 4); }
    // (row, first group) of item i; a row's last item starts four groups from its end, so that it never reads past it
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

// A wave's iterations of a panel: every eighth one (the workgroup's waves together read contiguous
// pieces of each row), starting at a place that differs from workgroup to workgroup (rows are a power
// of two apart at the usual widths: in step, all workgroups would read from a few memory channels).
struct WaveIters {
    int n, first, rot;
    __device__ __forceinline__ static WaveIters of(int ni, int wave) {
        WaveIters I;
        I.n = (ni - wave + kWideWaves - 1) / kWideWaves;
        I.first = I.n > 0 ? wave : 0;
        I.rot = (int)(((u32)blockIdx.x * (u32)I.n >> 8) % (u32)max(I.n, 1));
        return I;
    }
    // iteration number i (in the wave's order) as an iteration of the panel; past the end: the last one again
    __device__ __forceinline__ int at(int i) const {
        int c = min(i, n - 1) + rot;
        if (c >= n) c -= n;
        return max(c, 0) * kWideWaves + first;
    }
};

// The wave's iterations of a panel; the ring's first D slots of weights and inputs have been
// requested (slots past the end hold repeats).
template <int WD, int NC, int T>
__device__ __forceinline__ void panel_run(const PanelSrc<WD, T>& S, PanelRing<WD, NC, T>& R, __amdgpu_buffer_rsrc_t img, const WaveIters& I, const lds_u32* sz, int lane,
                                          mfma_f4 (&acc)[T]) {
    constexpr int D = PanelRing<WD, NC, T>::D;
    int i = 0;
    for (; i + 2 * D <= I.n; i += D) {
#pragma unroll
        for (int j = 0; j < D; j++) {
            panel_multiply<WD, NC, T>(R, j, I.at(i + j), sz, lane, acc);
            __builtin_amdgcn_sched_barrier(0);
            const int nx = I.at(i + D + j);
            R.load_w(S, j, nx, lane);
            R.load_x(img, j, nx, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // fewer than 2 D iterations left: slot j holds iteration i + j
#pragma unroll
    for (int j = 0; j < D; j++) {
        if (i + j < I.n) {
            panel_multiply<WD, NC, T>(R, j, I.at(i + j), sz, lane, acc);
            __builtin_amdgcn_sched_barrier(0);
            if (i + D + j < I.n) {
                const int nx = I.at(i + D + j);
                R.load_w(S, j, nx, lane);
                R.load_x(img, j, nx, lane);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int j = 0; j < D - 1; j++)
        if (i + D + j < I.n) panel_multiply<WD, NC, T>(R, j, I.at(i + D + j), sz, lane, acc);
}

// A wave's partial tiles into LDS: [wave][tile][sequence % 4][lane].
template <int T>
__device__ __forceinline__ void panel_put(lds_float* red, const mfma_f4 (&acc)[T], int wave, int lane) {
#pragma unroll
    for (int t = 0; t < T; t++)
#pragma unroll
        for (int i = 0; i < 4; i++) red[((wave * T + t) * 4 + i) * 64 + lane] = acc[t][i];
}
// Rows 4 q .. 4 q + 3 of tile t for sequence n, summed over the waves (and over heads and remainders).
template <int NC, int T>
__device__ __forceinline__ f32x4 panel_get(const lds_float* red, int t, int q, int n) {
    typedef __attribute__((address_space(3))) f32x4 lds_f4;
    const lds_f4* p = (const lds_f4*)(red + ((size_t)t * 4 + (n & 3)) * 64 + (n >> 2) * 16 + 4 * q);
    f32x4 v[kWideWaves];
#pragma unroll
    for (int w = 0; w < kWideWaves; w++) {
        v[w] = p[w * T * 64];
        if constexpr (NC == 8) v[w] += p[w * T * 64 + 8];   // sequence n's remainders: operand row n + 8
    }
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

}  // namespace ff
