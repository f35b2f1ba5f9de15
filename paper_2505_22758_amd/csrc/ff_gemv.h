// Weight-streaming GEMV engine: activation staging into LDS, a register ring of weight tiles kept
// in flight ahead of the FMAs, and the per-format dot products.  Used by the fused whole-model
// kernel (which requests a projection's first tiles before it waits for the projection's input)
// and by the per-operation baseline kernels.
#pragma once
#include "ff_device.h"

namespace ff {

template <int WD> struct WTraits;
template <> struct WTraits<W_BF16> { static constexpr int EPU = 8; };   // elements per 16-byte unit
template <> struct WTraits<W_INT8> { static constexpr int EPU = 16; };
template <> struct WTraits<W_INT4> { static constexpr int EPU = 32; };

// 16-byte units per row and pipeline stage (per lane).  A unit of int4 weights spans 32 columns, so
// four units per lane would cover 8192 columns per stage: rows of 4096 columns would leave half
// the lanes multiplying padding.  int4 stages are therefore half as wide and its ring twice as deep.
#ifndef FF_UNR
#define FF_UNR 4   // 16-byte units per row, lane and stage for bf16 / int8 weights (can be overridden at build time for sweeps)
#endif
template <int WD> constexpr int kUnrOf = WD == W_INT4 ? 2 : FF_UNR;
// Pipeline stages (register ring slots) per wave.  Two stages (16 loads of 16 bytes per lane) keep
// the memory pipe full; deeper rings measured slower in the fused kernel, because every byte
// prefetched across a projection boundary queues in front of the loads of the next input vector
// (a wave's loads return in issue order).  FF_DEPTH can be overridden at build time for sweeps.
#ifndef FF_DEPTH
#define FF_DEPTH 2
#endif
template <int WD> constexpr int kDepthOf = WD == W_INT4 ? 2 * FF_DEPTH : FF_DEPTH;
template <int WD> constexpr int kChunkUnitsOf = 64 * kUnrOf<WD>;   // units of one row covered by one stage of one wave
// Refill granularity of the streams: a ring slot is refilled in kRefillParts parts,
// each right behind the multiply-accumulates that freed its registers, so that 16 - 8 / parts of
// the wave's 16 loads stay in flight while a stage is being multiplied (8 with whole-stage refills).
#ifndef FF_REFILL_PARTS
#define FF_REFILL_PARTS 2
#endif
#ifndef FF_REFILL_PARTS_I4
#define FF_REFILL_PARTS_I4 1
#endif
template <int WD, int B> constexpr int kRefillPartsOf = B != 1 ? 1 : WD == W_INT4 ? FF_REFILL_PARTS_I4 : (kUnrOf<WD> % FF_REFILL_PARTS == 0 ? FF_REFILL_PARTS : 1);
template <int U0, int U1> struct StageUnits { static constexpr int u0 = U0, u1 = U1; };   // units [U0, U1) of a stage
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(StageUnits<I, N>{});   // (I of N: the callee derives its unit range)
        static_for<I + 1, N>(f);
    }
}
constexpr int kAccFloatsPerWave = (kLdsAuxBytes - kLdsAuxTailBytes) / 4 / kWaves;   // partial sums a wave can carry between K segments
// Arrival counters of the staged h chunks (glu_run).
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) u32 lds_u32;
__device__ __forceinline__ lds_u32* glu_counters_of(const float4* xs) {
    return (lds_u32*)((uint8_t*)xs + kLdsActBytes + kLdsAuxBytes + kLdsRopeBytes + kLdsMiscBytes);
}

// ---------------------------------------------------------------- reductions
// Sum over the 64 lanes with DPP row operations; the result is wave-uniform.
__device__ __forceinline__ float wave_sum_uniform(float v) {
    int x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
    x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
    x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true));   // row_half_mirror
    x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, true));   // row_mirror
    x = __float_as_int(v);
    float r0 = __int_as_float(__builtin_amdgcn_readlane(x, 0));
    float r1 = __int_as_float(__builtin_amdgcn_readlane(x, 16));
    float r2 = __int_as_float(__builtin_amdgcn_readlane(x, 32));
    float r3 = __int_as_float(__builtin_amdgcn_readlane(x, 48));
    return (r0 + r1) + (r2 + r3);
}

// Sum over aligned groups of W lanes (W = 8 or 16), every lane of a group receiving the group's sum:
// DPP steps inside one 16-lane row, no LDS permute traffic.
template <int W>
__device__ __forceinline__ float group_sum(float v) {
    static_assert(W == 8 || W == 16, "group width");
    int x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
    x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
    x = __float_as_int(v);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true));   // row_half_mirror
    if constexpr (W == 16) {
        x = __float_as_int(v);
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, true));   // row_mirror
    }
    return v;
}

// Maximum over aligned groups of 16 lanes, for every lane of a group.
__device__ __forceinline__ float group_max16(float v) {
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true)));
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, true)));
}

// ---------------------------------------------------------------- staging
// Where a GEMV phase takes its input vector(s) from, and what is folded into the staging.
struct ActSrc {
    const float* base = nullptr;    // fp32 exchange buffer [B][stride] ...
    size_t stride = 0;
    const bf16_t* embed = nullptr;  // ... or (tokens != null) rows of the bf16 embedding table
    const int* tokens = nullptr;
    const float* add = nullptr;     // optional second fp32 vector added element-wise (residual + sublayer output)
    size_t add_stride = 0;
    float* wb = nullptr;            // optional: the summed, un-normalised vector is written back here,
    size_t wb_stride = 0;           //   each workgroup storing an interleaved slice
    const bf16_t* gain = nullptr;   // non-null: RMSNorm with this gain is applied while staging
    float eps = 0.f;
};

// Stage elements [k0, k0 + nunits*EPU) of every batch row into LDS, quad-planar so that a wave's
// 64 lanes read 64 consecutive float4: quad qd of unit j of row b lives at xs[(b*NQ + qd)*nup + j].
// Units [nunits, nup) are zero filled (the weight stream reads clamped addresses there).  With a
// gain, RMSNorm (paper Section 2.1: pre-RMSNorm in front of the QKV and GLU in/gate projections) is
// applied; that needs k0 == 0 and the whole row.  NT threads take part (tid in [0, NT)): 64 = one
// wave (reduction by DPP), otherwise the whole workgroup (reduction through `red` in LDS, with
// __syncthreads).  All global loads of a batch of kStageBatch quads per thread are issued before any
// is used.  The caller synchronises before the staged vector is read.
constexpr int kStageBatch = 8;
template <int EPU, class IO, int NT>
__device__ void stage_act(const ActSrc& S, int batch, int K, int k0, int nunits, int nup, float4* xs, float* red, int tid) {
    constexpr int NQ = EPU / 4;
    const int nquads = nunits * NQ;
    const int padquads = nup * NQ;
    for (int b = 0; b < batch; b++) {
        float4* xb = xs + (size_t)b * NQ * nup;
        const float* src = S.base + (size_t)b * S.stride;
        const float* add = S.add ? S.add + (size_t)b * S.add_stride : nullptr;
        const bf16_t* erow = S.tokens ? S.embed + (size_t)max(as_global(S.tokens)[b], 0) * K : nullptr;
        float ss = 0.f;
        for (int q0 = tid; q0 < padquads; q0 += NT * kStageBatch) {
            float4 v[kStageBatch], a[kStageBatch];
            u32x2 g[kStageBatch];
#pragma unroll
            for (int u = 0; u < kStageBatch; u++) {
                int qi = min(q0 + u * NT, nquads - 1);   // clamped: the load is always issued
                int k = k0 + qi * 4;
                if (erow) {
                    u32x2 w = *as_global((const u32x2*)(erow + k));
                    v[u] = make_float4(bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y));
                } else {
                    v[u] = IO::ld4(src, k);
                }
                if (add) a[u] = IO::ld4(add, k);
                if (S.gain) g[u] = *as_global((const u32x2*)(S.gain + k));
            }
#pragma unroll
            for (int u = 0; u < kStageBatch; u++) {
                int qi = q0 + u * NT;
                if (qi < padquads) {
                    float4 t = v[u];
                    if (add) { t.x += a[u].x; t.y += a[u].y; t.z += a[u].z; t.w += a[u].w; }
                    if (qi >= nquads) t = make_float4(0.f, 0.f, 0.f, 0.f);
                    else if (S.wb && (qi % (int)gridDim.x) == (int)blockIdx.x) IO::st4(S.wb + (size_t)b * S.wb_stride + k0 + qi * 4, t);
                    if (S.gain && qi < nquads) {
                        ss += t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
                        t.x *= bf_lo(g[u].x); t.y *= bf_hi(g[u].x); t.z *= bf_lo(g[u].y); t.w *= bf_hi(g[u].y);
                    }
                    xb[(size_t)(qi % NQ) * nup + qi / NQ] = t;
                }
            }
        }
        if (S.gain) {
            float tot;
            if constexpr (NT == 64) {
                tot = wave_sum_uniform(ss);
            } else {
                ss = wave_sum_uniform(ss);
                __syncthreads();
                if ((tid & 63) == 0) red[tid >> 6] = ss;
                __syncthreads();
                tot = 0.f;
#pragma unroll
                for (int w = 0; w < NT / 64; w++) tot += red[w];
            }
            float r = 1.0f / sqrtf(tot / (float)K + S.eps);
            for (int qi = tid; qi < nquads; qi += NT) {   // each thread rescales the quads it wrote
                int j = qi / NQ, qd = qi % NQ;
                float4 v = xb[(size_t)qd * nup + j];
                v.x *= r; v.y *= r; v.z *= r; v.w *= r;
                xb[(size_t)qd * nup + j] = v;
            }
        }
    }
}

// ---------------------------------------------------------------- one stage of weights
template <int WD> struct Stage {
    u32x4 w[2][kUnrOf<WD>];
};
template <> struct Stage<W_INT8> {
    u32x4 w[2][kUnrOf<W_INT8>];
    u32 rs[2];                 // raw fp16 row scales (loaded with the row's last chunk)
};
template <> struct Stage<W_INT4> {
    u32x4 w[2][kUnrOf<W_INT4>];
    u32 s[2][kUnrOf<W_INT4>], z[2][kUnrOf<W_INT4>];   // raw fp16 group scale / zero of each unit
};

__device__ __forceinline__ float dot_bf16(const u32x4& w, const float4& a, const float4& b, float acc) {
    acc = fmaf(bf_lo(w.x), a.x, acc);
    acc = fmaf(bf_hi(w.x), a.y, acc);
    acc = fmaf(bf_lo(w.y), a.z, acc);
    acc = fmaf(bf_hi(w.y), a.w, acc);
    acc = fmaf(bf_lo(w.z), b.x, acc);
    acc = fmaf(bf_hi(w.z), b.y, acc);
    acc = fmaf(bf_lo(w.w), b.z, acc);
    acc = fmaf(bf_hi(w.w), b.w, acc);
    return acc;
}
__device__ __forceinline__ float dot_i8x4(u32 w, const float4& x, float acc) {
    acc = fmaf((float)(int)(int8_t)(w), x.x, acc);
    acc = fmaf((float)(int)(int8_t)(w >> 8), x.y, acc);
    acc = fmaf((float)(int)(int8_t)(w >> 16), x.z, acc);
    acc = fmaf((float)((int)w >> 24), x.w, acc);
    return acc;
}
// int4 group-128: a 16-byte unit holds 32 codes of ONE group, so its contribution is
//   sum_i (code_i - z) s x_i  =  s (sum_i code_i x_i  -  z sum_i x_i):
// the inner loop only converts codes and multiplies (about 2.4 operations per weight); scale and
// zero are applied once per unit.  Even codes of a word are isolated with one mask, odd ones with a
// shift and the same mask, and the byte-to-float conversions pick them up.
__device__ __forceinline__ float dot_i4x8_codes(u32 w, const float4& x0, const float4& x1, float acc) {
    u32 e = w & 0x0F0F0F0Fu, o = (w >> 4) & 0x0F0F0F0Fu;
    // value barriers (no instruction): keep the compiler from folding the masks back into one
    // bit-field extract per code, which would cost an extra operation per weight
    asm("" : "+v"(e));
    asm("" : "+v"(o));
    acc = fmaf((float)(e & 0xFFu), x0.x, acc);
    acc = fmaf((float)(o & 0xFFu), x0.y, acc);
    acc = fmaf((float)((e >> 8) & 0xFFu), x0.z, acc);
    acc = fmaf((float)((o >> 8) & 0xFFu), x0.w, acc);
    acc = fmaf((float)((e >> 16) & 0xFFu), x1.x, acc);
    acc = fmaf((float)((o >> 16) & 0xFFu), x1.y, acc);
    acc = fmaf((float)(e >> 24), x1.z, acc);
    acc = fmaf((float)(o >> 24), x1.w, acc);
    return acc;
}
__device__ __forceinline__ float sum4(const float4& v) { return (v.x + v.y) + (v.z + v.w); }

// Division by a launch constant (waves or workgroups in the grid) that is a power of two on the
// usual 256-workgroup launch: a shift there, a division otherwise.  It sits on the path between two
// projections, where a 32-bit division is a thirty-instruction sequence.
struct UDiv {
    u32 n; int sh;   // sh >= 0: n == 1 << sh
    __device__ __forceinline__ static UDiv of(u32 n) { return UDiv{n, (n & (n - 1)) == 0 ? (int)__builtin_ctz(n) : -1}; }
    __device__ __forceinline__ u32 div(u32 x) const { return sh >= 0 ? x >> sh : x / n; }
    __device__ __forceinline__ u32 mod(u32 x) const { return sh >= 0 ? x & (n - 1) : x % n; }
};

// ---------------------------------------------------------------- per-wave view of one GEMV
// A projection is cut along K into segments whose staged input fits the LDS activation region
// (one segment except for the widest inputs at batch 4); along N every wave of the grid owns a
// contiguous range of row pairs.  All fields are wave-uniform.
template <int WD, int B>
struct Stream {
    const uint8_t* w; const f16_t* s; const f16_t* z;
    size_t rowb;
    int N, K, ng;
    int nseg, seg, j0, nunits, cpr, nup;
    int p0, n_it;   // first row pair, iterations

    static constexpr int EPU = WTraits<WD>::EPU;
    static constexpr int kChunkUnits = kChunkUnitsOf<WD>;
    static constexpr int seg_units = (kLdsActBytes / (B * EPU * 4)) / kChunkUnits * kChunkUnits;

    __device__ __forceinline__ static Stream make(const PMat& M, int seg, int gwave, const UDiv& n_gwaves) {
        Stream S;
        S.w = M.w; S.s = M.s; S.z = M.z; S.N = M.n; S.K = M.k; S.ng = M.k / 128;
        S.rowb = WD == W_BF16 ? (size_t)M.k * 2 : WD == W_INT8 ? (size_t)M.k : (size_t)M.k / 2;
        const int total_units = M.k / EPU;
        S.nseg = (total_units + seg_units - 1) / seg_units;
        S.seg = seg;
        S.j0 = seg * seg_units;
        S.nunits = min(seg_units, total_units - S.j0);
        S.nup = (S.nunits + kChunkUnits - 1) / kChunkUnits * kChunkUnits;
        S.cpr = S.nup / kChunkUnits;
        // row pairs [p0, p1) of this wave; the products fit 32 bits (rows * waves < 2^32)
        const u32 npairs = (u32)(M.n + 1) / 2;
        S.p0 = (int)n_gwaves.div(npairs * (u32)gwave);
        S.n_it = ((int)n_gwaves.div(npairs * (u32)(gwave + 1)) - S.p0) * S.cpr;
        return S;
    }
};

// Issue the loads of iteration (pair, chunk).  Every load is issued unconditionally from a clamped
// address: out-of-range units meet zeros in the staged input, out-of-range rows are dropped by the
// epilogue.  Nothing is converted here, so no load result is waited for at issue time.
template <int WD, int B, int U0 = 0, int U1 = kUnrOf<WD>>
__device__ __forceinline__ void load_stage(const Stream<WD, B>& S, int pair, int chunk, Stage<WD>& st, int lane) {
    constexpr int kUnr = kUnrOf<WD>;
#pragma unroll
    for (int u = U0; u < U1; u++) {
        const int j = min((chunk * kUnr + u) * 64 + lane, S.nunits - 1);
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const int row = min(2 * pair + r, S.N - 1);
            st.w[r][u] = ldg_stream(S.w + (size_t)row * S.rowb + (size_t)(S.j0 + j) * 16);
            if constexpr (WD == W_INT4) {
                const size_t gi = (size_t)row * S.ng + (S.j0 + j) / 4;
                st.s[r][u] = as_global(S.s)[gi];
                st.z[r][u] = as_global(S.z)[gi];
            }
        }
    }
    if constexpr (WD == W_INT8 && U1 == kUnr) {
        if (chunk == S.cpr - 1) {
            st.rs[0] = as_global(S.s)[min(2 * pair, S.N - 1)];
            st.rs[1] = as_global(S.s)[min(2 * pair + 1, S.N - 1)];
        }
    }
}

// Issue iterations [s0, min(s1, n_it)) of a stream into ring slots of the same index (by default the
// whole ring: the first min(kDepth, n_it) iterations).
// FF_PREFETCH_STAGES: how many of them the fused kernel requests BEFORE it waits for a projection's
// input (what is requested across a hand-over queues in front of the input's loads); the rest of the
// ring is requested once the input is there.
#ifndef FF_PREFETCH_STAGES
#define FF_PREFETCH_STAGES FF_DEPTH
#endif
template <int WD> constexpr int kPrefetchOf = (WD == W_INT4 ? 2 : 1) * (FF_PREFETCH_STAGES < FF_DEPTH ? FF_PREFETCH_STAGES : FF_DEPTH);
template <int WD, int B>
__device__ __forceinline__ void prefetch_stream(const Stream<WD, B>& S, Stage<WD> (&ring)[kDepthOf<WD>], int lane, int s0 = 0, int s1 = kDepthOf<WD>) {
    constexpr int kDepth = kDepthOf<WD>;
    int pair = S.p0, chunk = 0;
#pragma unroll
    for (int s = 0; s < kDepth; s++) {
        if (s >= s0 && s < s1 && s < S.n_it) load_stage(S, pair, chunk, ring[s], lane);
        if (++chunk == S.cpr) { chunk = 0; ++pair; }
    }
}

// The multiply-accumulates of one stage: chunk cc of a row pair against the staged input.
template <int WD, int B, int U0 = 0, int U1 = kUnrOf<WD>>
__device__ __forceinline__ void stage_fma(const Stage<WD>& st, const float4* xs, int nup, int cc, int lane, float (&acc)[2][B]) {
    constexpr int kUnr = kUnrOf<WD>;
    constexpr int NQ = WTraits<WD>::EPU / 4;
#pragma unroll
    for (int u = U0; u < U1; u++) {
        const int j = (cc * kUnr + u) * 64 + lane;
#pragma unroll
        for (int b = 0; b < B; b++) {
            const float4* xq = xs + (size_t)b * NQ * nup + j;
            if constexpr (WD == W_BF16) {
                float4 x0 = xq[0], x1 = xq[nup];
                acc[0][b] = dot_bf16(st.w[0][u], x0, x1, acc[0][b]);
                acc[1][b] = dot_bf16(st.w[1][u], x0, x1, acc[1][b]);
            } else if constexpr (WD == W_INT8) {
                float4 x0 = xq[0], x1 = xq[nup], x2 = xq[2 * nup], x3 = xq[3 * nup];
#pragma unroll
                for (int r = 0; r < 2; r++) {
                    float a = acc[r][b];
                    a = dot_i8x4(st.w[r][u].x, x0, a); a = dot_i8x4(st.w[r][u].y, x1, a);
                    a = dot_i8x4(st.w[r][u].z, x2, a); a = dot_i8x4(st.w[r][u].w, x3, a);
                    acc[r][b] = a;
                }
            } else {
                float4 x[8];
#pragma unroll
                for (int q = 0; q < 8; q++) x[q] = xq[q * nup];
                const float xsum = ((sum4(x[0]) + sum4(x[1])) + (sum4(x[2]) + sum4(x[3]))) + ((sum4(x[4]) + sum4(x[5])) + (sum4(x[6]) + sum4(x[7])));
#pragma unroll
                for (int r = 0; r < 2; r++) {
                    const float sc = f16_to_f((f16_t)st.s[r][u]), zp = f16_to_f((f16_t)st.z[r][u]);
                    float t = dot_i4x8_codes(st.w[r][u].x, x[0], x[1], 0.f);
                    t = dot_i4x8_codes(st.w[r][u].y, x[2], x[3], t);
                    t = dot_i4x8_codes(st.w[r][u].z, x[4], x[5], t);
                    t = dot_i4x8_codes(st.w[r][u].w, x[6], x[7], t);
                    acc[r][b] = fmaf(sc, fmaf(-zp, xsum, t), acc[r][b]);
                }
            }
        }
    }
}

// The staged inputs of a whole stage read from LDS ahead of its multiply-accumulates (single
// sequence): with one wave per SIMD nothing else hides the latency of an LDS read,
// and a read issued right in front of its use costs that latency once per unit.  With
// FF_X_PRELOAD the reads of all units of a stage (int8: of a part) are issued when its first part
// (the part) starts (8B bf16, batch 1: 2968 -> 2946 us per step; issuing them a whole stage ahead
// gained nothing further).
#ifndef FF_X_PRELOAD
#define FF_X_PRELOAD 1
#endif
#ifndef FF_X_PRELOAD_I4
#define FF_X_PRELOAD_I4 1   // int4: both units of a stage (8B int4, batch 1: 2395 -> 2384 us per step)
#endif
template <int WD, int B> constexpr bool kXPreloadOf = FF_X_PRELOAD && (WD == W_BF16 || WD == W_INT8 || (WD == W_INT4 && FF_X_PRELOAD_I4)) && B == 1;
template <int WD> constexpr int kXQuadsOf = WTraits<WD>::EPU / 4;   // float4 reads per unit (bf16: 2, int8: 4)
// Units [U0, U1) of a stage: bf16 reads the whole stage's inputs with its first part (16 registers per
// part), int8 each part's inputs when the part starts (its units are twice as wide).
template <int WD, int U0, int U1>
__device__ __forceinline__ void stage_x_load(const float4* xs, int nup, int cc, int lane, float4 (&xr)[kUnrOf<WD>][kXQuadsOf<WD>]) {
    constexpr int kUnr = kUnrOf<WD>, NX = kXQuadsOf<WD>;
    constexpr int L0 = WD == W_INT8 ? U0 : 0, L1 = WD == W_INT8 ? U1 : (U0 == 0 ? kUnr : 0);   // int4 (whole-stage parts only): like bf16
#pragma unroll
    for (int u = L0; u < L1; u++) {
        const float4* xq = xs + (cc * kUnr + u) * 64 + lane;
#pragma unroll
        for (int q = 0; q < NX; q++) xr[u][q] = xq[q * nup];
    }
}
template <int WD, int U0, int U1>
__device__ __forceinline__ void stage_fma_x(const Stage<WD>& st, const float4 (&xr)[kUnrOf<WD>][kXQuadsOf<WD>], float (&acc)[2][1]) {
#pragma unroll
    for (int u = U0; u < U1; u++) {
        if constexpr (WD == W_BF16) {
            acc[0][0] = dot_bf16(st.w[0][u], xr[u][0], xr[u][1], acc[0][0]);
            acc[1][0] = dot_bf16(st.w[1][u], xr[u][0], xr[u][1], acc[1][0]);
        } else if constexpr (WD == W_INT8) {
#pragma unroll
            for (int r = 0; r < 2; r++) {
                float a = acc[r][0];
                a = dot_i8x4(st.w[r][u].x, xr[u][0], a); a = dot_i8x4(st.w[r][u].y, xr[u][1], a);
                a = dot_i8x4(st.w[r][u].z, xr[u][2], a); a = dot_i8x4(st.w[r][u].w, xr[u][3], a);
                acc[r][0] = a;
            }
        } else {
            const float4 (&x)[8] = xr[u];
            const float xsum = ((sum4(x[0]) + sum4(x[1])) + (sum4(x[2]) + sum4(x[3]))) + ((sum4(x[4]) + sum4(x[5])) + (sum4(x[6]) + sum4(x[7])));
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const float sc = f16_to_f((f16_t)st.s[r][u]), zp = f16_to_f((f16_t)st.z[r][u]);
                float t = dot_i4x8_codes(st.w[r][u].x, x[0], x[1], 0.f);
                t = dot_i4x8_codes(st.w[r][u].y, x[2], x[3], t);
                t = dot_i4x8_codes(st.w[r][u].z, x[4], x[5], t);
                t = dot_i4x8_codes(st.w[r][u].w, x[6], x[7], t);
                acc[r][0] = fmaf(sc, fmaf(-zp, xsum, t), acc[r][0]);
            }
        }
    }
}

// Weight-streaming GEMV over one stream for up to B batch rows (paper Section 4.2: batch-one
// projections are matrix-vector products with the input cached on chip and each workgroup owning
// some rows of W; Section 5.2: for a few rows the weights are still read exactly once and the inputs
// replicated, which the per-operation path does).  On entry ring[s] holds iteration s (s < min(kDepth, n_it)); iteration i+kDepth is
// issued into the slot iteration i has just freed, so 2*kDepth*kUnr 16-byte non-temporal loads
// per lane stay in flight across row boundaries.  epi(pair, b, v0, v1) runs on lane 0 with the two
// finished dot products of rows (2*pair, 2*pair+1); partial sums of earlier K segments are carried
// in `myacc` (LDS, private to the wave).
template <int WD, int B, class Epi>
__device__ __forceinline__ void gemv_run(const Stream<WD, B>& S, Stage<WD> (&ring)[kDepthOf<WD>], const float4* xs, float* myacc,
                                         int batch, int lane, Epi& epi) {
    constexpr int kDepth = kDepthOf<WD>;
    const int nup = S.nup;
    float acc[2][B];
#pragma unroll
    for (int b = 0; b < B; b++) acc[0][b] = acc[1][b] = 0.f;
    int pc = S.p0, cc = 0;          // (pair, chunk) of the next compute
    int pl = S.p0, cl = 0;          // (pair, chunk) of the next load = iteration kDepth
    for (int s = 0; s < kDepth; s++) if (++cl == S.cpr) { cl = 0; ++pl; }

    constexpr int kUnr = kUnrOf<WD>, kParts = kRefillPartsOf<WD, B>;
    float4 xr[kUnr][kXQuadsOf<WD>];   // (kXPreloadOf) the stage's inputs, read ahead of their multiply-accumulates
    auto compute = [&](const Stage<WD>& st, auto units) {   // units: the StageUnits range multiplied by this call; the last one finishes the iteration
        constexpr int U0 = decltype(units)::u0, U1 = decltype(units)::u1;
        if constexpr (kXPreloadOf<WD, B>) {
            stage_x_load<WD, U0, U1>(xs, nup, cc, lane, xr);
            stage_fma_x<WD, U0, U1>(st, xr, acc);
        } else stage_fma<WD, B, U0, U1>(st, xs, nup, cc, lane, acc);
        if constexpr (U1 < kUnr) return;
        if (cc == S.cpr - 1) {   // row pair finished (for this K segment)
            const int lp = pc - S.p0;
#pragma unroll
            for (int b = 0; b < B; b++) {
                float v0 = wave_sum_uniform(acc[0][b]), v1 = wave_sum_uniform(acc[1][b]);
                acc[0][b] = acc[1][b] = 0.f;
                if constexpr (WD == W_INT8) { v0 *= f16_to_f((f16_t)st.rs[0]); v1 *= f16_to_f((f16_t)st.rs[1]); }
                if (lane == 0 && b < batch) {
                    if (S.nseg > 1) {
                        float* a = myacc + ((size_t)lp * B + b) * 2;
                        if (S.seg > 0) { v0 += a[0]; v1 += a[1]; }
                        if (S.seg < S.nseg - 1) { a[0] = v0; a[1] = v1; }
                    }
                    if (S.seg == S.nseg - 1) epi(pc, b, v0, v1);
                }
            }
        }
        if (++cc == S.cpr) { cc = 0; ++pc; }
    };
    auto load = [&](Stage<WD>& st, auto units) {
        constexpr int U0 = decltype(units)::u0, U1 = decltype(units)::u1;
        load_stage<WD, B, U0, U1>(S, pl, cl, st, lane);
        if constexpr (U1 < kUnr) return;
        if (++cl == S.cpr) { cl = 0; ++pl; }
    };
    int it = 0;
    // steady state: every slot is consumed and refilled
    for (; it + 2 * kDepth <= S.n_it; it += kDepth) {
#pragma unroll
        for (int s = 0; s < kDepth; s++) {
            // keep the instruction scheduler from hoisting a slot's refill above the FMAs that
            // still read the slot: that doubles the live tile registers and ends in spills
            static_for<0, kParts>([&](auto part) {
                constexpr int P = decltype(part)::u0;
                typedef StageUnits<P * kUnr / kParts, (P + 1) * kUnr / kParts> Units;
                compute(ring[s], Units{});
                __builtin_amdgcn_sched_barrier(0);
                load(ring[s], Units{});
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    }
    // tail
    for (; it < S.n_it; it += kDepth) {
#pragma unroll
        for (int s = 0; s < kDepth; s++) {
            if (it + s < S.n_it) {
                compute(ring[s], StageUnits<0, kUnr>{});
                __builtin_amdgcn_sched_barrier(0);
                if (it + s + kDepth < S.n_it) load(ring[s], StageUnits<0, kUnr>{});
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

typedef short mfma_s4 __attribute__((ext_vector_type(4)));
typedef float mfma_f4 __attribute__((ext_vector_type(4)));

}  // namespace ff
