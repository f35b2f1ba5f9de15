// Split-KV attention and the projection epilogues of the decode step.  Workgroup-collective
// device functions used by the fused kernel (ordered by tagged dataflow) and, with launch
// boundaries as the ordering, by the per-operation baseline kernels.
#pragma once
#include <type_traits>
#include "ff_gemv.h"

namespace ff {

// ---------------------------------------------------------------- tagged exchange format
// Inside the fused kernel the small exchanged values (queries, the step's own k and v, attention
// partials) travel as 8-byte pairs (fp32 bits, tag) written with one coherent 8-byte store; the big
// vectors use the compact format further down.  The tag names the phase instance that
// produced the value (it grows monotonically over phases and over decode steps), so a consumer can
// tell from the data itself whether its producer has run: it simply re-reads until every tag it
// needs matches.  Dependencies are thereby resolved by dataflow -- no device-wide barrier, no
// waiting for store acknowledgements -- and a vector is on the critical path for one store->load
// hop only (paper Section 4.1 needs a fence + global barrier on its hardware for the same RAW hazard).
#ifndef FF_TLD_AUX
#define FF_TLD_AUX 17   /* sc0 | sc1 */
#endif
typedef u32x2 tagged_t;
constexpr int kPollLanes = 8;
__device__ __forceinline__ void tst(tagged_t* p, float v, u32 tag) { xst2((float*)p, v, __uint_as_float(tag)); }
__device__ __forceinline__ void tst2(tagged_t* p, float v0, float v1, u32 tag) {
    tst(p, v0, tag);
    tst(p + 1, v1, tag);
}
__device__ __forceinline__ u32x2 tld1(const tagged_t* base, int i) {
    u64 a = __hip_atomic_load(as_global((const u64*)(base + i)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return u32x2{(u32)a, (u32)(a >> 32)};
}
// Two consecutive tagged values (base + i, i even) as (v0, tag0, v1, tag1).  8-byte agent-scope
// atomic loads are used on purpose: 16-byte buffer loads with the same cache-policy bits were
// observed to keep returning a stale copy while polling, and inline-assembly loads cannot be kept
// asynchronous safely (the compiler may copy their destination registers before the data lands).
__device__ __forceinline__ u32x4 tld2(const tagged_t* base, int i) {
    u32x2 a = tld1(base, i), b = tld1(base, i + 1);
    return u32x4{a.x, a.y, b.x, b.y};
}

// All of the wave's loads have arrived, and the compiler knows it.  Said where that is so anyway (behind the words of an input, which come after all
// that was asked for before them): what the compiler may take for loads still on their way, because their waits lie on branches of their own, it
// would wait for where it next needs the registers, and the ring with them: at the head of every run of tiles, and ahead of the words.
__device__ __forceinline__ void settled() { __builtin_amdgcn_s_waitcnt(0xF70); }   // vmcnt(0)

// ---------------------------------------------------------------- compact exchange format
// The vectors that every workgroup reads whole (residual stream, sublayer outputs, merged attention
// output, SwiGLU output) travel as 4-byte words: the fp32 value rounded to 22 mantissa bits, with
// the low 2 bits of a per-buffer WRITE COUNTER in the freed bits.  Every element of such a buffer
// (for the sequences of the step) is rewritten each time the buffer is written, and the counter
// grows by exactly one per write, so whatever a reader can find in a slot is either the value it
// waits for or the previous write, whose counter bits differ (one bit would tell the two apart; two
// leave a margin and cost a quarter of an fp32 ulp).  The counter is derived from the number of
// steps EXECUTED on the buffers (kept on the device: a skipped step changes nothing), the layer and
// the phase.  Rows of sequences beyond the previous step's batch are re-initialised by the host
// side (a small fill) before a larger batch runs.  Two elements move per 8-byte coherent access.
typedef u32 cword_t;
constexpr u32 kCntMask = 3u;   // counter bits of a compact word
__device__ __forceinline__ u32 cpack(float v, u32 cnt) {
    const u32 b = __float_as_uint(v);
    const u32 r = (b & 0x7F800000u) == 0x7F800000u ? b : b + (kCntMask + 1u) / 2u;   // round to nearest; infinities and NaNs keep their class
    return (r & ~kCntMask) | (cnt & kCntMask);
}
__device__ __forceinline__ float cvalue(u32 w) { return __uint_as_float(w & ~kCntMask); }
__device__ __forceinline__ bool cfresh(u32 w, u32 cnt) { return ((w ^ cnt) & kCntMask) == 0; }
__device__ __forceinline__ void cst1(cword_t* p, float v, u32 cnt) { xst_u32(p, cpack(v, cnt)); }
__device__ __forceinline__ void cst2(cword_t* p, float v0, float v1, u32 cnt) {   // p 8-byte aligned
    xst2((float*)p, __uint_as_float(cpack(v0, cnt)), __uint_as_float(cpack(v1, cnt)));
}
__device__ __forceinline__ u32 cld1(const cword_t* base, int i) { return xld_u32(base + i); }
__device__ __forceinline__ u32x2 cld2(const cword_t* base, int i) {   // elements i, i+1 (i even)
    u64 a = __hip_atomic_load(as_global((const u64*)(base + i)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return u32x2{(u32)a, (u32)(a >> 32)};
}

// Workgroup-wide AND of a predicate with ONE barrier: every wave votes with a ballot, its first
// lane drops the result into an LDS slot, and after the barrier every thread reads all slots.
// Consecutive votes alternate between two sets of slots, so a wave that runs ahead to the next vote
// cannot overwrite a slot another wave has yet to read (the vote after that lies behind the next
// vote's barrier, which that other wave only reaches after its read).  All threads must take part
// in every vote, in the same order.
struct WgVote {
    static constexpr int kMaxSums = 4;
    u32* slots;   // LDS, 2 * (1 + kMaxSums) * (waves per workgroup) words
    u32 par;
    template <int NT>
    __device__ __forceinline__ bool all(bool ok) {
        const float none[1] = {0.f};
        float unused[1];
        return all_sum<NT, 1>(ok, none, unused);
    }
    // The same vote, which also adds up N (wave-uniform) floats per wave over the workgroup.
    template <int NT, int N>
    __device__ __forceinline__ bool all_sum(bool ok, const float (&part)[N], float (&total)[N]) {
        static_assert(N <= kMaxSums, "too many sums");
        constexpr int NW = NT / 64;
        const u32 w = __all(ok) ? 1u : 0u;
        u32* f = slots + par * (1 + kMaxSums) * NW;
        par ^= 1u;
        if ((threadIdx.x & 63) == 0) {
            f[threadIdx.x >> 6] = w;
#pragma unroll
            for (int n = 0; n < N; n++) f[(1 + n) * NW + (threadIdx.x >> 6)] = __float_as_uint(part[n]);
        }
        __syncthreads();
        u32 r = 1u;
#pragma unroll
        for (int i = 0; i < NW; i++) r &= f[i];
#pragma unroll
        for (int n = 0; n < N; n++) {
            float t = 0.f;
#pragma unroll
            for (int i = 0; i < NW; i++) t += __uint_as_float(f[(1 + n) * NW + i]);
            total[n] = t;
        }
        return __builtin_amdgcn_readfirstlane(r) != 0;
    }
};

// Input of a projection inside the fused kernel.
struct TSrc {
    const cword_t* base = nullptr; size_t stride = 0; u32 tag = 0;         // compact vector [B][stride] (tag = write counter) ...
    const bf16_t* embed = nullptr; const int* tokens = nullptr;            // ... or rows of the embedding table
    const cword_t* add = nullptr; size_t add_stride = 0; u32 add_tag = 0;  // optional: + sublayer output
    cword_t* wb = nullptr; size_t wb_stride = 0; u32 wb_tag = 0;           // optional: publish the sum (residual stream)
    const bf16_t* gain = nullptr; float eps = 0.f;                         // optional: RMSNorm
    UDiv ncta = {1, 0};                                                    // workgroups in the grid (each publishes 1/ncta of wb)
};

// Waits (bounded) until kPollLanes sampled elements of the source vector(s) carry their tags: a
// cheap way to sit out a producer that is still running -- a few 8-byte loads with pauses in
// between cost the memory system next to nothing even with every workgroup waiting at once.
template <bool HAS_ADD>
__device__ __forceinline__ bool light_wait(const TSrc& S, int batch, int k0, int nel, int lane) {
    const int sample = min(k0 + (int)(((long)(lane % kPollLanes) * nel) / kPollLanes) + (int)(blockIdx.x % 16) * 2, k0 + nel - 1);
    const cword_t* sb = S.base + (size_t)(batch - 1) * S.stride;
    const cword_t* sa = HAS_ADD ? S.add + (size_t)(batch - 1) * S.add_stride : nullptr;
    for (int spins = 0; spins < kSpinLimit; spins++) {
        bool ok = true;
        if (lane < kPollLanes) {
            ok = cfresh(cld1(sb, sample), S.tag);
            if constexpr (HAS_ADD) ok = ok && cfresh(cld1(sa, sample), S.add_tag);
        }
        if (__all(ok)) return true;
        __builtin_amdgcn_s_sleep(4);
    }
    return false;
}

// (a, b) rounded to bf16 (nearest even) and packed, a in the low half: v_cvt_pk_bf16_f32.
typedef float pk_f2 __attribute__((ext_vector_type(2)));
typedef __bf16 pk_bf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32 pack_bf16(float a, float b) {
    return __builtin_bit_cast(u32, __builtin_convertvector(pk_f2{a, b}, pk_bf2));
}
// fp32 pair -> packed bf16 heads and packed bf16 remainders, both round to nearest even:
// |error| <= 2^-18 |v|.
__device__ __forceinline__ void split_bf16x2(float a, float b, u32& hi, u32& lo) {
    hi = pack_bf16(a, b);
    lo = pack_bf16(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}
// The same in three parts: head, remainder and the remainder's remainder, |error| <= 2^-27 |v| (both subtractions are exact).
__device__ __forceinline__ void split3_bf16x2(float a, float b, u32& hi, u32& mid, u32& lo) {
    hi = pack_bf16(a, b);
    const float ra = a - __uint_as_float(hi << 16), rb = b - __uint_as_float(hi & 0xFFFF0000u);
    split_bf16x2(ra, rb, mid, lo);
}
// Wide pass (see ff_wide.h): a global image of a projection's inputs in the matrix cores' operand order,
// for `batch` sequences.  A k-step (32 columns) takes wide_step_bytes(nc, batch): 16-byte pieces (8 columns of one
// sequence) for each of the operand's four lane groups g.  Its form depends on nc, the sequences an operand holds:
//   1: one sequence in three parts (operand rows 0, 1, 2), group by group, with room for a fourth piece, so that a
//      step is 256 bytes and no load straddles a line;
//   8: group by group the heads of all sequences, then their remainders (operand rows 0..7 and 8..15);
//   16: the heads of all groups, then the remainders of all groups (an operand each).
// Which 8 columns lane group g multiplies in a k-step follows from the weights it loads, 16 bytes per lane:
// 8 << e columns (e = 0 bf16, 1 int8, 2 int4) used up in 1 << e k-steps.
__host__ __device__ __forceinline__ int wide_step_bytes(int nc, int batch) { return nc == 1 ? 256 : 128 * batch; }
struct WideImg {
    uint8_t* p; int e; int batch; int nc;
    __device__ __forceinline__ int planes() const { return nc == 1 ? 3 : 2; }
    __device__ __forceinline__ uint8_t* at(int n, int plane, int col) const {
        const int j = col >> 3, unit = j >> e, step = ((unit >> 2) << e) + (j & ((1 << e) - 1)), g = unit & 3;
        const int piece = nc == 1 ? 4 * g + plane : nc == 8 ? (2 * g + plane) * batch + n : (4 * plane + g) * batch + n;
        return p + (size_t)step * wide_step_bytes(nc, batch) + (piece * 16 + (col & 7) * 2);
    }
    // Columns col, col + 1 (col even) of sequence n.
    __device__ __forceinline__ void put2(int n, int col, float a, float b) const {
        u32 v[3];
        if (nc == 1) split3_bf16x2(a, b, v[0], v[1], v[2]);
        else split_bf16x2(a, b, v[0], v[1]);
#pragma unroll
        for (int pl = 0; pl < 3; pl++) if (pl < planes()) xst_u32((u32*)at(n, pl, col), v[pl]);
    }
    // Columns col .. col + 3 (col a multiple of four).
    __device__ __forceinline__ void put4(int n, int col, float a, float b, float c, float d) const {
        u32 v[3], w[3];
        if (nc == 1) { split3_bf16x2(a, b, v[0], v[1], v[2]); split3_bf16x2(c, d, w[0], w[1], w[2]); }
        else { split_bf16x2(a, b, v[0], v[1]); split_bf16x2(c, d, w[0], w[1]); }
#pragma unroll
        for (int pl = 0; pl < 3; pl++) if (pl < planes()) xst2((float*)at(n, pl, col), __uint_as_float(v[pl]), __uint_as_float(w[pl]));
    }
};

// Writes quad qi (elements 4*qi .. 4*qi+3) of sequence b into the staged vector: the quad-planar fp32 layout of stage_act.
template <int EPU>
__device__ __forceinline__ void stage_store(float4* xs, int nup, int b, int qi, const float4& t) {
    constexpr int NQ = EPU / 4;
    xs[((size_t)b * NQ + qi % NQ) * nup + qi / NQ] = t;
}

// Several-pass form (vectors longer than one pass of stage_tagged_onepass; one row at a time).
// The workgroup stages elements [k0, k0 + nunits*EPU) of every batch row into LDS in the
// quad-planar layout of stage_act, re-reading the tagged sources until their producers have
// written them.  Every thread issues all loads of its share of a batch at once and speculatively
// (a load issued behind a wave's weight prefetch takes microseconds to return, so round trips are
// what count); only if some tag in the workgroup is stale does it fall back to light polling.
// The first workgroup barrier inside doubles as the hand-over of the LDS region from the previous
// projection.  NT = threads of the workgroup.  Returns false (uniformly) on a time-out.
// QB = quads per thread and pass (2 8-byte loads per quad and source, all in flight at once; their
// 4*QB destination registers per source must fit beside the wave's prefetched weight tiles, or the
// compiler parks those tiles elsewhere and has to wait for them first).
template <int EPU, bool HAS_ADD, bool HAS_GAIN, int NT, int QB>
__device__ __forceinline__ bool stage_tagged_multipass(const TSrc& S, int batch, int K, int k0, int nunits, int nup, float4* xs, float* red, int tid, WgVote& vote, u64* ev) {
    constexpr int NQ = EPU / 4;
    if (ev && tid == 0) { as_global(ev)[0] = wall_clock64(); as_global(ev)[2] = 0; as_global(ev)[5] = 0; }
    const int lane = tid & 63;
    const int nquads = nunits * NQ;
    const int padquads = nup * NQ;
    const u32 wb_lo = S.ncta.div((u32)nquads * blockIdx.x), wb_hi = S.ncta.div((u32)nquads * (blockIdx.x + 1));
    for (int b = 0; b < batch; b++) {
        float4* xb = xs + (size_t)b * NQ * nup;
        const cword_t* src = S.base + (size_t)b * S.stride;
        const cword_t* add = HAS_ADD ? S.add + (size_t)b * S.add_stride : nullptr;
        const bf16_t* erow = nullptr;   // embedding rows only come through the (no add, gain) instance
        if constexpr (!HAS_ADD && HAS_GAIN) erow = S.tokens ? S.embed + (size_t)max(as_global(S.tokens)[b], 0) * K : nullptr;
        float ss = 0.f;
        for (int q0 = tid; q0 < padquads; q0 += NT * QB) {
            u32x4 v[QB], a[HAS_ADD ? QB : 1];   // four compact words per quad and source
            u32x2 g[HAS_GAIN ? QB : 1];
            bool all_ok = false;
            u32 stale = (1u << QB) - 1;   // quads (bit u) this lane still has to (re)load
            for (int spins = 0; spins < kSpinLimit && !all_ok; spins++) {
                // first pass: every quad of every lane; later passes: only what came back stale, so
                // a vector that was mostly complete is not fetched twice
#pragma unroll
                for (int u = 0; u < QB; u++) {
                    const int k = k0 + min(q0 + u * NT, nquads - 1) * 4;   // clamped: every load is issued
                    if (spins == 0 || ((stale >> u) & 1)) {
                        if (erow) {   // bf16 values are exact in the compact format: mark them fresh
                            u32x2 w = *as_global((const u32x2*)(erow + k));
                            const u32 t = S.tag & kCntMask;
                            v[u] = u32x4{(w.x << 16) | t, (w.x & 0xFFFF0000u) | t, (w.y << 16) | t, (w.y & 0xFFFF0000u) | t};
                        } else {
                            const u32x2 lo = cld2(src, k), hi = cld2(src, k + 2);
                            v[u] = u32x4{lo.x, lo.y, hi.x, hi.y};
                        }
                        if constexpr (HAS_ADD) {
                            const u32x2 lo = cld2(add, k), hi = cld2(add, k + 2);
                            a[u] = u32x4{lo.x, lo.y, hi.x, hi.y};
                        }
                    }
                    if constexpr (HAS_GAIN) { if (spins == 0) g[u] = *as_global((const u32x2*)(S.gain + k)); }
                }
                stale = 0;
#pragma unroll
                for (int u = 0; u < QB; u++) {
                    bool ok = cfresh(v[u].x, S.tag) && cfresh(v[u].y, S.tag) && cfresh(v[u].z, S.tag) && cfresh(v[u].w, S.tag);
                    if constexpr (HAS_ADD)
                        ok = ok && cfresh(a[u].x, S.add_tag) && cfresh(a[u].y, S.add_tag) && cfresh(a[u].z, S.add_tag) && cfresh(a[u].w, S.add_tag);
                    if (!ok) stale |= 1u << u;
                }
                all_ok = vote.all<NT>(stale == 0);
                if (ev && tid == 0 && spins == 0 && b == 0) as_global(ev)[1] = wall_clock64();
                if (!all_ok) {
                    bool lw = true;
                    if (tid < 64) lw = light_wait<HAS_ADD>(S, batch, k0, nunits * EPU, lane);
                    if (!vote.all<NT>(lw)) return false;
                    if (ev && tid == 0) { as_global(ev)[2] = wall_clock64(); as_global(ev)[5] += 1; }
                }
            }
            if (!all_ok) return false;
            if (ev && tid == 0) as_global(ev)[3] = wall_clock64();
#pragma unroll
            for (int u = 0; u < QB; u++) {
                const int qi = q0 + u * NT;
                if (qi < padquads) {
                    float4 t = make_float4(cvalue(v[u].x), cvalue(v[u].y), cvalue(v[u].z), cvalue(v[u].w));
                    if constexpr (HAS_ADD) { t.x += cvalue(a[u].x); t.y += cvalue(a[u].y); t.z += cvalue(a[u].z); t.w += cvalue(a[u].w); }
                    if (qi >= nquads) t = make_float4(0.f, 0.f, 0.f, 0.f);
                    else if (S.wb && (u32)qi >= wb_lo && (u32)qi < wb_hi) {   // this workgroup's slice of the published sum
                        cword_t* w = S.wb + (size_t)b * S.wb_stride + k0 + qi * 4;
                        cst2(w, t.x, t.y, S.wb_tag);
                        cst2(w + 2, t.z, t.w, S.wb_tag);
                    }
                    if constexpr (HAS_GAIN) {
                        if (qi < nquads) {
                            ss += t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
                            t.x *= bf_lo(g[u].x); t.y *= bf_hi(g[u].x); t.z *= bf_lo(g[u].y); t.w *= bf_hi(g[u].y);
                        }
                    }
                    stage_store<EPU>(xs, nup, b, qi, t);
                }
            }
        }
        if constexpr (HAS_GAIN) {
            ss = wave_sum_uniform(ss);
            if (lane == 0) red[tid >> 6] = ss;
            __syncthreads();
            float tot = 0.f;
#pragma unroll
            for (int w = 0; w < NT / 64; w++) tot += red[w];
            const float r = rsqrtf(tot / (float)K + S.eps);
            for (int qi = tid; qi < nquads; qi += NT) {   // each thread rescales the quads it wrote
                int j = qi / NQ, qd = qi % NQ;
                float4 v4 = xb[(size_t)qd * nup + j];
                v4.x *= r; v4.y *= r; v4.z *= r; v4.w *= r;
                xb[(size_t)qd * nup + j] = v4;
            }
            if (b + 1 < batch) __syncthreads();   // `red` is rewritten for the next row
        }
    }
    __syncthreads();
    return true;
}

// The common case, where one pass of QB quads per thread covers the whole vector (nup * EPU / 4 <=
// NT * QB): every thread keeps its quads in registers from the load to the LDS write, and the sums
// of squares of the normalisation travel with the freshness vote, so a row costs a single workgroup
// barrier and the staged vector is written once, already scaled.
template <int EPU, bool HAS_ADD, bool HAS_GAIN, int NT, int QB>
__device__ __forceinline__ bool stage_tagged_onepass(const TSrc& S, int batch, int K, int k0, int nunits, int nup, float4* xs, int tid, WgVote& vote, u64* ev) {
    constexpr int NQ = EPU / 4;
    if (ev && tid == 0) { as_global(ev)[0] = wall_clock64(); as_global(ev)[2] = 0; as_global(ev)[5] = 0; }
    const int lane = tid & 63;
    const int nquads = nunits * NQ;
    const int padquads = nup * NQ;
    const u32 wb_lo = S.ncta.div((u32)nquads * blockIdx.x), wb_hi = S.ncta.div((u32)nquads * (blockIdx.x + 1));
    for (int b = 0; b < batch; b++) {
        const cword_t* src = S.base + (size_t)b * S.stride;
        const cword_t* add = HAS_ADD ? S.add + (size_t)b * S.add_stride : nullptr;
        const bf16_t* erow = nullptr;   // embedding rows only come through the (no add, gain) instance
        if constexpr (!HAS_ADD && HAS_GAIN) erow = S.tokens ? S.embed + (size_t)max(as_global(S.tokens)[b], 0) * K : nullptr;
        u32x4 v[QB], a[HAS_ADD ? QB : 1];   // four compact words per quad and source
        u32x2 g[HAS_GAIN ? QB : 1];
        bool all_ok = false;
        float tot[1] = {0.f};
        u32 stale = (1u << QB) - 1;   // quads (bit u) this lane still has to (re)load
        // first every quad of every lane, unconditionally (no per-lane branches on the way to the
        // first request); after a failed vote only what came back stale, so a vector that was
        // mostly complete is not fetched twice
        auto load_quads = [&](auto ALL) {
            constexpr bool kAll = decltype(ALL)::value;
#pragma unroll
            for (int u = 0; u < QB; u++) {
                const int k = k0 + min(tid + u * NT, nquads - 1) * 4;   // clamped: every load is issued
                if (kAll || ((stale >> u) & 1)) {
                    if (erow) {   // bf16 values are exact in the compact format: mark them fresh
                        u32x2 w = *as_global((const u32x2*)(erow + k));
                        const u32 t = S.tag & kCntMask;
                        v[u] = u32x4{(w.x << 16) | t, (w.x & 0xFFFF0000u) | t, (w.y << 16) | t, (w.y & 0xFFFF0000u) | t};
                    } else {
                        const u32x2 lo = cld2(src, k), hi = cld2(src, k + 2);
                        v[u] = u32x4{lo.x, lo.y, hi.x, hi.y};
                    }
                    if constexpr (HAS_ADD) {
                        const u32x2 lo = cld2(add, k), hi = cld2(add, k + 2);
                        a[u] = u32x4{lo.x, lo.y, hi.x, hi.y};
                    }
                }
                if constexpr (HAS_GAIN && kAll) { g[u] = *as_global((const u32x2*)(S.gain + k)); }
            }
        };
        load_quads(std::true_type{});
        for (int spins = 0; spins < kSpinLimit && !all_ok; spins++) {
            float ss[1] = {0.f};   // only meaningful if the vote passes
            // The lane first ORs the counter mismatches of all its words together (one operation per
            // word) and looks at single quads only if something is stale.
            u32 dirty = 0;
#pragma unroll
            for (int u = 0; u < QB; u++) {
                dirty |= (v[u].x ^ S.tag) | (v[u].y ^ S.tag) | (v[u].z ^ S.tag) | (v[u].w ^ S.tag);
                if constexpr (HAS_ADD) dirty |= (a[u].x ^ S.add_tag) | (a[u].y ^ S.add_tag) | (a[u].z ^ S.add_tag) | (a[u].w ^ S.add_tag);
            }
            dirty &= kCntMask;
            stale = 0;
#pragma unroll
            for (int u = 0; u < QB; u++) {
                if (dirty) {
                    bool ok = cfresh(v[u].x, S.tag) && cfresh(v[u].y, S.tag) && cfresh(v[u].z, S.tag) && cfresh(v[u].w, S.tag);
                    if constexpr (HAS_ADD)
                        ok = ok && cfresh(a[u].x, S.add_tag) && cfresh(a[u].y, S.add_tag) && cfresh(a[u].z, S.add_tag) && cfresh(a[u].w, S.add_tag);
                    if (!ok) stale |= 1u << u;
                }
                if constexpr (HAS_GAIN) {
                    float4 t = make_float4(cvalue(v[u].x), cvalue(v[u].y), cvalue(v[u].z), cvalue(v[u].w));
                    if constexpr (HAS_ADD) { t.x += cvalue(a[u].x); t.y += cvalue(a[u].y); t.z += cvalue(a[u].z); t.w += cvalue(a[u].w); }
                    if (tid + u * NT < nquads) ss[0] += t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
                }
            }
            if constexpr (HAS_GAIN) ss[0] = wave_sum_uniform(ss[0]);
            if constexpr (HAS_GAIN) all_ok = vote.all_sum<NT, 1>(stale == 0, ss, tot);
            else all_ok = vote.all<NT>(stale == 0);
            if (ev && tid == 0 && spins == 0 && b == 0) as_global(ev)[1] = wall_clock64();
            if (!all_ok) {
                // A producer that is still streaming weights should not have to compete with 256
                // workgroups re-reading its output: wait on a few samples.
                bool lw = true;
                if (tid < 64) lw = light_wait<HAS_ADD>(S, batch, k0, nunits * EPU, lane);
                if (!vote.all<NT>(lw)) return false;
                if (ev && tid == 0) { as_global(ev)[2] = wall_clock64(); as_global(ev)[5] += 1; }
            }
            if (!all_ok) load_quads(std::false_type{});
        }
        if (!all_ok) return false;
        if (ev && tid == 0) as_global(ev)[3] = wall_clock64();
        // Usually every (lane, u) holds a real quad (the vector is a whole number of NT*QB quads,
        // no padding): that case runs without the per-lane range tests, each of which is a
        // divergent branch -- expensive for a wave that has its SIMD to itself.
        const bool exact = nquads == padquads && padquads == QB * NT;
        auto write_quad = [&](auto EX, int u, float rs) {
            constexpr bool kExact = decltype(EX)::value;
            const int qi = tid + u * NT;
            if (kExact || qi < padquads) {
                float4 t = make_float4(cvalue(v[u].x), cvalue(v[u].y), cvalue(v[u].z), cvalue(v[u].w));
                if constexpr (HAS_ADD) { t.x += cvalue(a[u].x); t.y += cvalue(a[u].y); t.z += cvalue(a[u].z); t.w += cvalue(a[u].w); }
                if (!kExact && qi >= nquads) t = make_float4(0.f, 0.f, 0.f, 0.f);
                else {
                    if (S.wb && (u32)qi >= wb_lo && (u32)qi < wb_hi) {   // this workgroup's slice of the published sum
                        cword_t* w = S.wb + (size_t)b * S.wb_stride + k0 + qi * 4;
                        cst2(w, t.x, t.y, S.wb_tag);
                        cst2(w + 2, t.z, t.w, S.wb_tag);
                    }
                    if constexpr (HAS_GAIN) {
                        t.x *= bf_lo(g[u].x) * rs; t.y *= bf_hi(g[u].x) * rs; t.z *= bf_lo(g[u].y) * rs; t.w *= bf_hi(g[u].y) * rs;
                    }
                }
                stage_store<EPU>(xs, nup, b, qi, t);
            }
        };
        const float rs = HAS_GAIN ? rsqrtf(tot[0] / (float)K + S.eps) : 1.f;
        if (exact) {
#pragma unroll
            for (int u = 0; u < QB; u++) write_quad(std::true_type{}, u, rs);
        } else {
#pragma unroll
            for (int u = 0; u < QB; u++) write_quad(std::false_type{}, u, rs);
        }
    }
    __syncthreads();
    return true;
}

// Picks the pass size that covers the vector in one pass with the fewest registers.
template <int EPU, bool HAS_ADD, int NT>
__device__ __forceinline__ bool stage_tagged(const TSrc& S, int batch, int K, int k0, int nunits, int nup, float4* xs, float* red, int tid,
                                             WgVote& vote, u64* ev = nullptr) {
    const int per_thread = (nup * (EPU / 4) + NT - 1) / NT;
    if constexpr (HAS_ADD) {   // residual stream + sublayer output, always normalised
        if (per_thread <= 4) return stage_tagged_onepass<EPU, true, true, NT, 4>(S, batch, K, k0, nunits, nup, xs, tid, vote, ev);
        if (per_thread <= 8) return stage_tagged_onepass<EPU, true, true, NT, 8>(S, batch, K, k0, nunits, nup, xs, tid, vote, ev);
        return stage_tagged_multipass<EPU, true, true, NT, 8>(S, batch, K, k0, nunits, nup, xs, red, tid, vote, ev);
    } else if (S.gain) {       // embedding rows
        if (per_thread <= 8) return stage_tagged_onepass<EPU, false, true, NT, 8>(S, batch, K, k0, nunits, nup, xs, tid, vote, ev);
        return stage_tagged_multipass<EPU, false, true, NT, 8>(S, batch, K, k0, nunits, nup, xs, red, tid, vote, ev);
    } else {
        if (per_thread <= 4) return stage_tagged_onepass<EPU, false, false, NT, 4>(S, batch, K, k0, nunits, nup, xs, tid, vote, ev);
        if (per_thread <= 8) return stage_tagged_onepass<EPU, false, false, NT, 8>(S, batch, K, k0, nunits, nup, xs, tid, vote, ev);
        if (per_thread <= 14) return stage_tagged_onepass<EPU, false, false, NT, 14>(S, batch, K, k0, nunits, nup, xs, tid, vote, ev);
        return stage_tagged_multipass<EPU, false, false, NT, 14>(S, batch, K, k0, nunits, nup, xs, red, tid, vote, ev);
    }
}

// 2^x straight from the hardware unit (v_exp_f32, about 1 ulp): the library routine wraps it in a
// rescaling sequence so that results below the normal range come out as denormals; here the
// arguments are differences to a running maximum (<= 0) and the results softmax weights, for which
// a flush to zero at 2^-126 is immaterial, and the sequence would be executed dozens of times on
// the attention's critical path.
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

// The thread's index, unknown to the compiler: what depends on the lane only is cheap to compute again in every layer, and hoisted out of the loop over layers it
// takes registers from the projections' loops (spilled there, 8B bf16 x 8: 20 of them).
__device__ __forceinline__ int thread_again() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ---------------------------------------------------------------- split-KV attention
// One work item = (sequence b, kv head j, rows [t0, t1) of its cache [+ this step's own k,v]).
// All G query heads that share kv head j are processed together, so each cached K and V element
// is read exactly once (paper Section 4.2, core attention: workgroups are split among KV heads and
// hold the queries of that head; the current token's k,v are taken from the exchange buffer, not
// from the cache).  Result: per query head the partial (max score, denominator, unnormalised
// output) of a FlashDecoding-style split, in base-2 exponent units.
//
// XIO supplies the exchange accesses (plain buffers for the per-operation kernels, tagged buffers for the decode kernels).
//
struct PlainAttnIO {
    // Workgroup-collective: the G query rows of kv head j, then (with_cur) this step's own key and
    // value row, as floats into dst[G*HD + 2*HD] (LDS); ends with a workgroup barrier.
    template <int HD, int G, int NT>
    __device__ __forceinline__ bool stage_inputs(const DevModel& M, int b, int j, bool with_cur, float* dst) const {
        const int nq = G * HD, n = nq + (with_cur ? 2 * HD : 0);
        for (int e = threadIdx.x; e < n; e += NT) {
            float v;
            if (e < nq) v = PlainIO::ld(M.q, (b * M.Hq + j * G) * HD + e);
            else v = PlainIO::ld(M.kvcur, ((b * 2 + (e - nq) / HD) * M.Hkv + j) * HD + (e - nq) % HD);
            dst[e] = v;
        }
        __syncthreads();
        return true;
    }
    // Four neighbouring output dims of query head h: the slice's unnormalised output, its maximum and denominator.
    template <int HD>
    __device__ __forceinline__ void put(const DevModel& M, int b, int h, int split, int nsplit, int dim, const f32x4& o, float mx, float lt) const {
        const size_t hs = ((size_t)b * M.Hq + h) * kMaxSplits + split;
        PlainIO::st4(M.part_o + hs * HD + dim, make_float4(o.x, o.y, o.z, o.w));
        if (dim == 0) { PlainIO::st(M.part_m + hs, mx); PlainIO::st(M.part_l + hs, lt); }
    }
};
// Staged inputs of the attention on the matrix cores (attn_item_mfma), in words of two bf16: rows of 16 bytes more than a query's
// (without them the 16 rows of an operand would lie in the same banks): the G queries' heads, their remainders, their third parts, rows of zeros up to whole
// operands; then the step's own key and value.
template <int HD, int G>
struct AttnParts {
    static constexpr int kOps = (3 * G + 15) / 16, kRows = 16 * kOps, kZeroRows = kRows - 3 * G, kRow = HD / 2 + 4;
    static constexpr int kWords = kRows * kRow + HD;
};
struct TaggedAttnIO {
    u32 in_tag;    // tag of q / kvcur (this layer's QKV projection)
    u32 out_tag;   // tag of the partials (this layer's attention)
    u32 out_cnt;   // write counter of the merged output's compact vector ...
    const WideImg* img;   // ... or (wide pass) the output projection's input image, which takes its place
    WgVote* vote;
    // Workgroup-collective, same contract as PlainAttnIO::stage_inputs.  The whole input of an
    // item is a few kilobytes (one or two 16-byte pairs per thread), so the workgroup simply
    // re-reads it until the QKV projection's tag is on every element; returns false on a time-out.
    // PARTS: for the matrix cores (AttnParts): the queries in three bf16 parts, key and value as they are in the cache.
    template <int HD, int G, int NT, bool PARTS = false>
    __device__ __forceinline__ bool stage_inputs(const DevModel& M, int b, int j, bool with_cur, float* dst) const {
        const int tid = thread_again();
        constexpr int NQ2 = G * HD / 2, NK2 = HD / 2;       // pairs of queries, of one k or v row
        constexpr int PP = (NQ2 + 2 * NK2 + NT - 1) / NT;   // pairs per thread
        const int np = NQ2 + (with_cur ? 2 * NK2 : 0);
        const tagged_t* qb = M.tq + (size_t)(b * M.Hq + j * G) * HD;
        const tagged_t* kb = M.tkvcur + (size_t)((b * 2 + 0) * M.Hkv + j) * HD;
        const tagged_t* vb = M.tkvcur + (size_t)((b * 2 + 1) * M.Hkv + j) * HD;
        u32x4 r[PP];
        bool done = false;
        for (int spins = 0; spins < kSpinLimit && !done; spins++) {
            bool ok = true;
#pragma unroll
            for (int u = 0; u < PP; u++) {
                const int p = min(tid + u * NT, np - 1);   // clamped: every load is issued
                const tagged_t* src = p < NQ2 ? qb + 2 * p : p < NQ2 + NK2 ? kb + 2 * (p - NQ2) : vb + 2 * (p - NQ2 - NK2);
                r[u] = tld2(src, 0);
            }
#pragma unroll
            for (int u = 0; u < PP; u++) ok = ok && r[u].y == in_tag && r[u].w == in_tag;
            done = vote->all<NT>(ok);
            if (!done) __builtin_amdgcn_s_sleep(2);
        }
        if (!done) { atomicCAS(M.status, 0, -51); return false; }
        if constexpr (PARTS) {
            typedef AttnParts<HD, G> P;
            u32* w = (u32*)dst;
            for (int i = tid; i < P::kZeroRows * (HD / 2); i += NT) w[(3 * G + i / (HD / 2)) * P::kRow + i % (HD / 2)] = 0u;
#pragma unroll
            for (int u = 0; u < PP; u++) {
                const int p = tid + u * NT;
                if (p < NQ2) {
                    u32 hi, mid, lo;
                    split3_bf16x2(__uint_as_float(r[u].x), __uint_as_float(r[u].z), hi, mid, lo);
                    u32* q = w + p / (HD / 2) * P::kRow + p % (HD / 2);
                    q[0] = hi; q[G * P::kRow] = mid; q[2 * G * P::kRow] = lo;
                } else if (p < np) w[P::kRows * P::kRow + (p - NQ2)] = (r[u].x >> 16) | (r[u].z & 0xFFFF0000u);   // (bf16 values)
            }
            __syncthreads();
            return true;
        }
#pragma unroll
        for (int u = 0; u < PP; u++) {
            const int p = tid + u * NT;
            if (p < np) { dst[2 * p] = __uint_as_float(r[u].x); dst[2 * p + 1] = __uint_as_float(r[u].z); }
        }
        __syncthreads();
        return true;
    }
    __device__ __forceinline__ void put_merged(const DevModel& M, int b, int h, int hd, int dim, float a, float c) const {   // two neighbouring dims
        if (img) img->put2(b, h * hd + dim, a, c);
        else cst2(M.cattn_o + ((size_t)b * M.Hq + h) * hd + dim, a, c, out_cnt);
    }
    template <int HD>
    __device__ __forceinline__ void put(const DevModel& M, int b, int h, int split, int nsplit, int dim, const f32x4& o, float mx, float lt) const {
        if (nsplit == 1) {   // the only slice: nothing to merge it with
            const float inv = 1.0f / lt;
            put_merged(M, b, h, HD, dim, o.x * inv, o.y * inv);
            put_merged(M, b, h, HD, dim + 2, o.z * inv, o.w * inv);
            return;
        }
        const size_t hs = ((size_t)b * M.Hq + h) * kMaxSplits + split;
        if (dim == 0) { tst(M.tpart_m + hs, mx, out_tag); tst(M.tpart_l + hs, lt, out_tag); }
        tst2(M.tpart_o + hs * HD + dim, o.x, o.y, out_tag);
        tst2(M.tpart_o + hs * HD + dim + 2, o.z, o.w, out_tag);
    }
};

// ---- row groups of a wave (attn_item) meeting in registers ----
// Lanes l and l ^ D exchange: the lane whose bit D is clear gets (own a, other's a), the other one (other's b, own b).
// D = 32, 16: one permlane swap; D = 8: a rotation within the row of 16 lanes.
template <int D>
__device__ __forceinline__ void lane_exchange(float& a, float& b, int lane) {
    if constexpr (D == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
    } else if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
    } else {
        static_assert(D == 8, "exchange distance");
        const bool up = (lane & 8) != 0;
        const float give = up ? a : b, keep = up ? b : a;
        a = keep;
        b = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xF, 0xF, true));   // row_ror:8
    }
}
template <int D> __device__ __forceinline__ float lane_pair_max(float v, int lane) { float a = v, b = v; lane_exchange<D>(a, b, lane); return fmaxf(a, b); }
template <int D> __device__ __forceinline__ float lane_pair_sum(float v, int lane) { float a = v, b = v; lane_exchange<D>(a, b, lane); return a + b; }
// v[0..N) summed over lanes l and l ^ D; the lane keeps the half of the sums that its bit D names, in v[0..N/2).
template <int D, int N, int M>
__device__ __forceinline__ void lane_halve(float (&v)[M], int lane) {
#pragma unroll
    for (int i = 0; i < N / 2; i++) {
        float a = v[i], b = v[i + N / 2];
        lane_exchange<D>(a, b, lane);
        v[i] = a + b;
    }
}

#ifndef FF_ATTN_BATCH
#define FF_ATTN_BATCH 4   // wave loads of K and of V in flight per wave (can be overridden at build time for sweeps; 8 measured no faster)
#endif
// LDS of attn_item: the waves' states, then the staged queries and the step's own key and value.
template <int HD, int G, int NW> constexpr int kAttnStateFloats = NW * G * HD + 2 * NW * G;
// The waves' maxima and denominators, behind their outputs.
template <int HD, int G, int NW>
__device__ __forceinline__ float2& attn_state_ml(uint8_t* lds, int wave, int g) { return ((float2*)((float*)lds + (size_t)NW * G * HD))[wave * G + g]; }
// The waves' states (spread over the lanes: of the list (head, element of a lane's eight dims) lane n holds G * 8 / (64 / LPR) values from first(n) on,
// in o[0 ..]; maxima and denominators stored) meet in LDS and leave through xio.  Workgroup-collective.
template <int HD, int G, int NW, class XIO, class First, int M_>
__device__ __forceinline__ void attn_finish(const DevModel& M, const XIO& xio, int b, int j, int split, int nsplit, uint8_t* lds, const float (&o)[M_], int lane, int wave, First&& first_of) {
    const int tid = thread_again();
    constexpr int LPR = HD / 8, RPW = 64 / LPR, NT = NW * 64;
    constexpr int NV = G * 8 / RPW;   // values a lane keeps
    // quad c (of NV / 4) of the lane: values 4 c .. 4 c + 3; planes of 64 float4, so that neither side has bank conflicts
    f32x4* so = (f32x4*)lds;                                            // [wave][NV / 4][64]
#pragma unroll
    for (int c = 0; c < NV / 4; c++) so[(wave * (NV / 4) + c) * 64 + lane] = f32x4{o[4 * c], o[4 * c + 1], o[4 * c + 2], o[4 * c + 3]};
    __syncthreads();
    for (int i = tid; i < NV / 4 * 64; i += NT) {
        const int c = i >> 6, n = i & 63;
        const int first = first_of(n) + 4 * c;
        const int g = first >> 3, dim = (n % LPR) * 8 + (first & 7);
        float2 ml[NW];
        f32x4 v[NW];
#pragma unroll
        for (int w = 0; w < NW; w++) { ml[w] = attn_state_ml<HD, G, NW>(lds, w, g); v[w] = so[(w * (NV / 4) + c) * 64 + n]; }
        float mx = ml[0].x;
#pragma unroll
        for (int w = 1; w < NW; w++) mx = fmaxf(mx, ml[w].x);
        float lt = 0.f;
        f32x4 ot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const float f = exp2_hw(ml[w].x - mx);   // empty states have m = -inf -> weight 0
            lt = fmaf(ml[w].y, f, lt);
#pragma unroll
            for (int e = 0; e < 4; e++) ot[e] = fmaf(v[w][e], f, ot[e]);
        }
        xio.template put<HD>(M, b, j * G + g, split, nsplit, dim, ot, mx, lt);
    }
}

// One item with both products on the matrix cores (head dimension 128).  A wave takes 16 cached rows at a time; as in the row-wise form it loads values
// with 16 lanes per row, load i of lane group g holding row 4 i + g of the batch.
//   * Scores: v_mfma_f32_16x16x32_bf16, keys as A operand, the queries' three bf16 parts (24 bits) as columns of B.  Key row 4 (r % 4) + r / 4 of the batch is
//     operand row r, so that lane (column, g) gets the scores of rows 4 i + g, i = 0..3: those whose values lane group g holds.  The parts' columns are added by row rotations, after
//     which every lane has the scores of head n % G, and their weights are computed where they are needed:
//   * output: v_mfma_f32_16x16x16_bf16, A = the weights' three parts (rows: part, head; lane (m, g), element i: row 4 i + g), B = for each
//     element e of the lanes' eight dims the values (the same rows; two 16-bit halves of two loads' words put together by one permutation).  The sums over lane groups, which
//     the row-wise form ends with, come out of the products.
// What bounds it is the cached rows' way from memory; a batch is about 100 vector instructions, where a form with the scores alone on the matrix cores had 400 with
// four query heads and 700 with eight, and the row-wise form 530 cycles per row with eight.  Us per step, before (the best of those per kernel) / with this form: one sequence
// 8B bf16 context 1024 693 / 677, int8 4096 488 / 479, int4 2048 360 / 343, 70B bf16 2048 1658 / 1636; several: 8B bf16 x 2 737 / 719, x 8 782 / 771, int4 x 4 514 /
// 512, int8 x 4 543 / 533, x 11 745 / 731, int4 x 16 724 / 728, 70B x 16 1935 / 1893.  With two batches of rows in flight several sequences are
// slower (733, 783, 525, 535, 742, 752, 1906): the registers of the second batch are spilled over the projections' loops.
typedef __bf16 attn_bf8 __attribute__((ext_vector_type(8)));
typedef short attn_s4 __attribute__((ext_vector_type(4)));
template <int HD, int G, int NW, class XIO>
__device__ __forceinline__ bool attn_item_mfma(const DevModel& M, const DevKV& KV, const XIO& xio, int layer, int b, int j, int t0, int t1, bool with_cur,
                                               int split, int nsplit, uint8_t* lds, u64* ev) {
    static_assert(HD == 128 && (G == 4 || G == 8), "operand layouts");
    typedef AttnParts<HD, G> P;
    constexpr int NT = NW * 64, kStride = NW * 16, kOps = P::kOps;
    const int tid = thread_again(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, g4 = lane >> 4;
    const float sc = 1.4426950408889634f / sqrtf((float)HD);   // alpha * log2(e)
    const bf16_t* Kp = KV.plane(M, layer, b, j, 0);
    const bf16_t* Vp = KV.plane(M, layer, b, j, 1);
    u32x4 kw[4], vw[4];
    auto issue = [&](int tb) {
        const u32 tk = (u32)min(tb + 4 * (n & 3) + (n >> 2), t1 - 1);   // clamped: every load is issued
#pragma unroll
        for (int kk = 0; kk < 4; kk++) kw[kk] = ldg_stream(Kp + (size_t)tk * HD + 32 * kk + 8 * g4);
#pragma unroll
        for (int i = 0; i < 4; i++) vw[i] = ldg_stream(Vp + (size_t)(u32)min(tb + 4 * i + g4, t1 - 1) * HD + n * 8);
    };
    int tb = t0 + 16 * wave;
    if (tb < t1) issue(tb);   // (an empty range has no row to clamp to)
    u32* parts = (u32*)((float*)lds + kAttnStateFloats<HD, G, NW>);
    const bool ok = xio.template stage_inputs<HD, G, NT, true>(M, b, j, with_cur, (float*)parts);
    if (ev && threadIdx.x == 0) as_global(ev)[1] = wall_clock64();
    if (!ok) return false;   // uniform
    float m = -INFINITY, l = 0.f;   // of head n % G: maximum over the wave's rows, sum over this lane's
    mfma_f4 d[8];                   // element e: rows (part, head) 4 g4 .. 4 g4 + 3 of the A operand(s)
#pragma unroll
    for (int e = 0; e < 8; e++) d[e] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    const bool works = tb < t1 || (with_cur && wave == NW - 1);
    u32x4 qb[kOps][4];
    if (works) {
#pragma unroll
        for (int op = 0; op < kOps; op++)
#pragma unroll
            for (int kk = 0; kk < 4; kk++) qb[op][kk] = *(const u32x4*)(parts + (16 * op + n) * P::kRow + 16 * kk + 4 * g4);
    }
    auto ror = [](float v, auto C) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(C)::value, 0xF, 0xF, true)); };
    typedef std::integral_constant<int, 0x124> Ror4;
    typedef std::integral_constant<int, 0x128> Ror8;
    // rows first .. : row 4 i + g4 of the batch counts if it is below `rows`
    auto consume = [&](const u32x4* k, const u32x4* v, int rows) {
        mfma_f4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int op = 0; op < kOps; op++)
#pragma unroll
            for (int kk = 0; kk < 4; kk++)
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(attn_bf8, k[kk]), __builtin_bit_cast(attn_bf8, qb[op][kk]), c, 0, 0, 0);
        float s[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float t = c[i];
            t += ror(t, Ror8{});   // (in this order all lanes of a head add up the same pairs: below, a weight's three parts come from three of them)
            if constexpr (G == 4) t += ror(t, Ror4{});
            s[i] = 4 * i + g4 < rows ? t * sc : -INFINITY;
        }
        float mb = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
        mb = lane_pair_max<16>(lane_pair_max<32>(mb, lane), lane);
        const float mn = fmaxf(m, mb), mref = mn == -INFINITY ? 0.f : mn;
        if (__builtin_amdgcn_ballot_w64(mn > m && m != -INFINITY)) {   // (nothing to rescale while the maximum stands, or before the first row)
            const float corr = m == -INFINITY ? 1.f : exp2_hw(m - mref);
            l *= corr;
            float f[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                f[r] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(corr), r));
                if constexpr (G == 8) { const float h = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(corr), 4 + r)); f[r] = g4 & 1 ? h : f[r]; }
            }
#pragma unroll
            for (int e = 0; e < 8; e++)
#pragma unroll
                for (int r = 0; r < 4; r++) d[e][r] *= f[r];
        }
        m = mn;
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; i++) p[i] = exp2_hw(s[i] - mref);
        l += (p[0] + p[1]) + (p[2] + p[3]);
        u32 hi[2], mid[2], lo[2];
        split3_bf16x2(p[0], p[1], hi[0], mid[0], lo[0]);
        split3_bf16x2(p[2], p[3], hi[1], mid[1], lo[1]);
        u32x2 a[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            if constexpr (G == 4) a[0][h] = n < 8 ? (n < 4 ? hi[h] : mid[h]) : (n < 12 ? lo[h] : 0u);
            else { a[0][h] = n < 8 ? hi[h] : mid[h]; a[1][h] = n < 8 ? lo[h] : 0u; }
        }
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const u32 sel = e & 1 ? 0x07060302u : 0x05040100u;
            const u32x2 bv = {__builtin_amdgcn_perm(v[1][e >> 1], v[0][e >> 1], sel), __builtin_amdgcn_perm(v[3][e >> 1], v[2][e >> 1], sel)};
#pragma unroll
            for (int op = 0; op < kOps; op++)
                d[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(attn_s4, a[op]), __builtin_bit_cast(attn_s4, bv), d[e], 0, 0, 0);
        }
    };
    for (bool first = true; tb < t1; tb += kStride, first = false) {
        if (!first) issue(tb);
        consume(kw, vw, t1 - tb);
    }
    settled();
    if (with_cur && wave == NW - 1) {   // this step's own key and value: a batch of one row (by the wave that has the fewest of the others)
        const u32* own = parts + P::kRows * P::kRow;
        const u32x4 none = {0u, 0u, 0u, 0u};
        u32x4 ck[4], cv[4] = {*(const u32x4*)(own + HD / 2 + 4 * n), none, none, none};
#pragma unroll
        for (int kk = 0; kk < 4; kk++) ck[kk] = *(const u32x4*)(own + 16 * kk + 4 * g4);   // (the same key in all rows)
        if (g4 != 0) cv[0] = none;
        consume(ck, cv, 1);
    }
    // the wave's state: parts added up by halving, see below; denominators over the lane groups
    l = lane_pair_sum<16>(lane_pair_sum<32>(l, lane), lane);
    if (lane < G) attn_state_ml<HD, G, NW>(lds, wave, lane) = make_float2(m, l);
    float o[32];
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int e = 0; e < 8; e++) o[r * 8 + e] = d[e][r];
    lane_halve<32, 32>(o, lane);
    if constexpr (G == 4) lane_halve<16, 16>(o, lane);
    if (ev && threadIdx.x == 0) as_global(ev)[2] = wall_clock64();
    // (eight heads: lane group g holds heads 4 (g % 2) .., and of these two by the upper bit)
    attn_finish<HD, G, NW>(M, xio, b, j, split, nsplit, lds, o, lane, wave, [&](int q) { return G == 4 ? 8 * (q >> 4) : 32 * ((q >> 4) & 1) + 16 * (q >> 5); });
    if (ev && threadIdx.x == 0) as_global(ev)[3] = wall_clock64();
    return true;
}
// One item, row by row on the vector ALU (head dimension 64, and the per-operation kernels).  A cache row is hd*2 bytes = LPR lanes x 16 bytes, so one wave load covers 64/LPR rows; lane
// (grp, sub) holds dims [8*sub, 8*sub+8) of row grp.  Every (wave, grp) keeps its own online-softmax state; a wave's merge in registers, the waves' through LDS (NW = waves of the
// workgroup, all of which take part).  Returns false on a time-out.
template <int HD, int G, int NW, class XIO, bool MFMA = false>   // MFMA: attn_item_mfma where the head dimension allows it
__device__ __forceinline__ bool attn_item(const DevModel& M, const DevKV& KV, const XIO& xio, int layer, int b, int j, int t0, int t1, bool with_cur,
                          int split, int nsplit, uint8_t* lds, u64* ev = nullptr) {
    if constexpr (MFMA && HD == 128) return attn_item_mfma<HD, G, NW, XIO>(M, KV, xio, layer, b, j, t0, t1, with_cur, split, nsplit, lds, ev);
    constexpr int LPR = HD / 8;        // lanes per cache row
    constexpr int RPW = 64 / LPR;      // rows per wave load
    constexpr int NT = NW * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane / LPR, sub = lane % LPR;
    const float sc = 1.4426950408889634f / sqrtf((float)HD);   // alpha * log2(e)

    float m[G], l[G], o[G * 8];
#pragma unroll
    for (int g = 0; g < G; g++) {
        m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) o[g * 8 + e] = 0.f;
    }
    const bf16_t* Kp = KV.plane(M, layer, b, j, 0);
    const bf16_t* Vp = KV.plane(M, layer, b, j, 1);
    float qr[G][8];
    // one row (keys kf, values vf of the lane's eight dims) into head g's state; q: the head's query
    auto update_head = [&](int g, const float (&q)[8], const float (&kf)[8], const float (&vf)[8], bool valid) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < 8; e++) s = fmaf(q[e], kf[e], s);
            s = group_sum<LPR>(s) * sc;
            if (valid) {
                float mn = fmaxf(m[g], s);
                float corr = exp2_hw(m[g] - mn), p = exp2_hw(s - mn);
                l[g] = l[g] * corr + p;
#pragma unroll
                for (int e = 0; e < 8; e++) o[g * 8 + e] = fmaf(p, vf[e], o[g * 8 + e] * corr);
                m[g] = mn;
            }
    };
    auto update = [&](const float (&kf)[8], const float (&vf)[8], bool valid) {
#pragma unroll
        for (int g = 0; g < G; g++) update_head(g, qr[g], kf, vf, valid);
    };
    // Cached rows do not depend on this step: the first kAttnBatch wave-loads are issued BEFORE the
    // queries are waited for, so the wait for the QKV projection overlaps them.
    constexpr int kAttnBatch = FF_ATTN_BATCH;
    constexpr int kStride = NW * RPW * kAttnBatch;
    u32x4 kw[kAttnBatch], vw[kAttnBatch];
    auto issue = [&](int tb0) {
#pragma unroll
        for (int i = 0; i < kAttnBatch; i++) {
            const int t = min(tb0 + i * NW * RPW + grp, t1 - 1);   // clamped: every load is issued
            kw[i] = ldg_stream(Kp + (size_t)t * HD + sub * 8);
            vw[i] = ldg_stream(Vp + (size_t)t * HD + sub * 8);
        }
    };
    int tb0 = t0 + wave * RPW;
    if (tb0 < t1) issue(tb0);
    // queries of the G heads and this step's own k, v: staged once per workgroup behind the state
    // merge area, then read by every lane from LDS
    float* xin = (float*)lds + kAttnStateFloats<HD, G, NW>;
    const bool ok = xio.template stage_inputs<HD, G, NT>(M, b, j, with_cur, xin);
    if (ev && threadIdx.x == 0) as_global(ev)[1] = wall_clock64();
    if (!ok) return false;   // uniform
    auto load_q = [&](int g, float (&q)[8]) {
        const float4 q0 = *(const float4*)(xin + g * HD + sub * 8), q1 = *(const float4*)(xin + g * HD + sub * 8 + 4);
        q[0] = q0.x; q[1] = q0.y; q[2] = q0.z; q[3] = q0.w;
        q[4] = q1.x; q[5] = q1.y; q[6] = q1.z; q[7] = q1.w;
    };
#pragma unroll
    for (int g = 0; g < G; g++) load_q(g, qr[g]);
    for (bool first = true; tb0 < t1; tb0 += kStride, first = false) {
        if (!first) issue(tb0);
#pragma unroll
        for (int i = 0; i < kAttnBatch; i++) {
            // (head dimension 64: a batch is 256 rows, most slices are far shorter.  Tiny shape, context 128: 94.9 -> 92.8 us per step; at
            // 128 the branch costs as much as it saves: 8B int4 x 4, context 2048, eight layers, 512 -> 516)
            if (HD == 64 && i > 0 && tb0 + i * NW * RPW >= t1) break;
            const bool valid = tb0 + i * NW * RPW + grp < t1;
            float kf[8] = {bf_lo(kw[i].x), bf_hi(kw[i].x), bf_lo(kw[i].y), bf_hi(kw[i].y), bf_lo(kw[i].z), bf_hi(kw[i].z), bf_lo(kw[i].w), bf_hi(kw[i].w)};
            float vf[8] = {bf_lo(vw[i].x), bf_hi(vw[i].x), bf_lo(vw[i].y), bf_hi(vw[i].y), bf_lo(vw[i].z), bf_hi(vw[i].z), bf_lo(vw[i].w), bf_hi(vw[i].w)};
            update(kf, vf, valid);
        }
    }
    settled();
    if (with_cur && wave == 0) {   // this step's own key/value (uniform branch per wave)
        float kf[8], vf[8];
        const float* kc = xin + G * HD + sub * 8;
        const float* vc = kc + HD;
#pragma unroll
        for (int e = 0; e < 8; e++) { kf[e] = kc[e]; vf[e] = vc[e]; }
        update(kf, vf, grp == 0);   // scores reduce over the lanes of one row group: only group 0 is valid
    }
    // ---- the row groups of a wave merge in registers, the waves' states through LDS ----
    // Every wave first brings its groups to one maximum per head, then the sums over groups are formed by
    // exchanging halves: of a lane's G * 8 values (head g, element e of its eight dims) it keeps those that
    // the group bits of its lane number select, so the wave's state ends up spread over all lanes and is
    // written and read once, in a fourth of the LDS (HD 64: an eighth) that the groups' states took.  (From the queries to the
    // stored partial, 8B, groups' states through LDS / this: bf16 x 2 3.9 / 3.5 us, int4 x 4 7.0 / 6.8, int4 x 16 19.2 / 19.0.)
    static_assert((RPW == 4 && LPR == 16) || (RPW == 8 && LPR == 8 && G == 4), "group bits of the lane number");
#pragma unroll
    for (int g = 0; g < G; g++) {
        float mw = lane_pair_max<32>(m[g], lane);
        mw = lane_pair_max<16>(mw, lane);
        if constexpr (RPW == 8) mw = lane_pair_max<8>(mw, lane);
        const float f = exp2_hw(m[g] - (mw == -INFINITY ? 0.f : mw));   // groups (or waves) without a row: weight 0
        l[g] = lane_pair_sum<16>(lane_pair_sum<32>(l[g] * f, lane), lane);
        if constexpr (RPW == 8) l[g] = lane_pair_sum<8>(l[g], lane);
        m[g] = mw;
#pragma unroll
        for (int e = 0; e < 8; e++) o[g * 8 + e] *= f;
    }
    lane_halve<32, G * 8>(o, lane);
    lane_halve<16, G * 4>(o, lane);
    if constexpr (RPW == 8) lane_halve<8, G * 2>(o, lane);
    if (ev && threadIdx.x == 0) as_global(ev)[2] = wall_clock64();
    if (lane == 0) {
#pragma unroll
        for (int g = 0; g < G; g++) attn_state_ml<HD, G, NW>(lds, wave, g) = make_float2(m[g], l[g]);
    }
    attn_finish<HD, G, NW>(M, xio, b, j, split, nsplit, lds, o, lane, wave, [&](int n) { return RPW == 8 ? 16 * (n >> 5) + 8 * ((n >> 4) & 1) + 4 * ((n >> 3) & 1) : G * 2 * (n >> 4); });
    if (ev && threadIdx.x == 0) as_global(ev)[3] = wall_clock64();
    return ok;
}

// Final merge for (b, kv head j) over nsplit partials (paper Section 4.2: combine per-block maximum
// and denominator, rescale by own/global denominator ratio, sum): writes attn_o[b][h][:].
// Workgroup-collective; uses 2*G*kMaxSplits floats of LDS.
template <int HD, int G, int NT>
__device__ void attn_merge(const DevModel& M, int b, int j, int nsplit, float* lds) {
    typedef PlainIO IO;
    float* ms = lds;                       // [G][nsplit] maxima, then normalised weights
    float* ls = lds + G * kMaxSplits;      // [G][nsplit] denominators
    __syncthreads();
    for (int idx = threadIdx.x; idx < G * nsplit; idx += NT) {
        int g = idx / nsplit, s = idx % nsplit;
        int hs = (b * M.Hq + (j * G + g)) * kMaxSplits + s;
        ms[g * kMaxSplits + s] = IO::ld(M.part_m, hs);
        ls[g * kMaxSplits + s] = IO::ld(M.part_l, hs);
    }
    __syncthreads();
    if (threadIdx.x < G) {
        int g = threadIdx.x;
        float mx = -INFINITY;
        for (int s = 0; s < nsplit; s++) mx = fmaxf(mx, ms[g * kMaxSplits + s]);
        float lt = 0.f;
        for (int s = 0; s < nsplit; s++) {
            float w = exp2_hw(ms[g * kMaxSplits + s] - mx);
            ms[g * kMaxSplits + s] = w;
            lt = fmaf(ls[g * kMaxSplits + s], w, lt);
        }
        float inv = 1.0f / lt;
        for (int s = 0; s < nsplit; s++) ms[g * kMaxSplits + s] *= inv;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < G * HD / 4; idx += NT) {
        int g = idx / (HD / 4), d4 = (idx % (HD / 4)) * 4;
        int hs = (b * M.Hq + (j * G + g)) * kMaxSplits;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
        for (int s = 0; s < nsplit; s++) {
            float4 o = IO::ld4(M.part_o, (hs + s) * HD + d4);
            float w = ms[g * kMaxSplits + s];
            acc.x = fmaf(o.x, w, acc.x); acc.y = fmaf(o.y, w, acc.y); acc.z = fmaf(o.z, w, acc.z); acc.w = fmaf(o.w, w, acc.w);
        }
        IO::st4(M.attn_o + ((size_t)b * M.Hq + (j * G + g)) * HD + d4, acc);
    }
}

// The same merge on tagged partials (fused kernel), shared out: each of the nsplit workgroups of the head
// group merges its share of the output dims, in pairs, out of all slices' partials.  Nothing goes through
// LDS and no wave waits for another: a lane requests the partial outputs, maxima and denominators it needs
// in one round and repeats that until all of them carry this layer's attention tag.  Up to four slices: a
// lane has a pair to itself; more: eight or sixteen lanes share a pair, each taking one slice or every sixteenth, and add up with
// row operations.  What bounds it is the hop from the stores to the loads.  (The workgroup of the last slice alone
// gathering all partials, which first waited for the maxima and then re-read what was stale: from the stored partials to the
// merged output 7.7 us at 8B int4 x 1, context 2048, 5.7 at x 4 and 4.7 at x 16; shared out 3.2, 2.6 and 2.1.)
// A workgroup whose item has several slices has no other item (attn_share_of), so the waits are never circular.
// Returns false (per wave) on a time-out.
template <int HD, int G, int NT>
__device__ __forceinline__ bool attn_merge_tagged(const DevModel& M, const TaggedAttnIO& xio, int b, int j, int split, int nsplit) {
    constexpr int E = G * HD / 2;   // pairs of the head group
    const int tid = thread_again();
    const u32 tag = xio.out_tag;
    const int e0 = (int)((u32)(E * split) / (u32)nsplit), e1 = (int)((u32)(E * (split + 1)) / (u32)nsplit);
    const int h0 = b * M.Hq + j * G;
    bool all_ok = true;
    // N partials per lane: slices s, s + STEP, ... (the last one again behind the end, with weight 0)
    auto gather = [&](auto N_, auto STEP_, int e, int s, float& a0, float& a1) {
        constexpr int N = decltype(N_)::value, STEP = decltype(STEP_)::value;
        const int hs = (h0 + e / (HD / 2)) * kMaxSplits, d2 = (e % (HD / 2)) * 2;
        u32x4 o[N];
        u32x2 pm[N], pl[N];
        bool ok = false;
        for (int spins = 0; spins < kSpinLimit && !ok; spins++) {
            bool mine = true;
#pragma unroll
            for (int u = 0; u < N; u++) {
                const int k = hs + min(s + STEP * u, nsplit - 1);
                o[u] = tld2(M.tpart_o, k * HD + d2);
                pm[u] = tld1(M.tpart_m, k);
                pl[u] = tld1(M.tpart_l, k);
            }
#pragma unroll
            for (int u = 0; u < N; u++) mine = mine && o[u].y == tag && o[u].w == tag && pm[u].y == tag && pl[u].y == tag;
            ok = __all(mine);
            if (!ok) __builtin_amdgcn_s_sleep(1);
        }
        if (!ok) { atomicCAS(M.status, 0, -53); all_ok = false; return; }
        float mx = __uint_as_float(pm[0].x);
#pragma unroll
        for (int u = 1; u < N; u++) mx = fmaxf(mx, __uint_as_float(pm[u].x));
        if constexpr (STEP > 1) mx = group_max<STEP>(mx);
        float lt = 0.f;
        a0 = a1 = 0.f;
#pragma unroll
        for (int u = 0; u < N; u++) {
            const float w = s + STEP * u < nsplit ? exp2_hw(__uint_as_float(pm[u].x) - mx) : 0.f;
            lt = fmaf(__uint_as_float(pl[u].x), w, lt);
            a0 = fmaf(__uint_as_float(o[u].x), w, a0);
            a1 = fmaf(__uint_as_float(o[u].z), w, a1);
        }
        if constexpr (STEP > 1) { lt = group_sum<STEP>(lt); a0 = group_sum<STEP>(a0); a1 = group_sum<STEP>(a1); }
        const float inv = 1.0f / lt;
        a0 *= inv; a1 *= inv;
    };
    typedef std::integral_constant<int, 1> One;
    if (nsplit <= 4) {
        for (int e = e0 + tid; e < e1; e += NT) {   // (a wave's lanes past the end do not vote)
            float a0, a1;
            gather(std::integral_constant<int, 4>{}, One{}, e, 0, a0, a1);
            if (all_ok) xio.put_merged(M, b, j * G + e / (HD / 2), HD, (e % (HD / 2)) * 2, a0, a1);
        }
        return all_ok;
    }
    if (nsplit <= 8) {   // (with sixteen lanes per pair five to seven slices' shares took two rounds)
        for (int e = e0 + (tid >> 3); e < e1; e += NT / 8) {
            float a0, a1;
            gather(One{}, std::integral_constant<int, 8>{}, e, tid & 7, a0, a1);
            if (all_ok && (tid & 7) == 0) xio.put_merged(M, b, j * G + e / (HD / 2), HD, (e % (HD / 2)) * 2, a0, a1);
        }
        return all_ok;
    }
    const int s = tid & 15;
    for (int e = e0 + (tid >> 4); e < e1; e += NT / 16) {
        float a0, a1;
        typedef std::integral_constant<int, 16> Row;
        if (nsplit <= 16) gather(One{}, Row{}, e, s, a0, a1);
        else if (nsplit <= 32) gather(std::integral_constant<int, 2>{}, Row{}, e, s, a0, a1);
        else gather(std::integral_constant<int, kMaxSplits / 16>{}, Row{}, e, s, a0, a1);
        if (all_ok && s == 0) xio.put_merged(M, b, j * G + e / (HD / 2), HD, (e % (HD / 2)) * 2, a0, a1);
    }
    return all_ok;
}

// Number of KV splits for a sequence with `ncache` cached rows when `share` workgroups are
// available per (sequence, kv head).
// Slices for workgroups of four waves at head dimension 64 (row-partitioned kernel): whole 64 rows, up to 16, then 16 for every 4096 rows.  (Shorter ones are
// done sooner there by less than the merge of more parts takes.  Us per step, three layers of d 2048 on 40 workgroups, by attn_nsplit / this: context 100 bf16 311 / 306, int8 379 / 374, int4
// 435 / 430; 250 int4 437 / 436; 2500 bf16 336 / 334, int4 458 / 459.)
__device__ __forceinline__ int attn_nsplit_few(int ncache, int share) {
    const int ns = ncache / 64;
    return max(min(ns > 16 ? 16 * ((ncache + 4095) / 4096) : ns, min(share, kMaxSplits)), 1);
}
__device__ __forceinline__ int attn_nsplit(int ncache, int share, int hd) {
    // Up to 640 rows (head dimension 64: 320) slices are no longer than four of the workgroup's waves take at once (16 rows each; head dimension 64: 8): a fifth wave shares a SIMD with the
    // first, and both take longer than the merge gets shorter.  Up to eight slices their number is a power of two, whose shares of the merge are equal, unless there are fewer workgroups;
    // from eleven on it is sixteen, with as many rows as it takes.
    // (Us per step, one sequence, ncache / 64 slices / this.  8B int4, eight layers, context 200 295 / 291, 400 307 / 294, 512 297 / 295, 900 316 / 309; 600, as
    // 10 slices 305, as 16 311; 100 as one slice 289, as two 291; 70B bf16, six layers, 400 1628 / 1613; tiny, context 128 81.5 / 79.2, 400 87.2 / 81.0, 1000 85.6 / 83.3.
    // 8B int4 x 4, context 500, 459 / 440.)
    const int rows = hd == 64 ? 32 : 64;
    if (ncache < 2 * rows) return 1;
    int ns = (ncache + rows - 1) / rows;
    if (ns <= 8) ns = ns <= 2 ? 2 : ns <= 4 ? 4 : 8;
    // The merge gathers the partials 16 at a time, two or four to a lane: 16 slices up to 1599 rows (100 each), 32 up to 8192 (50 to 256), then whole rounds of 16 of at most 256 rows, up to
    // kMaxSplits; behind 16384 rows these grow.  (Us per step, one sequence, 16 / 32 slices: 8B, eight layers, int4, context 1600 321 / 318, 2048 325 / 321, 4096 343 / 330; int8, 1500
    // 418 / 423, 2500 430 / 425, 4096 441 / 431; bf16 4096 737 / 721; 70B bf16, six layers, 4096 1659 / 1646.  Head dimension 64, d 2048, eight layers, 1599 rows as 16 / 1600 as 32: bf16 297 / 294, int8
    // 225 / 220, int4 211 / 208; tiny 86 / 84, 84 / 81, 84 / 83.)
    constexpr int kRound = 16, kRoundRows = kRound * 256;
    if (ns > 10) ns = ncache >= 1600 && ncache <= 2 * kRoundRows ? 2 * kRound : kRound * ((ncache + kRoundRows - 1) / kRoundRows);
    return max(min(ns, min(share, kMaxSplits)), 1);
}

// ---------------------------------------------------------------- epilogues
// No epilogue of the fused kernel issues a global LOAD: vector-memory operations of a wave complete
// in issue order, so a load in the middle of the weight stream would drain the whole prefetch
// pipeline.  What an epilogue needs beyond the dot products comes from LDS (RoPE cos/sin) or from
// scalar loads (positions).
//
// QKV rows in packed order: q heads then k heads with RoPE partners (i, i+hd/2) adjacent, then v.
template <class IO>
struct EpiQKV {
    const DevModel& M; const DevKV& KV; const int* tokens; const int* pos; int layer;
    const float2* rope;   // [batch][hd/2] (cos, sin) of each sequence's position; LDS in the fused kernel
    __device__ __forceinline__ void operator()(int pair, int b, float v0, float v1) const {
        const int half = M.hd / 2;
        const int nq = M.Hq * half, nk = M.Hkv * half;
        const int p = as_global(tokens)[b] == kTokenSkip ? -1 : as_global(pos)[b];   // -1: the cache of this sequence is not touched
        if (pair < nq + nk) {
            bool isq = pair < nq;
            int pp = isq ? pair : pair - nq;
            int head = pp / half, i = pp % half;
            float2 cs = rope[b * half + i];
            float a = v0 * cs.x - v1 * cs.y;
            float c = v1 * cs.x + v0 * cs.y;
            if (isq) {
                float* qp = M.q + ((size_t)b * M.Hq + head) * M.hd;
                IO::st(qp + i, a); IO::st(qp + i + half, c);
            } else {
                bf16_t ab = f_to_bf(a), cb = f_to_bf(c);
                bf16_t* row = KV.plane(M, layer, b, head, 0) + (size_t)p * M.hd;
                if (p >= 0) { as_global(row)[i] = ab; as_global(row)[i + half] = cb; }
                float* kc = M.kvcur + ((size_t)b * 2 + 0) * M.Hkv * M.hd + (size_t)head * M.hd;
                IO::st(kc + i, bf_to_f(ab)); IO::st(kc + i + half, bf_to_f(cb));
            }
        } else {
            int pp = pair - nq - nk;
            int head = pp / half, i = (pp % half) * 2;
            bf16_t ab = f_to_bf(v0), cb = f_to_bf(v1);
            bf16_t* row = KV.plane(M, layer, b, head, 1) + (size_t)p * M.hd;
            if (p >= 0) *as_global((u32*)(row + i)) = (u32)ab | ((u32)cb << 16);
            float* vc = M.kvcur + ((size_t)b * 2 + 1) * M.Hkv * M.hd + (size_t)head * M.hd;
            IO::st2(vc + i, bf_to_f(ab), bf_to_f(cb));
        }
    }
};
// Per-operation kernels: x[b][row] += W row . input
struct EpiResidual {
    float* x; int d;
    __device__ __forceinline__ void operator()(int pair, int b, float v0, float v1) const {
        FF_GLOBAL f32x2* p = as_global((f32x2*)(x + (size_t)b * d + 2 * pair));
        f32x2 o = *p;
        *p = f32x2{o.x + v0, o.y + v1};
    }
};
// packed rows (2i, 2i+1) = (gate_i, up_i):  h_i = silu(gate_i) * up_i
template <class IO>
struct EpiSwiGLU {
    float* h; int F; GuPerm perm;
    __device__ __forceinline__ void operator()(int pair, int b, float g, float u) const {
        float s = g / (1.0f + expf(-g));
        IO::st(h + (size_t)b * F + perm.unit_of_pair(pair), s * u);
    }
};
// ---- fused-kernel epilogues: outputs go to the tagged exchange buffers ----
struct EpiQKVTagged {   // pos: positions of this step, staged in LDS (-1: the sequence sits the step out, its cache is not touched)
    const DevModel& M; const DevKV& KV; const int* pos; int layer; const float2* rope; u32 tag; int hd;   // hd: a constant of the kernel instance, so that the row arithmetic is shifts
    __device__ __forceinline__ void operator()(int pair, int b, float v0, float v1) const {
        const int half = hd / 2;
        const int nq = M.Hq * half, nk = M.Hkv * half;
        const int p = pos[b];
        if (pair < nq + nk) {
            bool isq = pair < nq;
            int pp = isq ? pair : pair - nq;
            int head = pp / half, i = pp % half;
            float2 cs = rope[b * half + i];
            float a = v0 * cs.x - v1 * cs.y;
            float c = v1 * cs.x + v0 * cs.y;
            if (isq) {
                tagged_t* qp = M.tq + ((size_t)b * M.Hq + head) * hd;
                tst(qp + i, a, tag); tst(qp + i + half, c, tag);
            } else {
                bf16_t ab = f_to_bf(a), cb = f_to_bf(c);
                bf16_t* row = KV.plane(M, layer, b, head, 0) + (size_t)p * hd;
                if (p >= 0) { as_global(row)[i] = ab; as_global(row)[i + half] = cb; }
                tagged_t* kc = M.tkvcur + ((size_t)b * 2 + 0) * M.Hkv * hd + (size_t)head * hd;
                tst(kc + i, bf_to_f(ab), tag); tst(kc + i + half, bf_to_f(cb), tag);
            }
        } else {
            int pp = pair - nq - nk;
            int head = pp / half, i = (pp % half) * 2;
            bf16_t ab = f_to_bf(v0), cb = f_to_bf(v1);
            bf16_t* row = KV.plane(M, layer, b, head, 1) + (size_t)p * hd;
            if (p >= 0) *as_global((u32*)(row + i)) = (u32)ab | ((u32)cb << 16);
            tagged_t* vc = M.tkvcur + ((size_t)b * 2 + 1) * M.Hkv * hd + (size_t)head * hd;
            tst2(vc + i, bf_to_f(ab), bf_to_f(cb), tag);
        }
    }
};
struct EpiDeltaTagged {   // projections feeding the residual stream: publish the output, the next
    cword_t* delta; int d; u32 tag;    // normalised staging adds it (paper Section 4.2: added to the residual)
    __device__ __forceinline__ void operator()(int pair, int b, float v0, float v1) const { cst2(delta + (size_t)b * d + 2 * pair, v0, v1, tag); }
};
struct EpiSwiGLUTagged {   // packed rows (2i, 2i+1) = (gate_i, up_i):  h_i = silu(gate_i) * up_i
    cword_t* h; int F; u32 tag; GuPerm perm;
    __device__ __forceinline__ void operator()(int pair, int b, float g, float u) const {
        float s = g / (1.0f + expf(-g));
        cst1(h + (size_t)b * F + perm.unit_of_pair(pair), s * u, tag);
    }
};
struct EpiStore {   // plain output rows (logits; per-op raw projections)
    float* y; int n;
    u32 skip = 0;   // bit b set: row b is not written (logits of a sequence that sits the step out)
    __device__ __forceinline__ void operator()(int pair, int b, float v0, float v1) const {
        if ((skip >> b) & 1u) return;
        FF_GLOBAL float* p = as_global(y + (size_t)b * n + 2 * pair);
        p[0] = v0;
        if (2 * pair + 1 < n) p[1] = v1;
    }
};

}  // namespace ff
