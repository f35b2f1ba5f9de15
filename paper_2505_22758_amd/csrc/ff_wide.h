// The wide pass: exchange between workgroups, epilogues and the kernel.
//
// In the kernels for one sequence every workgroup prepares the whole input itself (load
// the exchanged words, normalise, convert), replicated 256 times, which would grow with the batch.  The wide pass exchanges activations in
// the form their consumers multiply, produced once by the workgroup that OWNS the value:
//   * every workgroup owns a fixed range of rows of the residual stream (the rows of the output
//     and down projections it computes, N / workgroups) and keeps them in its LDS for the whole step;
//     the epilogue of those two projections adds the projection output to its rows, and writes
//     (gain of the next normalised projection) x (new value) as bf16 head + bf16 remainder (one sequence: three parts) straight
//     into a global IMAGE in the matrix cores' operand order, plus the workgroup's share of every
//     sequence's sum of squares (the 1/rms factor is applied by the consumer to its finished sums:
//     a scalar per sequence that commutes with the projection);
//   * the SwiGLU epilogue and the attention merge write their outputs into such images too;
//   * a consumer loads the image straight into operand registers, 16 bytes per lane and load.
// The dependency is carried by one epoch word per workgroup and phase (paper Section 4.1: the global
// barrier between dependent phases): a producer's waves make their exchange stores (all write-through,
// agent scope) and wait until they have completed; the last wave to get there publishes the phase's
// epoch; a consumer polls until all workgroups show it.  Images are read with plain cacheable loads,
// which the workgroups of an XCD serve each other out of their L2.  No cached copy can be stale,
// because no image is written twice in a launch: every layer has images of its own (M.wring of them;
// a launch starts with clean caches).  Where the caller's scratch has no room for that (wring == 1)
// a consumer drops its cached copies with an acquire fence, and write-after-read is ordered by the
// epochs (an image is rewritten only by workgroups that have waited for an epoch which every
// reader of the old contents published after its last read).
// Queries, keys, values and attention partials keep their tagged 8-byte format.
// Measured us per step of an 8-layer block, before (four waves, images copied through LDS, row-major weights) / with
// this kernel on row-major / on tiled weights: 8B bf16 x 8 1127 / 1003 / 834, int8 x 11 992 / 936 / 770, int4 x 16 1628 /
// 978 / 783, 70B bf16 x 16 3283 / 3098 / 2619; against a row-partitioned pass of up to four sequences (4x4x4 matrix-core
// tiles, inputs staged by every workgroup): bf16 x 2 858 / 769, int4 x 4 1038 / 570, int8 x 4 879 / 581.  Since (merge of the attention
// slices shared out, descriptors in LDS, attention scores on the matrix cores, int4 panels without tails): bf16 x 2 735, x 8 779, int8 x 4 534, x 11 701, int4 x 4
// 509, x 16 723.
// What bounds it: the weight stream, then the attention's chain of hand-overs (a third of a layer).
#pragma once
#include "ff_dense.h"

namespace ff {

// ---------------------------------------------------------------- LDS
constexpr int kWideAttnBytes = kWideRedBytes + kWideSzBytes;   // the projections' regions; the attention's (attn_item) lies inside
constexpr int kWideRopeOff = kWideAttnBytes;
constexpr int kWideResOff = kWideRopeOff + kMaxBatchWide * 64 * 8;     // residual rows of the workgroup: [sequence][kWideResRows]
constexpr int kWideResRows = 32;
constexpr int kWideRmsOff = kWideResOff + kMaxBatchWide * kWideResRows * 4;   // sums of squares: [wave][sequence]
constexpr int kWideIntOff = kWideRmsOff + kWideWaves * kMaxBatchWide * 4;     // positions, attention shares, epoch verdicts, arrival counter, vote slots
constexpr int kWideTabOff = kWideIntOff + 512;   // WideMat of the five projections
constexpr int kWideItemOff = kWideTabOff + 320;  // the workgroup's attention items
constexpr int kWideMaxCtas = 256;   // workgroups whose sums of squares a consumer gathers in one round (wide_project)
constexpr int kWideLdsBytes = kWideIntOff + 1024;
static_assert(kWideLdsBytes <= 160 * 1024, "LDS layout of the wide pass");
static_assert((kAttnStateFloats<128, 8, kWideWaves> + AttnParts<128, 8>::kWords) * 4 <= kWideAttnBytes, "attention state");

// A projection as its phases find it in LDS (kinds PH_QKV .. PH_LM): pointers of layer 0, advanced by the layers' stride, and the gains of the norm
// behind it.  (Read out of the layer table where they are needed, the descriptors of a layer that nobody has touched yet are
// misses all the way to memory between one projection and the next: 8B, eight layers, us per step, bf16 x 2 740 -> 735, x 8 784 -> 779,
// int8 x 4 540 -> 534, int4 x 16 731 -> 723; int4 x 4, whose code was the longest, lost: 525 -> 529, and has since gained more by panels
// without tails, panel_run.)
struct WideMat { u64 w, s, z, gain; int n, k, r0, r1, np, T; };   // r0, r1: the workgroup's rows; np panels of T tiles
typedef __attribute__((address_space(3))) WideMat lds_wmat;
static_assert(5 * sizeof(WideMat) <= 320 && kAttnListed * sizeof(AttnItem) <= 512 - 320, "descriptors and items in LDS");
// A value known to be the same in all lanes (in host code: the value).
__host__ __device__ __forceinline__ int uni(int v) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_readfirstlane(v);
#else
    return v;
#endif
}
__host__ __device__ __forceinline__ u64 uni(u64 v) { return (u64)(u32)uni((int)(u32)v) | ((u64)(u32)uni((int)(u32)(v >> 32)) << 32); }
// A projection's panels, as few as possible, of equal size (the same for every workgroup: the largest share decides).
struct WideShape {
    RowRange rr;
    int np, T;
    __device__ __forceinline__ static WideShape of(int n, const UDiv& n_ctas) {
        const int tiles = ((4 * (int)n_ctas.div((u32)(n + 3) / 4 + n_ctas.n - 1u)) + 15) >> 4, np = (tiles + kPanelTiles - 1) / kPanelTiles;
        return WideShape{wide_rows(n, n_ctas), np, (int)((u32)(tiles + np - 1) / (u32)np)};
    }
};
__device__ __forceinline__ void wide_table(lds_wmat* tab, const DevModel& M, const UDiv& n_ctas, int kind) {   // entry `kind`, by one thread
    const PLayer* L = M.layers + (kind == PH_LM ? M.L : 0);
    const PMat* W = &L->qkv + (kind & 3);
    tab[kind].w = (u64)W->w; tab[kind].s = (u64)W->s; tab[kind].z = (u64)W->z;
    tab[kind].n = W->n; tab[kind].k = W->k;
    const WideShape S = WideShape::of(W->n, n_ctas);
    tab[kind].r0 = S.rr.r0; tab[kind].r1 = S.rr.r1; tab[kind].np = S.np; tab[kind].T = S.T;
    tab[kind].gain = kind == PH_O ? (u64)L->g2 : kind == PH_DOWN ? (u64)L->g1 : 0;   // (the gains behind a down projection: the next layer's)
}
template <int WD>
__device__ __forceinline__ PMat wide_mat(const lds_wmat* tab, const DevModel& M, int kind, int l) {
    const lds_wmat* e = tab + kind;
    const size_t off = kind == PH_LM ? 0 : (size_t)l * M.layer_stride;
    PMat W{};
    W.w = (const uint8_t*)(uni(e->w) + off);
    W.s = (const f16_t*)(uni(e->s) + off); W.z = (const f16_t*)(uni(e->z) + off);
    W.n = uni(e->n); W.k = uni(e->k);
    W.wd = WD; W.tiled = 1;   // (tiled: not zero)
    return W;
}

__device__ __forceinline__ WideShape wide_shape(const lds_wmat* e) { return WideShape{RowRange{uni(e->r0), uni(e->r1)}, uni(e->np), uni(e->T)}; }

// ---------------------------------------------------------------- epochs
struct WideSync {
    u32* flags;       // [workgroups] last epoch each workgroup has published
    int ncta;
    bool fence;       // images are reused within the launch
    lds_u32* slots;   // [2] verdicts (alternating), [2] arrival counter
    u32 par;
    // This wave's exchange stores of the phase are made.  Every wave calls this once per epoch; the last one publishes it.
    __device__ __forceinline__ void arrive(u32 epoch, int lane) const {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the write-through stores have completed
        if (lane == 0) {
            const u32 old = __hip_atomic_fetch_add(slots + 2, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if ((old & (kWideWaves - 1)) == kWideWaves - 1) xst_u32(flags + blockIdx.x, epoch);
        }
        asm volatile("" ::: "memory");
    }
    // Every workgroup has published `epoch` (or a later one).  Returns false (uniformly) on a time-out.
    // (Four flags per lane; workgroups beyond ncta do not exist.  The verdict slots alternate, so one barrier will do:
    // a slot is rewritten two waits later, behind the barrier of the wait in between.)
    __device__ __forceinline__ bool wait(u32 epoch, int wave, int lane) {
        if (!flags) { __syncthreads(); return true; }   // (a projection on its own: nothing to wait for)
        par ^= 1u;
        if (wave == 0) {
            bool ok = false;
            for (int spins = 0; spins < kSpinLimit && !ok; spins++) {
                bool mine = true;
                for (int i = 2 * lane; i < ncta; i += 128) {
                    const u64 f = __hip_atomic_load(as_global((const u64*)(flags + i)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    mine = mine && (int)((u32)f - epoch) >= 0 && (i + 1 >= ncta || (int)((u32)(f >> 32) - epoch) >= 0);
                }
                ok = __all(mine);
                if (!ok) __builtin_amdgcn_s_sleep(1);
            }
            if (fence) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // cached copies of the images' earlier contents are dropped
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            if (lane == 0) slots[par] = ok ? 1u : 0u;
        }
        __syncthreads();
        return __builtin_amdgcn_readfirstlane((int)slots[par]) != 0;
    }
};

// ---------------------------------------------------------------- images
// Layer l's block of the exchange region: input images of the QKV (block L: LM head), gate/up, output and
// down projections, and the workgroups' sums of squares of the first two ([tile of the workgroup's rows][workgroup][16]).
__host__ __device__ inline int wide_img_cols(int K, int wd) {   // whole iterations
    const int cols = wd == W_INT4 ? 128 : 64;
    return (K + cols - 1) / cols * cols;
}
__host__ __device__ inline size_t wide_img_bytes(int K, int wd, int max_batch) { return (size_t)wide_img_cols(K, wd) / 32 * wide_step_bytes(max_batch == 1 ? 1 : kMaxBatchWide, max_batch); }   // (two sequences take what one does)
struct WideLayout {
    size_t x1, x2, a, h, ss1, ss2, bytes;
    __host__ __device__ static WideLayout of(int d, int qd, int F, int wd, int max_batch, int ncta) {
        WideLayout W;
        size_t o = 0;
        W.x1 = o; o += wide_img_bytes(d, wd, max_batch);
        W.x2 = o; o += wide_img_bytes(d, wd, max_batch);
        W.a = o; o += wide_img_bytes(qd, wd, max_batch);
        W.h = o; o += wide_img_bytes(F, wd, max_batch);
        W.ss1 = o; o += (size_t)2 * ncta * kMaxBatchWide * 4;
        W.ss2 = o; o += (size_t)2 * ncta * kMaxBatchWide * 4;
        W.bytes = (o + 255) & ~(size_t)255;
        return W;
    }
};

// ---------------------------------------------------------------- epilogues
struct WideCtx {
    const DevModel& M; const DevKV& KV; const int* pos; const float2* rope; float* logits;
    int batch, layer, kind;
    u32 tag;               // of q, k, v
    WideImg out;           // image this projection writes (SwiGLU, residual)
    float* ss;             // sums of squares beside it (residual)
    float* xres;           // LDS: residual rows of this workgroup
    RowRange own;
    int hd;                // head dimension (a constant of the kernel instance: the row arithmetic of q, k, v is shifts)
};
// Rows row .. row + 3 (nv of them real) for sequence n with the finished sums c; gw: the next norm's gains of these rows.
__device__ __forceinline__ float wide_residual(const WideCtx& C, int row, int n, const f32x4& c, const u32x2& gw) {
    float* xp = C.xres + n * kWideResRows + (row - C.own.r0);
    f32x4 x = *(const f32x4*)xp;
    x += c;
    *(f32x4*)xp = x;
    C.out.put4(n, row, x.x * bf_lo(gw.x), x.y * bf_hi(gw.x), x.z * bf_lo(gw.y), x.w * bf_hi(gw.y));
    return (x.x * x.x + x.y * x.y) + (x.z * x.z + x.w * x.w);
}
// Packed pair q of a tiled gate/up matrix is FFN unit q; a quad of rows gives the neighbouring units f, f + 1 (f even).
__device__ __forceinline__ void wide_swiglu(const WideCtx& C, int f, int n, const f32x4& c, bool two) {
    const float h0 = c.x / (1.0f + expf(-c.x)) * c.y, h1 = two ? c.z / (1.0f + expf(-c.z)) * c.w : 0.f;
    C.out.put2(n, f, h0, h1);   // (a missing second unit is padding, zero in the image)
}
// Four rows of the QKV projection (row a multiple of four, all of one head): two RoPE pairs (i, i + hd / 2) and
// (i + 1, i + 1 + hd / 2) of a query or key head, or four value rows.
__device__ __forceinline__ void wide_qkv(const WideCtx& C, int row, int n, const f32x4& c) {
    const DevModel& M = C.M;
    const int hd = C.hd, half = hd / 2, nq = M.Hq * hd, nk = M.Hkv * hd, p = C.pos[n];   // (p < 0: the sequence sits the step out, its cache is not touched)
    if (row < nq + nk) {
        const bool isq = row < nq;
        const int r = isq ? row : row - nq, head = r / hd, i = (r % hd) / 2;
        const float4 cs = *(const float4*)(C.rope + n * half + i);
        const float a0 = c.x * cs.x - c.y * cs.y, b0 = c.y * cs.x + c.x * cs.y, a1 = c.z * cs.z - c.w * cs.w, b1 = c.w * cs.z + c.z * cs.w;
        if (isq) {
            tagged_t* q = M.tq + ((size_t)n * M.Hq + head) * hd + i;
            tst2(q, a0, a1, C.tag);
            tst2(q + half, b0, b1, C.tag);
        } else {
            const u32 a = (u32)f_to_bf(a0) | ((u32)f_to_bf(a1) << 16), b = (u32)f_to_bf(b0) | ((u32)f_to_bf(b1) << 16);
            tagged_t* k = M.tkvcur + ((size_t)(n * 2) * M.Hkv + head) * hd + i;
            tst2(k, bf_lo(a), bf_hi(a), C.tag);
            tst2(k + half, bf_lo(b), bf_hi(b), C.tag);
            if (p >= 0) {
                bf16_t* kr = C.KV.plane(M, C.layer, n, head, 0) + (size_t)p * hd + i;
                *as_global((u32*)kr) = a;
                *as_global((u32*)(kr + half)) = b;
            }
        }
    } else {
        const int r = row - nq - nk, head = r / hd, i = r % hd;
        const u32 a = (u32)f_to_bf(c.x) | ((u32)f_to_bf(c.y) << 16), b = (u32)f_to_bf(c.z) | ((u32)f_to_bf(c.w) << 16);
        tagged_t* v = M.tkvcur + ((size_t)(n * 2 + 1) * M.Hkv + head) * hd + i;
        tst2(v, bf_lo(a), bf_hi(a), C.tag);
        tst2(v + 2, bf_lo(b), bf_hi(b), C.tag);
        if (p >= 0) *as_global((u32x2*)(C.KV.plane(M, C.layer, n, head, 1) + (size_t)p * hd + i)) = u32x2{a, b};
    }
}
__device__ __forceinline__ void wide_epilogue(const WideCtx& C, int row, int n, const f32x4& c, int nv) {
    const int pair = row >> 1;
    if (C.kind == PH_QKV) {
        wide_qkv(C, row, n, c);   // (the number of rows is a multiple of the head dimension: all four are there)
    } else if (C.kind == PH_GU) {
        wide_swiglu(C, pair, n, c, nv > 2);
    } else if (C.pos[n] >= 0) {   // LM head (no logits for a sequence that sits the step out)
        FF_GLOBAL float* y = as_global(C.logits + (size_t)n * C.M.V + row);
        if (nv == 4 && (C.M.V & 3) == 0 && ((uintptr_t)C.logits & 15) == 0) *(FF_GLOBAL f32x4*)y = c;
        else {
            y[0] = c.x;
            if (nv > 1) y[1] = c.y;
            if (nv > 2) y[2] = c.z;
            if (nv > 3) y[3] = c.w;
        }
    }
}
// The residual epilogue's sums of squares over the tile's rows: lanes n, n + 16, n + 32, n + 48 hold the four quads of sequence n.
__device__ __forceinline__ void wide_store_ss(float* ss, int ncta, int t, int lane, float v) {
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (lane < kMaxBatchWide) xst(ss + ((size_t)t * ncta + blockIdx.x) * kMaxBatchWide + lane, v);
}

// ---------------------------------------------------------------- one projection
// img: the input image; ssin: the workgroups' sums of squares of a normalised input (null: not normalised).
// epoch: what to wait for.  Returns false (uniformly) on a time-out.
// RES: the projections that add to the residual (output, down), whose outputs the next norm's gains multiply; at most two tiles, one panel.
// FAR: int4 rows too long for their panel's scales in LDS (panel_scales_far).
// LATE: where the panel's end takes what it knows of the lane anew, behind the products: else its addresses are computed ahead of them.  They are then spilled over the products with int4
// weights, with head dimension 64 and in the bf16 and int8 steps of one sequence, which are the faster for it all the same.  (Us per step, ahead / late: int4, 8B, eight layers, one
// sequence 426 / 421, x 4 447 / 440; bf16 x 2 681 / 671, x 8 737 / 729; one sequence, head dimension 64, eight layers, bf16 353 / 351, int8 300 / 298; but one sequence 8B bf16 684 / 693, int8 477 /
// 485, and int8, tiny, x 16 124 / 128.)
template <int WD, int NC, int HD> constexpr bool kWideLate = WD == W_INT4 || (WD == W_BF16 && NC > 1) || (NC == 1 && HD == 64);
template <int WD, int NC, int T, bool RES, bool FAR, bool LATE>
__device__ __forceinline__ bool wide_project(const PMat& W, const RowRange rr, int npanels, const uint8_t* img, const float* ssin, const bf16_t* gain, u32 epoch,
                                             WideSync& sync, const WideCtx& C, uint8_t* lds, int wave, int lane_in, int ph) {
    // (what depends on the lane only is cheap to compute again: kept from being hoisted out of the phase loop, where it would be spilled)
    int lane = lane_in;
    asm volatile("" : "+v"(lane));
    const int tid = wave * 64 + lane;
    auto timed = [&](int ev) { if (C.M.dbg && blockIdx.x == 0 && tid == 0) as_global(C.M.dbg)[ph * kEvSlots + ev] = wall_clock64(); };
    lds_float* red = (lds_float*)lds;
    lds_f16* sz = (lds_f16*)(lds + kWideRedBytes);
    float* rms = (float*)(lds + kWideRmsOff);
    const int ni = (W.k + kWCols<WD> - 1) / kWCols<WD>;
    const WaveIters I = WaveIters::of(ni, wave);
    constexpr int D = PanelRing<WD, NC, T>::D;
    PanelRing<WD, NC, T> R;
    PanelSrc<T> S;
    u32x2 pre = {0u, 0u}, gpre = {0u, 0u};
    auto prows = [&](int p) { return min(16 * T, rr.r1 - (rr.r0 + 16 * T * p)); };   // rows of panel p (<= 0 for a workgroup without rows)
    auto item_row = [&](int p, int lane_) { return rr.r0 + 16 * (T * p + wave) + 4 * (lane_ >> 4); };   // first row of the item this thread finishes
    // Everything a panel needs that does not depend on this step's activations.  All of it is loaded unconditionally, from clamped addresses.
    auto prefetch = [&](int p) {
        const int p0 = min(rr.r0 + 16 * T * p, W.n - 1), nr = prows(p);
        if constexpr (WD == W_INT8) pre = *as_global((const u32x2*)(W.s + (min(item_row(p, lane), W.n - 1) & ~3)));   // row scales of the item
        if constexpr (WD == W_INT4 && !FAR) if (nr > 0) panel_scales_send(W, p0, nr, T, (u32)(size_t)(sz + (p & 1) * (kSzHalf / 2)), wave, lane);
        __builtin_amdgcn_sched_barrier(0);
        S = PanelSrc<T>::make(W, p0, max(rr.r1, p0 + 1), lane);
#pragma unroll
        for (int j = 0; j < D; j++) R.load_w(S, j, I.at(j), WD != W_INT4 || NC > 8 || j < I.n);
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (RES) gpre = *as_global((const u32x2*)(gain + (min(item_row(0, lane), W.n - 1) & ~3)));   // gains of the next norm
    prefetch(0);
    timed(EV_PF_ISSUED);
    if constexpr (WD == W_INT4 && !FAR) panel_scales_wait<D * T>();   // (read behind the barrier in the wait)
    if (!sync.wait(epoch, wave, lane)) return false;
    timed(EV_SYNCED);
    const PanelImg X = PanelImg::make<WD, NC>(img, W.k, C.batch, lane);
    for (int p = 0;; p++) {
        mfma_f4 acc[T];
#pragma unroll
        for (int t = 0; t < T; t++) acc[t] = mfma_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < PanelRing<WD, NC, T>::DX; j++) R.load_x(X, j, I.at(j), WD != W_INT4 || NC > 8 || j < I.n);
        __builtin_amdgcn_sched_barrier(0);
        const int p0 = min(rr.r0 + 16 * T * p, W.n - 1);
        const PanelSz from{sz + (p & 1) * (kSzHalf / 2) + panel_skew(p0, W.k), panel_zeros(W.k, T), W.k / 128};
        if constexpr (!FAR) panel_run<WD, NC, T>(S, R, X, I, from, nullptr, wave, lane, acc);
        else {
            const PanelSzFar far{W.s + (size_t)p0 * from.ng, W.z + (size_t)p0 * from.ng, from.ng, rr.r1 - p0};
            panel_run<WD, NC, T, true>(S, R, X, I, PanelSz{sz, 0, 0}, &far, wave, lane, acc);
        }
        timed(p == 0 ? 4 : 8);
        if (p == 0 && C.M.dbg && C.layer == 1 && lane == 0) as_global(C.M.dbg)[(size_t)(4 * C.M.L + 1) * kEvSlots + (blockIdx.x * kWideWaves + wave) * 4 + (C.kind & 3)] = wall_clock64();
        __builtin_amdgcn_sched_barrier(0);
        int late = lane;
        if constexpr (LATE) {
            late = lane_in;
            asm volatile("" : "+v"(late));
        }
        const int tid = wave * 64 + late, q = late >> 4, seq = late & 15;
        if (!RES && p == 0 && ssin) {   // the workgroups' sums of squares, in a fixed order
            float ssv[16], t = 0.f;
#pragma unroll
            for (int i = 0; i < 16; i++)
                ssv[i] = as_global(ssin)[((size_t)(i >> 3) * sync.ncta + min((tid >> 4) + 32 * (i & 7), sync.ncta - 1)) * kMaxBatchWide + seq];
#pragma unroll
            for (int i = 0; i < 16; i++) t += (tid >> 4) + 32 * (i & 7) < sync.ncta ? ssv[i] : 0.f;
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            if (late < kMaxBatchWide) rms[wave * kMaxBatchWide + late] = t;
        }
        if (p > 0) __syncthreads();   // the previous panel's partial tiles have been read
        panel_put<T, NC>(red, acc, wave, late);
        const u32x2 rowscale = pre;
        const bool more = !RES && p + 1 < npanels;
        if (more) {   // the next panel's first weights, while this one is finished
            prefetch(p + 1);
            if constexpr (WD == W_INT4 && !FAR) panel_scales_wait<D * T>();
        }
        __syncthreads();
        timed(p == 0 ? 5 : 9);
        if (wave < T) {
            const int row = item_row(p, late);
            float rs = 1.f;
            if (!RES && ssin) {
                float t = 0.f;
#pragma unroll
                for (int w = 0; w < kWideWaves; w++) t += rms[w * kMaxBatchWide + seq];
                rs = rsqrtf(t / (float)W.k + C.M.eps);
            }
            f32x4 c = panel_get<NC, T>(red, wave, q, NC == 8 ? seq & 7 : seq) * rs;
            if constexpr (WD == W_INT8)
                c *= f32x4{f16_to_f((f16_t)(rowscale.x & 0xFFFFu)), f16_to_f((f16_t)(rowscale.x >> 16)), f16_to_f((f16_t)(rowscale.y & 0xFFFFu)), f16_to_f((f16_t)(rowscale.y >> 16))};
            const bool mine = row < rr.r1 && seq < C.batch;
            if constexpr (RES) {
                const float v = mine ? wide_residual(C, row, seq, c, gpre) : 0.f;
                wide_store_ss(C.ss, sync.ncta, wave, late, v);
            } else if (mine) wide_epilogue(C, row, seq, c, min(4, rr.r1 - row));
        }
        if (!more) return true;
    }
}

// int4: whether rows of k columns are too long for LDS to hold the scales of a panel of T tiles.  (One or two tiles are one panel; for inputs of d_model columns, those
// of wider ones, the host checks that they fit.)
__host__ __device__ __forceinline__ bool wide_sz_far(int k, int T) { return T <= 2 && 4 * panel_zeros(k, T) > kWideSzBytes; }
// LONG: there may be such rows.
template <int WD, int NC, bool RES, bool LONG, bool LATE>
__device__ __forceinline__ bool wide_project_any(const PMat& W, const WideShape& S, const uint8_t* img, const float* ssin, const bf16_t* gain, u32 epoch, WideSync& sync, const WideCtx& C,
                                                 uint8_t* lds, int wave, int lane, int ph) {
#define FF_WIDE_T(t, far) case t: return wide_project<WD, NC, t, RES, far, LATE>(W, S.rr, S.np, img, ssin, gain, epoch, sync, C, lds, wave, lane, ph);
    if constexpr (WD == W_INT4 && LONG) if (wide_sz_far(W.k, S.T)) {
        switch (S.T) { FF_WIDE_T(1, true) FF_WIDE_T(2, true) }
        return false;
    }
    if constexpr (RES) {
        static_assert(kWideResRows <= 32, "tiles of a workgroup's residual rows");
        switch (S.T) { FF_WIDE_T(1, false) FF_WIDE_T(2, false) }
    } else
        switch (S.T) { FF_WIDE_T(1, false) FF_WIDE_T(2, false) FF_WIDE_T(3, false) FF_WIDE_T(4, false) FF_WIDE_T(5, false) FF_WIDE_T(6, false) FF_WIDE_T(7, false) }
#undef FF_WIDE_T
    return false;
}

// ---------------------------------------------------------------- the kernel
// One launch = one step of up to NC sequences (phases as in fused_decode_kernel).  One sequence has an instance of its own:
// its step on a model for several sequences is as exact as on a model for one.
// n_lm: 1 = the LM head runs here, 0 = launched separately.  LONG: rows of the output and down projections may be too long for their scales in LDS (wide_sz_far).  Above
// eight sequences they have an instance of their own: their code in the way of the others costs these up to 2 % (us per step, eight layers, x 16, with / without: 1b 334 / 332,
// 3b 397 / 394; tiny 127 / 125); up to eight it does not (8B int4 x 1 423 / 424, x 4 420 / 421, tiny x 8 127 / 128).
template <int WD, int NC> constexpr bool kWideLong = WD == W_INT4 && NC <= 8;
template <int WD, int NC, int HD, int G, bool LONG = kWideLong<WD, NC>>
__global__ void __launch_bounds__(kWideThreads) wide_decode_kernel(DevModel M, DevKV KV, const int* __restrict__ tokens, const int* __restrict__ pos,
                                                                   float* __restrict__ logits, int n_seq, int lm_in_kernel, int ncta, int mute_wg, int switches) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int batch = NC == 1 ? 1 : n_seq;
    if (!inputs_ok(M, KV, tokens, pos)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(M.status, kStatusRange);
        return;
    }
    if ((int)blockIdx.x == mute_wg) return;   // test hook for the time-out path: this workgroup publishes nothing
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float2* rope_lds = (float2*)(lds + kWideRopeOff);   // [batch][hd/2]
    float* xres = (float*)(lds + kWideResOff);
    int* pos_lds = (int*)(lds + kWideIntOff);
    int* share_lds = pos_lds + kMaxBatchWide;
    lds_u32* slots = (lds_u32*)(share_lds + kMaxBatchWide);
    for (int i = threadIdx.x; i < batch * (M.hd / 2); i += kWideThreads) {
        const int b = i / (M.hd / 2), f = i % (M.hd / 2);
        rope_lds[i] = KV.rope[(size_t)max(step_pos(tokens, pos, b), 0) * (M.hd / 2) + f];
    }
    if ((int)threadIdx.x < batch) {
        pos_lds[threadIdx.x] = step_pos(tokens, pos, threadIdx.x);   // -1: the sequence sits this step out
        share_lds[threadIdx.x] = attn_share_of(tokens, pos, batch, threadIdx.x, ncta, M.Hkv, (switches & kSwUniformShares) != 0);
    }
    if (threadIdx.x < 4) slots[threadIdx.x] = 0u;
    lds_wmat* tab = (lds_wmat*)(lds + kWideTabOff);
    const UDiv n_ctas = UDiv::of((u32)ncta);
    if (threadIdx.x < 5) wide_table(tab, M, n_ctas, threadIdx.x);
    const u32 steps_done = (u32)__builtin_amdgcn_readfirstlane(xld_u32(M.stepctr));
    const u32 tag_base = steps_done * (u32)(kTagsPerLayer * M.L + 1);
    const u32 ebase = steps_done * (u32)(4 * M.L + 1) + 1u;   // epochs of this step: ebase: embedding rows; + 4 l + {1: attention, 2: output, 3: gate/up, 4: down projection}
    WideSync sync{M.wflag, ncta, M.wring == 1, slots, 0u};
    WgVote vote{(u32*)(slots + 4), 0u};
    const WideLayout WL = WideLayout::of(M.d, M.Hq * M.hd, M.F, WD, M.wbatch, ncta);
    constexpr int kImgE = WD == W_BF16 ? 0 : WD == W_INT8 ? 1 : 2;
    const RowRange own = wide_rows(M.d, n_ctas);
    auto block = [&](int l) { return M.wimg + (size_t)(M.wring == 1 ? 0 : l) * WL.bytes; };
    auto image = [&](uint8_t* p) { return WideImg{p, kImgE, batch, NC}; };
    auto timed = [&](int ph, int ev) { if (M.dbg && blockIdx.x == 0 && threadIdx.x == 0) as_global(M.dbg)[ph * kEvSlots + ev] = wall_clock64(); };
    __syncthreads();
    lds_item* items = (lds_item*)(lds + kWideItemOff);
    attn_list<HD, kWideWaves>(items, pos_lds, share_lds, batch, M.Hkv, n_ctas);   // (read behind the first projection's barriers)
    WideCtx C{M, KV, pos_lds, rope_lds, logits, batch, 0, PH_DOWN, 0u, image(block(0) + WL.x1), (float*)(block(0) + WL.ss1), xres, own, HD};
    // the step's embedding rows enter like the output of a projection onto zero
    if (16 * wave < kWideResRows) {
        const int row = own.r0 + 16 * wave + 4 * (lane >> 4), seq = lane & 15;
        float v = 0.f;
        if (row < own.r1 && seq < batch) {
            const int t = max(tokens[seq], 0);
            const u32x2 e = *as_global((const u32x2*)(M.embed + (size_t)t * M.d + row)), g = *as_global((const u32x2*)(as_const(M.layers)->g1 + row));
            *(f32x4*)(xres + seq * kWideResRows + (row - own.r0)) = f32x4{0.f, 0.f, 0.f, 0.f};
            v = wide_residual(C, row, seq, f32x4{bf_lo(e.x), bf_hi(e.x), bf_lo(e.y), bf_hi(e.y)}, g);
        }
        wide_store_ss(C.ss, ncta, wave, lane, v);
    }
    // Columns behind the end of a width that is not a whole number of iterations meet zero weights and have to be finite:
    // the images' layout follows the batch, so their place holds what steps of other batches left.
    {
        const int widths[4] = {M.d, M.d, M.Hq * M.hd, M.F};
        const size_t offs[4] = {WL.x1, WL.x2, WL.a, WL.h};
        for (int l = blockIdx.x; l < M.wring; l += ncta)
            for (int i = 0; i < 4; i++) {
                const int pad = wide_img_cols(widths[i], WD) - widths[i];   // (even)
                const WideImg im = image(M.wimg + (size_t)l * WL.bytes + offs[i]);
                for (int e = threadIdx.x; e < pad / 2 * batch; e += kWideThreads) im.put2(e % batch, widths[i] + 2 * (e / batch), 0.f, 0.f);
            }
    }
    sync.arrive(ebase, lane);
    const int n_phases = 4 * M.L + lm_in_kernel;
    for (int ph = 0; ph < n_phases; ph++) {
        const int l = ph >> 2;
        const u32 e0 = ebase + 4u * (u32)l;
        uint8_t* blk = block(l);
        u32 epoch = e0;
        const uint8_t* img;
        const float* ssin = nullptr;
        const bf16_t* gain = nullptr;
        C.layer = l;
        C.kind = ph == 4 * M.L ? PH_LM : (ph & 3);
        C.tag = tag_of(tag_base, l, TAG_QKV);
        if (C.kind == PH_QKV) { img = blk + WL.x1; ssin = (const float*)(blk + WL.ss1); }
        else if (C.kind == PH_O) {
            __syncthreads();   // the QKV epilogues have read their sums out of LDS
            const WideImg ai = image(blk + WL.a);
            u64* aev = M.dbg && l == 1 ? M.dbg + (size_t)(4 * M.L + 1) * kEvSlots + (size_t)ncta * 32 + ((size_t)blockIdx.x * 5 + 4) * 8 : nullptr;
            if (aev && threadIdx.x == 0) { as_global(aev)[0] = wall_clock64(); as_global(aev)[4] = 0; as_global(aev)[5] = 0; }
            bool mine = true;
            if (!attention_phase_tagged<kWideWaves, HD, G, false>(M, KV, items, pos_lds, share_lds, batch, l, lds, tag_of(tag_base, l, TAG_QKV), tag_of(tag_base, l, TAG_ATT), 0u,
                                                              n_ctas, vote, mine, aev, &ai)) return;
            if (aev && threadIdx.x == 0) as_global(aev)[6] = wall_clock64();
            if (!vote.all<kWideThreads>(mine)) return;
            sync.arrive(e0 + 1u, lane);
            timed(ph, EV_ATT_END);
            epoch = e0 + 1u; img = blk + WL.a; gain = (const bf16_t*)(uni(tab[PH_O].gain) + (size_t)l * M.layer_stride);
            C.out = image(blk + WL.x2); C.ss = (float*)(blk + WL.ss2);
        } else if (C.kind == PH_GU) {
            epoch = e0 + 2u; img = blk + WL.x2; ssin = (const float*)(blk + WL.ss2);
            C.out = image(blk + WL.h);
        } else if (C.kind == PH_DOWN) {
            epoch = e0 + 3u; img = blk + WL.h; gain = l + 1 < M.L ? (const bf16_t*)(uni(tab[PH_DOWN].gain) + (size_t)(l + 1) * M.layer_stride) : M.gf;
            uint8_t* nb = block(l + 1);
            C.out = image(nb + WL.x1); C.ss = (float*)(nb + WL.ss1);
        } else { img = blk + WL.x1; ssin = (const float*)(blk + WL.ss1); }
        const PMat W = wide_mat<WD>(tab, M, C.kind, l);
        timed(ph, EV_H_START);
        const WideShape S = wide_shape(tab + C.kind);
        const bool ok = gain ? wide_project_any<WD, NC, true, LONG, kWideLate<WD, NC, HD>>(W, S, img, nullptr, gain, epoch, sync, C, lds, wave, lane, ph)
                             : wide_project_any<WD, NC, false, false, kWideLate<WD, NC, HD>>(W, S, img, ssin, nullptr, epoch, sync, C, lds, wave, lane, ph);
        timed(ph, EV_RUN_DONE);
        if (!ok) {
            if (threadIdx.x == 0) atomicCAS(M.status, 0, -55 - 10 * ph);
            return;
        }
        if (C.kind == PH_O) sync.arrive(e0 + 2u, lane);
        else if (C.kind == PH_GU) sync.arrive(e0 + 3u, lane);
        else if (C.kind == PH_DOWN) sync.arrive(e0 + 4u, lane);
    }
    if (!lm_in_kernel) {   // LM head launched separately: the final residual rows (the last down projection's epilogues are behind this workgroup's own epoch)
        if (!sync.wait(ebase + 4u * (u32)M.L, wave, lane)) {
            if (threadIdx.x == 0) atomicCAS(M.status, 0, -55 - 10 * n_phases);
            return;
        }
        const int nrows = own.r1 - own.r0;
        for (int i = threadIdx.x; i < batch * nrows; i += kWideThreads) {
            const int b = i / nrows, r = i - b * nrows;
            as_global(M.x)[(size_t)b * M.d + own.r0 + r] = xres[b * kWideResRows + r];
        }
    }
    // workgroup 0 can only get here after every workgroup has taken part in every phase, i.e. has read the counter
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        xst_u32(M.stepctr + 1, 0u);
        xst_u32(M.stepctr, steps_done + 1u);
    }
}

}  // namespace ff
