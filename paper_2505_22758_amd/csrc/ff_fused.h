// The row-partitioned whole-model decode kernel (one persistent launch per decode step of one sequence), for what the one-sequence
// kernel (ff_solo.h) and the wide pass do not take: models wider than 8192, grids whose workgroups would own more than 32 rows of
// d_model; there it also serves the sequences of a model for several one after another.
#pragma once
#include <algorithm>
#include <mutex>
#include "ff_solo.h"

namespace ff {

// Workgroup shape of the fused kernel: one wave per SIMD, so that each wave may use the whole
// 512-entry register file of its SIMD for its tile ring.
constexpr int kFusedWaves = 4;
constexpr int kFusedThreads = kFusedWaves * 64;

__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

// ---------------------------------------------------------------- the fused whole-model kernel
// One launch = one decode step for all layers (paper abstract, Section 4).  Phases per layer:
// [RMSNorm + QKV projection + RoPE + cache append] [split-KV attention + merge] [output projection]
// [residual + RMSNorm + gate/up projection + SwiGLU] [down projection]; then residual + final norm
// + LM head.  The residual additions are folded into the staging of the next normalised
// projection, so no projection epilogue reads global memory.
//
// Synchronisation between phases is by dataflow on tagged values (see tagged_t): a phase starts in
// a workgroup as soon as the vector it consumes carries the producing phase's tag.  The paper's
// kernel separates the same phases with an atomic device-wide barrier plus fences (Section 4.1);
// on this chip a barrier round trip, the wait for store acknowledgements before it and the input
// load after it are three dependent trips through a memory pipeline that is full of weight
// traffic, so the dependency is carried by the data instead.
//
// Memory pipeline (the paper's cross-layer overlap, Section 4.1, re-designed for CDNA4): each of
// wave owns a ring of kDepth register stages of 16-byte non-temporal weight loads.  When a phase
// ends, the first kDepth stages of the NEXT weight matrix are issued at once and the loads of the
// next input vector right behind them, speculatively: by the time they return (results come back
// in issue order) the other workgroups have usually published their part, so HBM keeps streaming
// while the dependency resolves.
//
// The projections of all phases run through ONE instance of the streaming loop; what differs per
// phase (input, epilogue) is selected at run time once per row pair.
// Optional profile (100 MHz wall clock), written only while a buffer is set through the debug entry
// point.  Layout in uint64 words, P = number of projection phases, W = workgroups:
//   [0, 12P)             workgroup 0, wave 0: kEvSlots stamps per phase (EV_* below)
//   [12P, 12P + 32W)     layer 1, every wave: 8 words per wave = run end of QKV/O/GU/DOWN (0..3),
//                        run start of the same (4..7)
//   [.. , .. + 40W)      layer 1, every workgroup: 8 words per projection kind about the staging of
//                        its input: 0 entered, 1 first load checked, 2 last light wait done,
//                        3 all tags fresh, 4 staged, 5 number of stale passes; then 8 words about
//                        its attention work: 0 start, 1 queries seen, 2 rows done, 3 partial stored,
//                        5 its share of the merged output stored, 6 end
__device__ __forceinline__ void dbg_event(const DevModel& M, int ph, int ev, int lane) {
    if (M.dbg && blockIdx.x == 0 && lane == 0) as_global(M.dbg)[ph * kEvSlots + ev] = wall_clock64();
}
__device__ __forceinline__ u64* dbg_wave_slots(const DevModel& M, int n_phases, int layer, int wave) {
    return M.dbg && layer == 1 ? M.dbg + (size_t)n_phases * kEvSlots + ((size_t)blockIdx.x * kFusedWaves + wave) * 8 : nullptr;
}
__device__ __forceinline__ u64* dbg_stage_slots(const DevModel& M, int n_phases, int ncta, int layer, int kind) {
    return M.dbg && layer == 1 && kind < 5 ? M.dbg + (size_t)n_phases * kEvSlots + (size_t)ncta * kFusedWaves * 8 + ((size_t)blockIdx.x * 5 + kind) * 8
                                           : nullptr;
}

struct EpiFused {
    int kind; u32 tag; u32 cnt;   // tag: 32-bit tag of q / k,v; cnt: write counter of the compact output vector
    const DevModel& M; const DevKV& KV; const int* pos; int layer; const float2* rope; float* logits; int hd;
    __device__ __forceinline__ void operator()(int pair, int b, float v0, float v1) const {
        switch (kind) {
            case PH_QKV: EpiQKVTagged{M, KV, pos, layer, rope, tag, hd}(pair, b, v0, v1); break;
            case PH_GU: EpiSwiGLUTagged{M.ch, M.F, cnt, M.gu}(pair, b, v0, v1); break;
            case PH_LM: if (pos[b] >= 0) EpiStore{logits, M.V}(pair, b, v0, v1); break;   // (no logits for a sequence that sits the step out)
            default: EpiDeltaTagged{M.cdelta, M.d, cnt}(pair, b, v0, v1); break;
        }
    }
};

// Everything that distinguishes one projection phase from another.
struct PhaseDesc {
    int kind, layer;
    TSrc src;
    PMat W;
    u32 out_tag;     // 32-bit tag of this phase's tagged outputs (q, k, v; attention partials)
    u32 out_cnt;     // write counter of this phase's compact output vector
};
struct PhaseState {   // the residual stream's ping-pong buffers
    cword_t* xcur; cword_t* xnext;
};
// The buffers swap roles after every QKV and every GU phase (each publishes the updated stream into
// xnext), so which is which follows from the phase number alone.
__device__ __forceinline__ PhaseState phase_state(const DevModel& M, int ph) {
    const int k = ph & 3;
    const bool odd = k == 1 || k == 2;
    return odd ? PhaseState{M.cx2, M.cx} : PhaseState{M.cx, M.cx2};
}

// `sl` = (steps executed so far) * L: the write counters of the compact vectors are sl + layer for the
// buffers written once per layer and 2 * (sl + layer) + {0, 1} for the sublayer output (O, then DOWN).
__device__ __forceinline__ PhaseDesc phase_desc(const DevModel& M, const int* tokens, u32 tb, u32 sl, int ph, int lm_in_kernel, const PhaseState& X) {
    PhaseDesc D;
    const int l = ph >> 2;
    const FF_CONST PLayer* Lp = as_const(M.layers) + min(l, M.L - 1);   // scalar loads (see as_const)
    D.layer = l;
    D.kind = ph == 4 * M.L ? PH_LM : (ph & 3);
    D.out_tag = 0;
    D.out_cnt = 0;
    TSrc& src = D.src;
    if (D.kind == PH_QKV) {
        if (l == 0) { src.embed = M.embed; src.tokens = tokens; src.tag = 0; }   // embedding rows are synthesised with tag 0
        else {
            src.base = X.xcur; src.stride = M.d; src.tag = sl + l - 1;
            src.add = M.cdelta; src.add_stride = M.d; src.add_tag = 2 * (sl + l - 1) + 1;
        }
        src.wb = X.xnext; src.wb_stride = M.d; src.wb_tag = sl + l;
        src.gain = Lp->g1; src.eps = M.eps;
        D.out_tag = tag_of(tb, l, TAG_QKV);
        D.W = FF_PMAT_FIELDS(Lp->qkv);
    } else if (D.kind == PH_O) {
        src.base = M.cattn_o; src.stride = (size_t)M.Hq * M.hd; src.tag = sl + l;
        D.out_cnt = 2 * (sl + l);
        D.W = FF_PMAT_FIELDS(Lp->o);
    } else if (D.kind == PH_GU) {
        src.base = X.xcur; src.stride = M.d; src.tag = sl + l;
        src.add = M.cdelta; src.add_stride = M.d; src.add_tag = 2 * (sl + l);
        src.wb = X.xnext; src.wb_stride = M.d; src.wb_tag = sl + l;
        src.gain = Lp->g2; src.eps = M.eps;
        D.out_cnt = sl + l;
        D.W = FF_PMAT_FIELDS(Lp->gu);
    } else if (D.kind == PH_DOWN) {
        src.base = M.ch; src.stride = M.F; src.tag = sl + l;
        D.out_cnt = 2 * (sl + l) + 1;
        D.W = FF_PMAT_FIELDS(Lp->down);
    } else {
        src.base = X.xcur; src.stride = M.d; src.tag = sl + M.L - 1;
        src.add = M.cdelta; src.add_stride = M.d; src.add_tag = 2 * (sl + M.L - 1) + 1;
        src.gain = M.gf; src.eps = M.eps;
        D.W = M.lm;
    }
    return D;
}

template <int WD, int HD, int G>
__global__ void __launch_bounds__(kFusedThreads) fused_decode_kernel(DevModel M, DevKV KV, const int* __restrict__ tokens,
                                                                     const int* __restrict__ pos, float* __restrict__ logits,
                                                                     int batch, int lm_in_kernel, int ncta, int mute_wg, int switches, int glu_off) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    if (!inputs_ok(M, KV, tokens, pos)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(M.status, kStatusRange);
        return;
    }
    // Test hook for the time-out path: the muted workgroup publishes nothing, so every workgroup
    // that needs its output runs into its own bounded wait, records the time-out and leaves.
    if ((int)blockIdx.x == mute_wg) return;
    constexpr int B = 1;   // (batch is 1)
    constexpr int EPU = WTraits<WD>::EPU;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float4* xs = (float4*)lds;
    float2* rope_lds = (float2*)(lds + kLdsActBytes + kLdsAuxBytes);   // [batch][hd/2]
    for (int i = threadIdx.x; i < batch * (M.hd / 2); i += kFusedThreads) {
        int b = i / (M.hd / 2), f = i % (M.hd / 2);
        rope_lds[i] = KV.rope[(size_t)max(step_pos(tokens, pos, b), 0) * (M.hd / 2) + f];
    }
    // Launch dimensions and positions are read again and again below; a vector load of them would
    // make the wave wait for everything it has in flight (its prefetched weight tiles included), so
    // the grid size is a kernel argument and the positions are staged in LDS once.
    static_assert(kLdsRopeBytes == kMaxBatchFused * 64 * sizeof(float2) && kLdsMiscBytes >= (16 + 2 * (1 + WgVote::kMaxSums) * kFusedWaves) * 4, "LDS layout");
    int* pos_lds = (int*)((float*)(lds + kLdsActBytes + kLdsAuxBytes) + 2 * kMaxBatchFused * 64 + 8);
    int* share_lds = pos_lds + kMaxBatch;   // workgroups per kv head of each sequence's attention (attn_share_of)
    static_assert(2 * kMaxBatch <= 8, "positions and attention shares in LDS");
    if ((int)threadIdx.x < batch) {
        pos_lds[threadIdx.x] = step_pos(tokens, pos, threadIdx.x);   // -1: the sequence sits this step out
        share_lds[threadIdx.x] = attn_share_of(tokens, pos, batch, threadIdx.x, ncta, M.Hkv, (switches & kSwUniformShares) != 0);
    }
    if (threadIdx.x < kGluMaxChunks) glu_counters_of(xs)[threadIdx.x] = 0u;
    __syncthreads();
    // projections only; attention runs right after each PH_QKV.  The LM head runs here unless its
    // weight type differs from the layers' (then the host launches it separately).
    const int n_phases = 4 * M.L + lm_in_kernel;
    // steps executed so far on the compact buffers (kept on the device: a skipped step does not count)
    const u32 steps_done = (u32)__builtin_amdgcn_readfirstlane(xld_u32(M.stepctr));
    const u32 sl = steps_done * (u32)M.L;
    // The 32-bit tags of this step's queries, keys, values and attention partials: a fresh range
    // per executed step, derived from the same device-side counter, so that a launch carries no
    // host-side step state (a launch recorded into a HIP graph replays correctly).  Tags wrap after
    // 2^32 / (5 L + 1) steps; a slot could only be mistaken for fresh if it had not been rewritten
    // for exactly that many steps, and every slot a step reads is rewritten by that step first.
    const u32 tag_base = steps_done * (u32)(kTagsPerLayer * M.L + 1);

    const int gwave = blockIdx.x * kFusedWaves + wave;
    const UDiv n_gwaves = UDiv::of((u32)ncta * kFusedWaves), n_ctas = UDiv::of((u32)ncta);
    float* myacc = (float*)(lds + kLdsActBytes) + (size_t)wave * kAccFloatsPerWave;
    float* red = (float*)(lds + kLdsActBytes + kLdsAuxBytes) + 2 * kMaxBatchFused * 64;   // behind the RoPE rows
    WgVote vote{(u32*)(red + 16), 0u};   // behind the reduction scratch and the positions
    // One iteration = one K segment of one projection; only (phase, segment) are carried from one
    // iteration to the next (pinning both to scalar registers measured slower for one sequence: 3.26 -> 3.30 ms).
    int ph = 0, seg = 0;
    for (;;) {
        const PhaseDesc D = phase_desc(M, tokens, tag_base, sl, ph, lm_in_kernel, phase_state(M, ph));
        EpiFused epi{D.kind, D.out_tag, D.out_cnt, M, KV, pos_lds, D.layer, rope_lds, logits, HD};
        const Stream<WD, B> S = Stream<WD, B>::make(D.W, seg, gwave, n_gwaves);
        // The wave's first tiles of this projection are requested before anything it has to wait
        // for (its input vector; for the output projection the whole attention), so the memory
        // pipe has work while the dependency resolves.  The ring lives from here to the end of
        // gemv_run only: keeping it out of the loop-carried state lets it stay in the registers
        // the loads were issued to (a copy would have to wait for the data).
        TSrc src = D.src;
        src.ncta = n_ctas;
        if (seg > 0) src.wb = nullptr;
        const bool att_first = D.kind == PH_O && seg == 0;
        Stage<WD> ring[kDepthOf<WD>];
        // (ablation switch, single-sequence bf16 instances only: with kSwNoOverlap the tiles are requested
        // after the input has arrived, as in a fused kernel without cross-layer memory overlap)
        constexpr bool kHasSwitch = WD == W_BF16;
        if (!kHasSwitch || !(switches & kSwNoOverlap)) prefetch_stream(S, ring, lane, 0, kPrefetchOf<WD>);
        if (wave == 0) dbg_event(M, min(ph, n_phases - 1), EV_PF_ISSUED, lane);
        if (att_first) {
            // split-KV attention + merge of this layer (the ring holds the output projection's tiles)
            __syncthreads();   // every wave has finished reading the staged input: LDS is free
            if (wave == 0) dbg_event(M, min(ph, n_phases - 1), EV_ATT_START, lane);
            u64* aev = dbg_stage_slots(M, n_phases, ncta, D.layer, 4);
            if (aev && threadIdx.x == 0) { as_global(aev)[0] = wall_clock64(); as_global(aev)[4] = 0; as_global(aev)[5] = 0; }
            bool mine = true;
            bool ok = attention_phase_tagged<kFusedWaves, HD, G, false>(M, KV, nullptr, pos_lds, share_lds, batch, D.layer, lds, tag_of(tag_base, D.layer, TAG_QKV),
                                                                tag_of(tag_base, D.layer, TAG_ATT), sl + D.layer, n_ctas, vote, mine, aev);
            ok = vote.all<kFusedThreads>(ok && mine);
            if (aev && threadIdx.x == 0) as_global(aev)[6] = wall_clock64();
            if (wave == 0) dbg_event(M, min(ph, n_phases - 1), EV_ATT_END, lane);
            if (!ok) return;
        }
        if (wave == 0) dbg_event(M, min(ph, n_phases - 1), EV_H_START, lane);
        bool ok;
        u64* ev = dbg_stage_slots(M, n_phases, ncta, D.layer, D.kind);
        if (src.add) ok = stage_tagged<EPU, true, kFusedThreads>(src, batch, S.K, S.j0 * EPU, S.nunits, S.nup, xs, red, threadIdx.x, vote, ev);
        else ok = stage_tagged<EPU, false, kFusedThreads>(src, batch, S.K, S.j0 * EPU, S.nunits, S.nup, xs, red, threadIdx.x, vote, ev);
        if (ev && threadIdx.x == 0) as_global(ev)[4] = wall_clock64();
        if (!ok) {
            if (threadIdx.x == 0) atomicCAS(M.status, 0, -55 - 10 * ph);
            return;
        }
        if (wave == 0) dbg_event(M, min(ph, n_phases - 1), EV_SYNCED, lane);
        if (kHasSwitch && (switches & kSwNoOverlap)) {
            prefetch_stream(S, ring, lane, 0, kPrefetchOf<WD>);
            // (a shorter ring has to have arrived: else the compiler has every pass of the loop below wait as on a ring that was never longer, half of it)
            if (S.n_it < kPrefetchOf<WD>) settled();
        }
        if constexpr (kPrefetchOf<WD> < kDepthOf<WD>) prefetch_stream(S, ring, lane, kPrefetchOf<WD>, kDepthOf<WD>);   // the rest of the ring, behind the input
        u64* wv = D.kind < 4 ? dbg_wave_slots(M, n_phases, D.layer, wave) : nullptr;
        if (wv && lane == 0) as_global(wv)[4 + D.kind] = wall_clock64();
        bool glu_done = false;
        if (glu_off >= 0 && D.kind == PH_GU) {
            // gate/up, SwiGLU and down projection as one stream, the down projection's input
            // staged chunk by chunk on the way (glu_run); the DOWN phase below is skipped
            const PhaseDesc Dd = phase_desc(M, tokens, tag_base, sl, ph + 1, lm_in_kernel, phase_state(M, ph + 1));
            const Stream<WD, B> Sd = Stream<WD, B>::make(Dd.W, 0, gwave, n_gwaves);
            const int pd = (int)n_gwaves.div((u32)(M.d / 2) + n_gwaves.n - 1u);   // most down-projection row pairs a wave owns
            float* lacc = (float*)(lds + kLdsActBytes + kLdsAuxBytes) - (size_t)(kFusedWaves - wave) * pd * 128;
            GluStager<WD> stg{M.ch, sl + (u32)D.layer, M.F, Sd.nup, Sd.cpr, (float4*)(lds + glu_off), glu_counters_of(xs)};
            EpiSwiGLUTagged epig{M.ch, M.F, D.out_cnt, M.gu};
            EpiDeltaTagged epid{M.cdelta, M.d, Dd.out_cnt};
            const bool okg = glu_run<WD>(S, Sd, ring, xs, stg, lacc, (u32)kFusedWaves * (u32)(D.layer + 1),
                                         kChunkUnitsOf<WD> * WTraits<WD>::EPU / M.gu.nw, lane, epig, epid);
            if (!okg) {
                if (lane == 0) atomicCAS(M.status, 0, -57 - 10 * ph);
                return;
            }
            if (wv && lane == 0) as_global(wv)[PH_DOWN] = wall_clock64();
            glu_done = true;
        }
        if (glu_done) { /* both projections are finished */ }
        else gemv_run<WD, B>(S, ring, xs, myacc, batch, lane, epi);
        if (wave == 0) dbg_event(M, min(ph, n_phases - 1), EV_RUN_DONE, lane);
        if (wv && lane == 0) as_global(wv)[D.kind] = wall_clock64();
        // next iteration: further K segment of the same projection, or the next projection
        if (glu_done) ++ph;   // the down projection ran inside glu_run
        if (seg + 1 < S.nseg) ++seg;
        else if (ph + 1 < n_phases) { ++ph; seg = 0; }
        else break;
    }
    // this step has been executed: the next one uses the next write counters (workgroup 0 can only
    // get here after every workgroup has taken part in every phase, i.e. has read the counter)
    // Word 1 of the counter block: rows of the compact exchange vectors that k_scrub_rows need not initialise.
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        xst_u32(M.stepctr + 1, (u32)batch);
        xst_u32(M.stepctr, steps_done + 1u);
    }
}

// Host-side launcher of one weight-type family; defined once per weight type in its own
// translation unit so that the instances compile in parallel.
struct FusedLaunch {
    DevModel M; DevKV KV; const int* tokens; const int* pos; float* logits;
    int batch; int lm_in_kernel; int n_cta; size_t lds_bytes; hipStream_t stream; int mute_wg; int switches;   // switches: kSw* bits
    int glu_off;   // >= 0: single-sequence passes run gate/up + down as one stream (glu_run), staged h at this LDS offset
    int wide;      // the pass runs on the wide kernel (ff_wide.h)
};
// One-time set-up of a kernel (thread-safe; a failure is remembered and reported by every call).
struct KernelSetup {
    std::once_flag once;
    hipError_t err = hipSuccess;
    const char* what = "";
    hipError_t run(const void* kern, int threads, size_t lds_bytes) {
        std::call_once(once, [&] {
            err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (err != hipSuccess) { what = "hipFuncSetAttribute"; return; }
            int occ = 0;
            err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, threads, lds_bytes);
            if (err != hipSuccess) { what = "hipOccupancyMaxActiveBlocksPerMultiprocessor"; return; }
            if (occ < 1) { what = "fused kernel does not fit on a compute unit"; err = hipErrorLaunchOutOfResources; }
        });
        return err;
    }
};
template <int WD, int HD, int G>
inline hipError_t launch_fused_instance(const FusedLaunch& a, const char** what) {
    auto kern = fused_decode_kernel<WD, HD, G>;
    static KernelSetup setup;
    if (hipError_t e = setup.run((const void*)kern, kFusedThreads, a.lds_bytes)) { *what = setup.what; return e; }
    kern<<<a.n_cta, kFusedThreads, a.lds_bytes, a.stream>>>(a.M, a.KV, a.tokens, a.pos, a.logits, a.batch, a.lm_in_kernel, a.n_cta, a.mute_wg, a.switches, a.glu_off);
    *what = "fused kernel launch";
    return hipGetLastError();
}
template <int WD, int NC, int HD, int G, bool LONG = kWideLong<WD, NC>>
inline hipError_t launch_wide_instance(const FusedLaunch& a, const char** what) {
    if constexpr (WD == W_INT4 && !LONG)
        if (wide_sz_far(std::max(a.M.Hq * a.M.hd, a.M.F), panel_tiles(a.M.d, a.n_cta))) return launch_wide_instance<WD, NC, HD, G, true>(a, what);
    auto kern = wide_decode_kernel<WD, NC, HD, G, LONG>;
    static KernelSetup setup;
    if (hipError_t e = setup.run((const void*)kern, kWideThreads, kWideLdsBytes)) { *what = setup.what; return e; }
    kern<<<a.n_cta, kWideThreads, kWideLdsBytes, a.stream>>>(a.M, a.KV, a.tokens, a.pos, a.logits, a.batch, a.lm_in_kernel, a.n_cta, a.mute_wg, a.switches);
    *what = "wide kernel launch";
    return hipGetLastError();
}
template <int WD, int HD, int G>
inline hipError_t launch_solo_instance(const FusedLaunch& a, const char** what) {
    auto kern = solo_decode_kernel<WD, HD, G>;
    static KernelSetup setup;
    if (hipError_t e = setup.run((const void*)kern, kSoloThreads, SoloLds<WD>::kBytes)) { *what = setup.what; return e; }
    kern<<<a.n_cta, kSoloThreads, SoloLds<WD>::kBytes, a.stream>>>(a.M, a.KV, a.tokens, a.pos, a.logits, a.lm_in_kernel, a.n_cta, a.mute_wg, a.switches);
    *what = "one-sequence kernel launch";
    return hipGetLastError();
}
template <int WD, int HD, int G>
inline hipError_t launch_fused_family(const FusedLaunch& a, const char** what) {
    // (the host decides whether a pass is wide, and sizes the buffers for it; up to eight sequences share an operand tile with their remainders)
    if (a.wide) return a.batch == 1 ? launch_wide_instance<WD, 1, HD, G>(a, what) : a.batch <= 8 ? launch_wide_instance<WD, 8, HD, G>(a, what) : launch_wide_instance<WD, 16, HD, G>(a, what);
    if (a.batch != 1) {
        *what = "several sequences on the row-partitioned kernel";
        return hipErrorInvalidValue;
    }
    return launch_fused_instance<WD, HD, G>(a, what);
}
// One definition per (weight type, head geometry), each in its own translation unit.
#define FF_FUSED_FAMILIES(X) \
    X(bf16, W_BF16, 64, 4) X(bf16, W_BF16, 128, 4) X(bf16, W_BF16, 128, 8) \
    X(int8, W_INT8, 64, 4) X(int8, W_INT8, 128, 4) X(int8, W_INT8, 128, 8) \
    X(int4, W_INT4, 64, 4) X(int4, W_INT4, 128, 4) X(int4, W_INT4, 128, 8)
#define FF_DECLARE_FAMILY(name, wd, hd, g) \
    hipError_t launch_fused_##name##_hd##hd##_g##g(const FusedLaunch& a, const char** what); \
    hipError_t launch_solo_##name##_hd##hd##_g##g(const FusedLaunch& a, const char** what);
FF_FUSED_FAMILIES(FF_DECLARE_FAMILY)
#undef FF_DECLARE_FAMILY

}  // namespace ff
