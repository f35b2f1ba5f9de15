// Kernels: the fused whole-model decode step, the per-operation baseline, and the loaders.
#pragma once
#include "ff_phases.h"
#include "ff_glu.h"

namespace ff {

constexpr int kTagsPerLayer = 5;   // phase instances (= exchange tags) per layer of the fused kernel
enum { PH_QKV = 0, PH_O = 1, PH_GU = 2, PH_DOWN = 3, PH_LM = 4 };
// Measurement switches of a launch (debug entry points): tiles requested only after the input has
// arrived; attention shares equal for every sequence instead of by length (attn_share_of).
enum { kSwNoOverlap = 1, kSwUniformShares = 2 };
enum { TAG_QKV = 0, TAG_ATT = 1, TAG_O = 2, TAG_GU = 3, TAG_DOWN = 4 };
__device__ __forceinline__ u32 tag_of(u32 tag_base, int l, int k) { return tag_base + 1u + (u32)(l * kTagsPerLayer + k); }
// Stamps of workgroup 0 per projection phase in the optional timeline buffer (layout: ff_fused.h).
enum { EV_SYNCED = 0, EV_RUN_DONE = 1, EV_PF_ISSUED = 2, EV_H_START = 3, EV_ATT_START = 6, EV_ATT_END = 7, kEvSlots = 12 };

// status codes written by kernels (mirror the C ABI's FF_ERR_*)
constexpr int kStatusRange = -3;
constexpr int kStatusTimeout = -5;

// tokens / pos point to the first sequence of the current pass; the check covers every sequence of
// the whole decode step (all passes), so that a bad token or position anywhere skips every pass.
__device__ __forceinline__ bool inputs_ok(const DevModel& M, const DevKV& KV, const int* tokens, const int* pos) {
    bool ok = true;
    for (int b = -KV.seq0; b < KV.step_batch - KV.seq0; b++) {
        int p = pos[b], t = tokens[b];
        ok = ok && (t == kTokenSkip || (p >= 0 && p < KV.max_ctx && t >= 0 && t < M.V));
    }
    return ok;
}

// Attention work distribution: the items (sequence b, kv head j, split s) of all sequences form
// one list that is dealt round-robin to the workgroups (a per-layer work queue with a static
// owner per entry; the split count follows each sequence's current length).
template <int NW>
__device__ void attention_phase_plain(const DevModel& M, const DevKV& KV, const int* tokens, const int* pos, int batch, int layer, uint8_t* lds) {
    const int G = M.Hq / M.Hkv;
    const int share = max(1, (int)gridDim.x / (batch * M.Hkv));
    int base = 0;
    PlainAttnIO xio;
    for (int b = 0; b < batch; b++) {
        const int T = max(step_pos(tokens, pos, b), 0);
        const int ns = attn_nsplit(T, share, M.hd);
        const int nitems = M.Hkv * ns;
        int first = ((int)blockIdx.x - base) % (int)gridDim.x;
        if (first < 0) first += gridDim.x;
        for (int it = first; it < nitems; it += gridDim.x) {
            int j = it / ns, s = it % ns;
            int t0 = (int)((long)T * s / ns), t1 = (int)((long)T * (s + 1) / ns);
            bool cur = s == ns - 1;
            if (M.hd == 64 && G == 4) attn_item<64, 4, NW>(M, KV, xio, layer, b, j, t0, t1, cur, s, ns, lds);
            else if (M.hd == 128 && G == 4) attn_item<128, 4, NW>(M, KV, xio, layer, b, j, t0, t1, cur, s, ns, lds);
            else if (M.hd == 128 && G == 8) attn_item<128, 8, NW>(M, KV, xio, layer, b, j, t0, t1, cur, s, ns, lds);
        }
        base = (base + nitems) % (int)gridDim.x;
    }
}

// Fused kernel: queries / current k,v are awaited through their tags; the workgroups of a
// head group's splits share out the merge of its outputs (paper Section 4.2: the reduction
// is fused into the attention pass instead of a separate kernel).  The head geometry is a template
// parameter here (one kernel instance per geometry) to keep the register footprint of the fused
// kernel down to what the model at hand needs.  `pos` points to the positions staged in LDS and
// ncta is the grid size: both are read often, and fetching them from global memory here would make
// the wave wait for every load it has in flight, weight tiles included.
// Workgroups per (sequence, kv head) for a step's attention, by the sequences' lengths: every
// sequence gets one per kv head, and what is left of the grid is dealt out in proportion to the
// rows each has to read (cached rows + its own).  A sequence much longer than its neighbours is cut
// into correspondingly more slices, so the slices of a ragged batch come out about equally long
// instead of the long sequence's being as many times longer as it is (the paper names load balance
// at variable context as the reason for scheduling at run time, Section 6); with equal lengths this
// is the equal division n_workgroups / (batch * Hkv).  The shares sum to at most n_workgroups / Hkv.
// Every workgroup computes the same list from the step's positions: the work list is rebuilt each
// step, its entries have fixed owners, nothing is claimed with atomics.
__device__ __forceinline__ int attn_share_of(const int* tokens, const int* pos, int batch, int b, int ncta, int Hkv, bool uniform) {
    const u32 floor_items = (u32)(batch * Hkv);
    const u32 budget = (u32)ncta > floor_items ? (u32)ncta - floor_items : 0u;
    if (uniform) return 1 + (int)(budget / floor_items);
    u32 tot = 0;
    for (int i = 0; i < batch; i++) tot += (u32)max(step_pos(tokens, pos, i), 0) + 1u;
    const u32 mine = (u32)max(step_pos(tokens, pos, b), 0) + 1u;
    return 1 + (int)((u32)((u64)budget * mine / tot) / (u32)Hkv);
}

// An item of a step's attention: slice `split` of ns of sequence b's KV head j, cached rows [t0, t1), and with the last slice the step's own.
struct AttnItem {
    u32 bj, sn;   // b | j << 8 (ns == 0: none), split | ns << 16
    int t0, t1;
};
typedef __attribute__((address_space(3))) AttnItem lds_item;
constexpr int kAttnListed = 8;   // items of a workgroup that are listed once per step; a layer works out again what is behind them
// Item number k of this workgroup.  (32-bit unsigned arithmetic throughout: 64-bit or signed divisions are long instruction sequences.)
template <int HD, int NW>
__device__ __forceinline__ AttnItem attn_item_at(const int* pos, const int* share, int batch, int Hkv, const UDiv& nc, int k) {
    const int ncta = (int)nc.n;
    int base = 0;
    for (int b = 0; b < batch; b++) {
        const int T = max(pos[b], 0);   // (-1: the sequence sits this step out and is carried as a placeholder with an empty cache)
        const int ns = HD == 64 && NW == 4 ? attn_nsplit_few(T, share[b]) : attn_nsplit(T, share[b], HD), nitems = Hkv * ns;
        const int first = (int)nc.mod((u32)blockIdx.x + (u32)ncta - (u32)base);   // base < ncta
        const int here = first < nitems ? (int)nc.div((u32)(nitems - first + ncta - 1)) : 0;
        if (k < here) {
            const int it = first + k * ncta, j = (int)((u32)it / (u32)ns), s = it - j * ns;
            return AttnItem{(u32)b | (u32)j << 8, (u32)s | (u32)ns << 16, (int)((u32)T * (u32)s / (u32)ns), (int)((u32)T * (u32)(s + 1) / (u32)ns)};   // T * 64 < 2^32
        }
        k -= here;
        base = (int)nc.mod((u32)base + (u32)nitems);
    }
    return AttnItem{0u, 0u, 0, 0};
}
// The workgroup's list, the same for every layer, by its first kAttnListed threads.  (Worked out layer by layer, sequence by sequence, it stood with
// its divisions between the QKV projection and the first request for a cached row.)
template <int HD, int NW>
__device__ __forceinline__ void attn_list(lds_item* list, const int* pos, const int* share, int batch, int Hkv, const UDiv& nc) {
    if (threadIdx.x < kAttnListed) {
        const AttnItem e = attn_item_at<HD, NW>(pos, share, batch, Hkv, nc, threadIdx.x);
        *(__attribute__((address_space(3))) u32x4*)(list + threadIdx.x) = __builtin_bit_cast(u32x4, e);
    }
}

// list: attn_list's (null: every item is worked out here); share: workgroups per kv head of each sequence (attn_share_of), staged in LDS like the positions.
// Returns false (uniformly) if the queries did not come; mine: whether this wave's part of the merge did.
// REUSE: the caller's waves write to lds as soon as they return.
template <int NW, int HD, int G, bool REUSE>
__device__ __forceinline__ bool attention_phase_tagged(const DevModel& M, const DevKV& KV, const lds_item* list, const int* pos, const int* share, int batch, int layer,
                                                       uint8_t* lds, u32 in_tag, u32 out_tag, u32 out_cnt, const UDiv& nc, WgVote& vote, bool& mine, u64* ev = nullptr,
                                                       const WideImg* merged_img = nullptr) {
    constexpr int NT = NW * 64;
    bool ok = true;
    TaggedAttnIO xio{in_tag, out_tag, out_cnt, merged_img, &vote};
    for (int k = 0;; k++) {
        u32x4 e;
        if (list && k < kAttnListed) e = *(const __attribute__((address_space(3))) u32x4*)(list + k);
        else e = __builtin_bit_cast(u32x4, attn_item_at<HD, NW>(pos, share, batch, M.Hkv, nc, k));
        const int bj = __builtin_amdgcn_readfirstlane((int)e.x), sn = __builtin_amdgcn_readfirstlane((int)e.y);
        const int t0 = __builtin_amdgcn_readfirstlane((int)e.z), t1 = __builtin_amdgcn_readfirstlane((int)e.w);
        const int ns = sn >> 16, s = sn & 0xFFFF, b = bj & 0xFF, j = bj >> 8;
        if (ns == 0) break;
        ok = attn_item<HD, G, NW, TaggedAttnIO, true>(M, KV, xio, layer, b, j, t0, t1, s == ns - 1, s, ns, lds, ev) && ok;
        if constexpr (REUSE) __syncthreads();   // the waves' states have been read
        if (ns > 1 && ok) {
            mine = attn_merge_tagged<HD, G, NT>(M, xio, b, j, s, ns) && mine;
            if (ev && threadIdx.x == 0) as_global(ev)[5] = wall_clock64();
        }
        if constexpr (REUSE) settled();
    }
    return ok;
}

}  // namespace ff
