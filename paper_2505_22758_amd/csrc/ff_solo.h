// The step of a model for one sequence: weights stream through a ring in LDS that never drains, the
// exchanged vectors are waited for word by word.
//
// With one sequence a layer is a chain of five small hand-overs (QKV -> attention -> output -> gate/up -> down
// projection -> next layer) between weight streams of 2 to 50 us.  What bounds a step is the stream at the memory's rate
// (bf16) and the chain of hand-overs (quantised weights, small models).  So
//   * projections are partitioned as in the wide pass (ff_dense.h): a workgroup owns rows, its eight
//     waves split K, weights lie in operand tiles (PMat), products come from v_mfma_f32_16x16x32_bf16
//     with the input's three bf16 parts (24 bits) as rows 0..2 of the A operand;
//   * tiles go from memory straight into LDS (buffer loads with the lds bit), kTiles units of them per wave in flight.  The
//     request for a tile is made when an earlier one has been used up, whatever projection that one belongs to:
//     a wave's requests are ONE sequence over panels, projections and layers (SoloFeed), running a ring's length ahead
//     of the products, so the next projection's first tiles (96 KB per compute unit, 3.4 us of the
//     memory's rate) travel while this one's sums are finished, published and waited for, and during the attention.  A register ring cannot be kept over
//     the branches between projections; LDS can, and costs nothing: a plain stream through it reads 6.85 TB/s (8 KB per wave
//     in flight) against 6.9 TB/s into registers;
//   * vectors travel in the compact format (22 bits and a write counter, ff_phases.h).  A wave reads the
//     words of ITS columns until they are there, and splits them into operand parts in an LDS area of its own: no flag, no store
//     acknowledgement, no barrier between a projection's inputs and its products.  The normalisation's sum of squares
//     comes out of the same words;
//   * the residual rows stay with the workgroup that owns them, which publishes residual + sublayer output;
//   * everything per tile is one code path for all panel widths (uniform branches pick the accumulator), so the kernel
//     stays inside the instruction cache (the wide pass has a copy per width).
// Exchange buffers: cx (input of QKV and LM head), cx2 (of gate/up), cattn_o, ch, each written once per layer.  A buffer's next write
// depends on outputs of every workgroup that reads its present contents, which it publishes behind its reads: the chain
// QKV -> attention -> output -> gate/up -> down consumes every word of each of the vectors.
//
// Us per step, row-partitioned kernel (ff_fused.h) / this one: 8B, eight layers, bf16 context 1024 719 / 711, int8 context 4096 576 / 494, int4
// context 2048 577 / 364; 70B, six layers, context 2048, bf16 1745 / 1688, int4 1105 / 634; tiny, four layers 101 / 93.
//
// No register may be spilled to memory in this kernel: a reload is a vector load, and the wait for it drains the ring (8 spilled
// registers outside of the loops cost 8 % of the 8B bf16 step).
//
// The waits for tiles are written out (s_waitcnt with the ring's length); loads with the lds bit are made in inline
// assembly, unknown to the compiler, whose own waits then only ever wait for more than they have to.  They have no register
// outputs, and a slot is read, in one block with the wait for it, before it is requested again.
#pragma once
#include "ff_wide.h"

namespace ff {

constexpr int kSoloWaves = 8;
constexpr int kSoloThreads = kSoloWaves * 64;
constexpr int kSoloPassCols = 512;                 // columns of a wave that one pass of its lanes covers (eight each)
constexpr int kSoloPasses = 2;                     // passes whose operands a wave's LDS area holds (8192 columns for the workgroup); inputs with
                                                   // more are taken pass by pass, the next one's words arriving in the second half meanwhile
constexpr int kSoloPassBytes = kSoloPassCols * 6;
constexpr int kSoloImgBytes = kSoloPasses * kSoloPassBytes;   // per wave
constexpr int kSoloPanelRows = 16 * kPanelTiles;
constexpr int kSoloScaleRows = 1024;               // int8: row scales of a projection's rows held in LDS
// The ring's unit is two kilobytes of a tile: the columns of one iteration (bf16) or two (quantised weights), neighbours in memory.  A wave needs some
// hundred instructions per unit besides the products, however large it is: 8B, eight layers, us per step, units of one / two kilobytes: int4 403 / 365, int8 538 / 492.
template <int WD> constexpr int kUIters = WD == W_BF16 ? 1 : 2;
template <int WD> constexpr int kUCols = kUIters<WD> * kWCols<WD>;
template <int WD> constexpr int kUSteps = kUIters<WD> * kWSteps<WD>;
template <int WD> struct SoloRing {
    static constexpr int kTileBytes = WD == W_INT4 ? 2048 + 128 : 2048;   // int4: codes, then (scale | zero << 16) of the 16 rows for both groups
    static constexpr int kTiles = 6;
    static constexpr int kLoads = WD == W_INT4 ? 3 : 2;   // per unit
    static constexpr int kBytes = kTiles * kTileBytes;    // per wave
};
// LDS: rings | operand areas (attention: its state) | partial sums | int8 row scales | RoPE row | residual rows | small words
template <int WD> struct SoloLds {
    static constexpr int kImg = kSoloWaves * SoloRing<WD>::kBytes;
    static constexpr int kRed = kImg + kSoloWaves * kSoloImgBytes;
    static constexpr int kScale = kRed + 2 * kSoloWaves * kSoloPanelRows * 4;
    static constexpr int kRope = kScale + (WD == W_INT8 ? 2 * kSoloScaleRows * 2 : 0);
    static constexpr int kRes = kRope + 64 * 8;
    static constexpr int kRms = kRes + kWideResRows * 4;                  // sums of squares [2][wave]
    static constexpr int kTab = kRms + 2 * kSoloWaves * 4;                // SoloMat of the five projections
    static constexpr int kInt = kTab + 5 * 64;                            // position, attention share, failure flag, vote slots
    static constexpr int kBytes = kInt + 16 + 2 * (1 + WgVote::kMaxSums) * kSoloWaves * 4;
    static_assert(kBytes <= 160 * 1024, "LDS of the one-sequence step");
    static_assert((kAttnStateFloats<128, 8, kSoloWaves> + (8 + 2) * 128 + kSoloWaves * 128) * 4 <= kSoloWaves * kSoloImgBytes, "attention state");
};

// The loads of a unit into LDS: 16 bytes per lane, lane i at lds + 16 i, from offsets voff + soff and voff2 + soff2 a kilobyte behind it; int4: then 4 bytes
// per lane of lanes 0..31 behind that.  All lanes are active.  (s_nop: M0 and scalar operands may have been written just before.)
template <int WD>
__device__ __forceinline__ void lds_load_unit(u32 lds, const __amdgpu_buffer_rsrc_t& r, u32 voff, u32 soff, u32 voff2, u32 soff2, const __amdgpu_buffer_rsrc_t& rz, u32 voffz,
                                              u32 soffz) {
    if constexpr (WD != W_INT4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %4, %2, %5 offen nt lds"
                     ::"s"(lds), "v"(voff), "s"(r), "s"(soff), "v"(voff2), "s"(soff2) : "memory", "scc");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %4, %2, %5 offen nt lds\n\t"
                     "s_add_u32 m0, m0, 0x400\n\ts_mov_b64 exec, 0xffffffff\n\tbuffer_load_dword %6, %7, %8 offen nt lds\n\ts_mov_b64 exec, -1"
                     ::"s"(lds), "v"(voff), "s"(r), "s"(soff), "v"(voff2), "s"(soff2), "v"(voffz), "s"(rz), "s"(soffz) : "memory", "scc");
}
__device__ __forceinline__ void wg_barrier_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }   // (leaves the ring's loads in flight)
__device__ __forceinline__ bool wave_all(bool p) { return __builtin_amdgcn_ballot_w64(!p) == 0; }   // (of the active lanes; known to be uniform)
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) uint8_t lds_u8;

// What the workgroup needs to know of a projection, in LDS (kinds PH_QKV .. PH_LM): pointers of layer 0, advanced by the layers'
// stride.  (Read out of the layer table in memory where they are needed, the descriptors of a layer nobody has touched yet are
// two dependent misses on the way from one projection to the next, and in the middle of the tile requests.  8B, eight layers, us per step, together
// with sums that are added up in LDS in place of registers picked by branches: int4 457 -> 413, int8 558 -> 537, bf16 728 -> 714.)
struct SoloMat {
    u64 w, sz, s, gain;        // w, sz: of the workgroup's first row
    int r0, rows, k, nu;       // its rows; columns; units of a row
    int tiles; u32 rowb; int pad[2];   // tiles of a panel; bytes of a row
};
static_assert(sizeof(SoloMat) == 64, "size in LDS");
typedef __attribute__((address_space(3))) SoloMat lds_mat;
template <int WD>
__device__ __forceinline__ void solo_table(lds_mat* tab, const DevModel& M, const UDiv& n_ctas, int kind, bool lm) {   // entry `kind`, by one thread
    const PLayer* L = M.layers + (kind == PH_LM ? M.L : 0);
    const PMat* W = &L->qkv + (kind & 3);
    SoloMat e{};
    if (kind != PH_LM || lm) {
        const RowRange rr = wide_rows(W->n, n_ctas);
        const int ni = (W->k + kWCols<WD> - 1) / kWCols<WD>;
        e.k = W->k; e.nu = (ni + kUIters<WD> - 1) / kUIters<WD>; e.rowb = (u32)ni * (WD == W_BF16 ? 128u : 64u);
        e.r0 = rr.r0; e.rows = max(rr.r1 - rr.r0, 0); e.tiles = W->panels;
        e.w = (u64)(W->w + (size_t)rr.r0 * e.rowb);
        e.sz = (u64)(W->sz + (size_t)rr.r0 * (e.rowb >> 6));
        e.s = (u64)W->s;
        e.gain = (u64)(kind == PH_GU ? L->g2 : L->g1);
    }
    u64* src = (u64*)&e;
    for (int i = 0; i < 8; i++) ((__attribute__((address_space(3))) u64*)(tab + kind))[i] = src[i];
}

// A wave's sequence of tile requests: for every phase, panel of the workgroup's rows, iteration of the wave and tile.
template <int WD>
struct SoloFeed {
    typedef SoloRing<WD> R;
    static constexpr u32 kNowhere = 0x7FFFFC00u;   // an offset behind every matrix: answered without an access
    __amdgpu_buffer_rsrc_t rw, rz;
    u32 ring;              // LDS address of the ring
    int ph, it, nu, t, T;  // position: phase, unit of the rows, tile of the panel
    int left, full;        // rows of the workgroup from the panel's first one on; whole tiles among them
    u32 panel, soff;       // the panel's first byte; offset of the next tile, if it is whole
    u32 rowb;              // bytes per row
    int last_half;         // the unit that has one iteration only (-1: none)
    int wave, lane, n_phases;
    bool bounded;          // (measurement switch) stop at the end of every phase
    static constexpr u32 kStep = 2048u;   // bytes of a unit of a whole tile

    __device__ __forceinline__ void nothing() { T = 0x7FFFFFFF; t = 0; left = 0; full = 0; }
    __device__ __forceinline__ void begin(const DevModel& M, const lds_mat* tab, int phase) {
        for (ph = phase; ph < n_phases; ph++) {
            const bool lm = ph == 4 * M.L;
            const lds_mat* e = tab + (lm ? (int)PH_LM : ph & 3);
            left = uni(e->rows); nu = uni(e->nu);
            if (left <= 0 || wave >= nu) continue;
            const size_t off = lm ? 0 : (size_t)(ph >> 2) * M.layer_stride;
            rowb = (u32)uni((int)e->rowb); T = uni(e->tiles); t = 0; it = wave; panel = 0;
            full = left >> 4; soff = (u32)it * kStep;
            last_half = kUIters<WD> == 2 && (rowb & 64u) ? nu - 1 : -1;   // (64 bytes per iteration of quantised rows)
            rw = __builtin_amdgcn_make_buffer_rsrc((void*)(uni(e->w) + off), 0, (int)((u32)left * rowb), 0x00020000);
            if constexpr (WD == W_INT4) rz = __builtin_amdgcn_make_buffer_rsrc((void*)(uni(e->sz) + off), 0, (int)((u32)left * (rowb >> 4)), 0x00020000);
            return;
        }
        nothing();
    }
    // Requests the next tile into the slot at `dst` (LDS address).
    __device__ __forceinline__ void request(const DevModel& M, const lds_mat* tab, u32 dst) {
        u32 so = soff, voff = (u32)lane * 16u, second = so + 1024u, voffz = (u32)(lane & 31) * 4u;
        if (__builtin_expect(t >= full, 0)) {   // the workgroup's last rows, or none: then nothing is read
            const int nt = left - 16 * t, n1 = max(nt, 1);
            so = nt > 0 ? panel + (u32)t * 16u * rowb + (u32)it * (kStep / 16u) * (u32)n1 : 0u;
            voff = nt > 0 ? (u32)((lane >> 4) * n1 + min(lane & 15, n1 - 1)) * 16u : kNowhere;
            voffz = nt > 0 ? (u32)(((lane >> 4) & 1) * n1 + min(lane & 15, n1 - 1)) * 4u : kNowhere;
            second = so + 64u * (u32)n1;
        }
        u32 voff2 = voff;
        const u32 soz = so >> 4;
        if constexpr (kUIters<WD> == 2)
            if (__builtin_expect(it == last_half, 0)) {   // rows of an odd number of iterations: the last unit has only the first
                voff2 = kNowhere;
                if (lane & 16) voffz = kNowhere;
            }
        lds_load_unit<WD>(dst, rw, voff, so, voff2, second, rz, voffz, soz);
        soff += 16u * rowb;
        if (++t < T) return;
        t = 0;
        if ((it += kSoloWaves) < nu) { soff = panel + (u32)it * kStep; return; }
        it = wave;
        panel += 16u * (u32)T * rowb;
        soff = panel + (u32)it * kStep;
        left -= 16 * T;
        full = left >> 4;
        if (left > 0) return;
        if (bounded) nothing();
        else begin(M, tab, ph + 1);
    }
    __device__ __forceinline__ void fill(const DevModel& M, const lds_mat* tab) {
#pragma unroll 1
        for (int i = 0; i < R::kTiles; i++) request(M, tab, ring + (u32)i * R::kTileBytes);
    }
};

// The words of a wave's columns (pass s: units of the wave from s * kSoloPassCols / kUCols on, eight columns per lane).
struct SoloWords {
    u32x2 w[kSoloPasses][4];
    // (scalar base and a 32-bit offset: one address register per load)
    __device__ __forceinline__ static u32x2 load(const cword_t* src, u32 el) {
        const u64 a = __hip_atomic_load((const FF_GLOBAL u64*)((const FF_GLOBAL uint8_t*)as_global(src) + (size_t)(el * 4u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return u32x2{(u32)a, (u32)(a >> 32)};
    }
    __device__ __forceinline__ void undefined() {   // (no instruction, see gw below)
#pragma unroll
        for (int s = 0; s < kSoloPasses; s++)
#pragma unroll
            for (int i = 0; i < 4; i++) asm volatile("" : "=v"(w[s][i]));
    }
    template <int WD>
    __device__ __forceinline__ static int col_of(int pass, int wave, int lane) {
        constexpr int LPU = kUCols<WD> / 8;   // lanes per unit
        return (wave + kSoloWaves * (pass * (64 / LPU) + lane / LPU)) * kUCols<WD> + (lane % LPU) * 8;
    }
    // Reads the words of passes p0 .. p0 + np - 1 until every one carries cnt.  False on a time-out.
    template <int WD>
    __device__ __forceinline__ bool wait(const cword_t* src, u32 cnt, int K, int p0, int np, int wave, int lane) {
        u32 stale = (1u << np) - 1u;
        for (int spins = 0; spins < kSpinLimit; spins++) {
#pragma unroll
            for (int s = 0; s < kSoloPasses; s++)
                if ((stale >> s) & 1u) {
                    const u32 c = (u32)min(col_of<WD>(p0 + s, wave, lane), K - 8);   // (lanes past the end read the last columns)
#pragma unroll
                    for (int i = 0; i < 4; i++) w[s][i] = load(src, c + 2 * i);
                }
#pragma unroll
            for (int s = 0; s < kSoloPasses; s++)
                if ((stale >> s) & 1u) {
                    u32 dirty = 0;
#pragma unroll
                    for (int i = 0; i < 4; i++) dirty |= (w[s][i].x ^ cnt) | (w[s][i].y ^ cnt);
                    if (wave_all((dirty & kCntMask) == 0)) stale &= ~(1u << s);
                }
            if (!stale) return true;
            // Samples until they are fresh (one pair of words for every 64 columns, another one each time): the full set read over and over by
            // every wave of the grid stands in the way of the stores that are waited for.
            for (;; spins++) {
                bool fresh = true;
                if ((lane & 7) < np) {
                    const u32x2 v = load(src, (u32)min(col_of<WD>(p0 + (lane & 7), wave, (lane & 56) + (spins & 7)), K - 8));
                    fresh = (((v.x ^ cnt) | (v.y ^ cnt)) & kCntMask) == 0;
                }
                if (wave_all(fresh)) break;
                if (spins >= kSpinLimit) return false;
                __builtin_amdgcn_s_sleep(2);
            }
        }
        return false;
    }
    // The same passes out of an embedding row.
    template <int WD>
    __device__ __forceinline__ void embed(const bf16_t* row, int K, int np, int wave, int lane) {
#pragma unroll
        for (int s = 0; s < kSoloPasses; s++)
            if (s < np) {
                const u32x4 e = *as_global((const u32x4*)(row + min(col_of<WD>(s, wave, lane), K - 8)));
                const u32 v[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
                for (int i = 0; i < 4; i++) w[s][i] = u32x2{v[i] << 16, v[i] & 0xFFFF0000u};
            }
    }
    // The words of pass `pass` on their way into LDS (two loads of 16 bytes per lane: 2 KB at `dst`); taken from there with `land`.
    template <int WD>
    __device__ __forceinline__ static void send(const __amdgpu_buffer_rsrc_t& src, u32 dst, int pass, int wave, int lane) {
        const u32 o = (u32)col_of<WD>(pass, wave, lane) * 4u;   // (behind the vector's end: nothing is read)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %3, 0 offen sc1 lds\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen sc1 lds"
                     ::"s"(dst), "v"(o), "v"(o + 16u), "s"(src) : "memory", "scc");
    }
    // The pass sent before the last V loads: are all its words fresh?
    template <int WD, int V>
    __device__ __forceinline__ bool land(u32 from, u32 cnt, int K, int pass, int wave, int lane) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(V) : "memory");
        const u32x4 a = *(const lds_u32x4*)(from + lane * 16), b = *(const lds_u32x4*)(from + 1024 + lane * 16);
        w[0][0] = u32x2{a.x, a.y}; w[0][1] = u32x2{a.z, a.w}; w[0][2] = u32x2{b.x, b.y}; w[0][3] = u32x2{b.z, b.w};
        const u32 dirty = (a.x ^ cnt) | (a.y ^ cnt) | (a.z ^ cnt) | (a.w ^ cnt) | (b.x ^ cnt) | (b.y ^ cnt) | (b.z ^ cnt) | (b.w ^ cnt);
        return wave_all((dirty & kCntMask) == 0 || col_of<WD>(pass, wave, lane) >= K);
    }
};

// Eight columns of a lane as operand parts into the wave's area: [iteration][k-step][part][lane group][16 bytes]; slot: pass of the area.
template <int WD>
__device__ __forceinline__ void solo_operands(lds_u8* area, int slot, int lane, const float (&t)[8]) {
    constexpr int LPI = kWCols<WD> / 8;
    const int sub = lane % LPI;   // (a pass is a whole number of iterations, in the order of the units)
    const int step = WD == W_BF16 ? sub >> 2 : WD == W_INT8 ? sub & 1 : sub & 3, g = WD == W_BF16 ? sub & 3 : WD == W_INT8 ? sub >> 1 : sub >> 2;
    lds_u8* p = area + (((slot * (64 / LPI) + lane / LPI) * kWSteps<WD> + step) * 12 + g) * 16;
    u32 v[3][4];
#pragma unroll
    for (int i = 0; i < 4; i++) split3_bf16x2(t[2 * i], t[2 * i + 1], v[0][i], v[1][i], v[2][i]);
#pragma unroll
    for (int k = 0; k < 3; k++) *(lds_u32x4*)(p + k * 64) = u32x4{v[k][0], v[k][1], v[k][2], v[k][3]};
}

// The products of n_it units (operands in the wave's area) with the T tiles of each: tiles in the order they were
// requested.  A tile is read out of the ring while the one before it is multiplied, and its slot requested again once it is in registers.
template <int WD>
struct SoloTile {
    u32x4 w[2];
    u32 sz[2];
    __device__ __forceinline__ void read(u32 a, int lane) {
        typedef SoloRing<WD> R;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R::kTiles - 1) * R::kLoads) : "memory");   // the oldest unit of a full ring is there
        w[0] = *(const lds_u32x4*)(a + lane * 16);
        w[1] = *(const lds_u32x4*)(a + 1024 + lane * 16);
        if constexpr (WD == W_INT4) {
            sz[0] = *(const lds_u32*)(a + 2048 + (lane & 15) * 4);
            sz[1] = *(const lds_u32*)(a + 2048 + 64 + (lane & 15) * 4);
        }
    }
    __device__ __forceinline__ void arrived() const {   // the registers are written: the slot may be overwritten
        if constexpr (WD == W_INT4) asm volatile("" ::"v"(w[0]), "v"(w[1]), "v"(sz[0]), "v"(sz[1]) : "memory");
        else asm volatile("" ::"v"(w[0]), "v"(w[1]) : "memory");
    }
};
template <int WD>
__device__ __forceinline__ void solo_run(SoloFeed<WD>& feed, const DevModel& M, const lds_mat* tab, u32& slot, const lds_u8* area, int lane, int n_it, int T,
                                         lds_float* sums) {
    typedef SoloRing<WD> R;
    constexpr int NX = kUSteps<WD>;
    if (n_it <= 0) return;
    const lds_u8* xa = area + (min(lane & 15, 2) * 4 + (lane >> 4)) * 16;
    const u32 end = feed.ring + R::kBytes;
    // (the constants of the int4 conversion in registers, unknown to the compiler: as literals they would cost an instruction each)
    u32 mask = 0x00780078u, offs = 0x41804180u;
    if constexpr (WD == W_INT4) { asm("" : "+s"(mask)); asm("" : "+v"(offs)); }
    SoloTile<WD> cur, nxt;
    u32x4 x[NX], xn[NX];
    cur.read(slot, lane);
#pragma unroll
    for (int k = 0; k < NX; k++) x[k] = *(const lds_u32x4*)(xa + k * 192);
    int n = n_it * T;   // tiles left, the one in cur included
    for (int i = 0; i < n_it; i++) {
        const int in = min(i + 1, n_it - 1);
#pragma unroll
        for (int k = 0; k < NX; k++) xn[k] = *(const lds_u32x4*)(xa + (in * NX + k) * 192);
        // int4: the groups' sums of inputs, by the same instruction (it truncates: sums made in another way would not take its bias off the
        // offset's share of the products again; relative error of the logits, one layer: 3.9e-6 in place of 4.0e-7)
        mfma_f4 X[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        if constexpr (WD == W_INT4) {
            const u32x4 ones{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
            for (int k = 0; k < NX; k++) X[k / 4] = mfma16(x[k], ones, X[k / 4]);
        }
        lds_float* sum = sums + lane;
        for (int t = 0; t < T; t++, sum += 16) {
            cur.arrived();
            feed.request(M, tab, slot);
            slot += R::kTileBytes;
            slot = slot == end ? feed.ring : slot;
            if (--n > 0) nxt.read(slot, lane);
            mfma_f4 d = {0.f, 0.f, 0.f, 0.f};
            float v;
            if constexpr (WD == W_BF16) {
                d = mfma16(x[0], cur.w[0], d);
                d = mfma16(x[1], cur.w[1], d);
                v = (d[0] + d[1]) + d[2];
            } else if constexpr (WD == W_INT8) {
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    d = mfma16(x[2 * h], i8_to_bf16(cur.w[h].x, cur.w[h].y), d);
                    d = mfma16(x[2 * h + 1], i8_to_bf16(cur.w[h].z, cur.w[h].w), d);
                }
                v = (d[0] + d[1]) + d[2];
            } else {
                v = 0.f;
#pragma unroll
                for (int h = 0; h < 2; h++) {   // (an iteration is one group)
                    d = mfma_f4{0.f, 0.f, 0.f, 0.f};
                    d = mfma16(x[4 * h], i4_to_bf16(cur.w[h].x, mask, offs), d);
                    d = mfma16(x[4 * h + 1], i4_to_bf16(cur.w[h].y, mask, offs), d);
                    d = mfma16(x[4 * h + 2], i4_to_bf16(cur.w[h].z, mask, offs), d);
                    d = mfma16(x[4 * h + 3], i4_to_bf16(cur.w[h].w, mask, offs), d);
                    const float s = f16_to_f((f16_t)(cur.sz[h] & 0xFFFFu)), zp = kI4Offset + f16_to_f((f16_t)(cur.sz[h] >> 16));
                    v = fmaf(s, (fmaf(-zp, X[h][0], d[0]) + fmaf(-zp, X[h][1], d[1])) + fmaf(-zp, X[h][2], d[2]), v);
                }
            }
            if (lane < 16) __builtin_amdgcn_ds_faddf(sum, v, 0, 0, false);   // (lanes 0..15: the tile's rows; operand rows 0..2 are the input's parts)
            cur = nxt;
        }
#pragma unroll
        for (int k = 0; k < NX; k++) x[k] = xn[k];
    }
}

template <int WD, int HD, int G>
__global__ void __launch_bounds__(kSoloThreads) solo_decode_kernel(DevModel M, DevKV KV, const int* __restrict__ tokens, const int* __restrict__ pos,
                                                                   float* __restrict__ logits, int lm_in_kernel, int ncta, int mute_wg, int switches) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    typedef SoloRing<WD> R;
    typedef SoloLds<WD> Lds;
    if (!inputs_ok(M, KV, tokens, pos)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(M.status, kStatusRange);
        return;
    }
    if ((int)blockIdx.x == mute_wg) return;   // test hook for the time-out path: this workgroup publishes nothing
    const int tid = threadIdx.x, lane0 = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float2* rope = (float2*)(lds + Lds::kRope);
    float* xres = (float*)(lds + Lds::kRes);
    int* pos_lds = (int*)(lds + Lds::kInt);
    int* share_lds = pos_lds + 1;
    volatile int* failed = pos_lds + 2;
    float* rms = (float*)(lds + Lds::kRms);
    lds_float* red = (lds_float*)(lds + Lds::kRed);
    lds_u8* area = (lds_u8*)(lds + Lds::kImg) + wave * kSoloImgBytes;
    const u32 steps_done = (u32)__builtin_amdgcn_readfirstlane(xld_u32(M.stepctr));
    if (tid == 0) xadd_u32(M.stepctr + 2, 1u);   // this workgroup has read the counter
    const u32 sl = steps_done * (u32)M.L;
    const u32 tag_base = steps_done * (u32)(kTagsPerLayer * M.L + 1);
    const UDiv n_ctas = UDiv::of((u32)ncta);
    const int n_phases = 4 * M.L + lm_in_kernel;
    SoloFeed<WD> feed;
    feed.ring = (u32)(size_t)(lds_u8*)lds + wave * R::kBytes;
    feed.wave = wave; feed.lane = lane0; feed.n_phases = n_phases;
    feed.bounded = WD == W_BF16 && (switches & kSwNoOverlap) != 0;
    lds_mat* tab = (lds_mat*)(lds + Lds::kTab);
    if (tid < 5) solo_table<WD>(tab, M, n_ctas, tid, lm_in_kernel != 0);
    wg_barrier_lds();
    feed.begin(M, tab, 0);
    if (!feed.bounded) feed.fill(M, tab);
    u32 slot = feed.ring;   // LDS address of the tile that is multiplied next: where the next request goes
    const int p0 = step_pos(tokens, pos, 0);   // -1: the sequence sits this step out
    const bf16_t* erow = M.embed + (size_t)max(as_global(tokens)[0], 0) * M.d;
    const RowRange own = wide_rows(M.d, n_ctas);
    if (tid < HD / 2) rope[tid] = KV.rope[(size_t)max(p0, 0) * (HD / 2) + tid];
    if (tid < own.r1 - own.r0) xres[tid] = bf_to_f(as_global(erow)[own.r0 + tid]);
    if (tid == 0) {
        pos_lds[0] = p0;
        share_lds[0] = attn_share_of(tokens, pos, 1, 0, ncta, M.Hkv, false);
        *failed = 0;
    }
    WgVote vote{(u32*)(pos_lds + 4), 0u};
    wg_barrier_lds();
    auto leave = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };   // nothing may arrive in LDS behind the kernel's end
    auto timed = [&](int ph, int ev) { if (M.dbg && blockIdx.x == 0 && tid == 0) as_global(M.dbg)[ph * kEvSlots + ev] = wall_clock64(); };
    int buf = 0;   // partial sums: the halves alternate from panel to panel
    for (int ph = 0; ph < n_phases; ph++) {
        const int l = ph >> 2, kind = ph == 4 * M.L ? PH_LM : ph & 3;
        // (what depends on the lane only is cheap to compute again: kept from being hoisted out of the loop over phases and spilled)
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        const lds_mat* W = tab + kind;
        const size_t off = kind == PH_LM ? 0 : (size_t)l * M.layer_stride;
        const int r0 = uni(W->r0), rows = uni(W->rows), K = uni(W->k), nu = uni(W->nu), T = uni(W->tiles);
        const f16_t* wscale = (const f16_t*)(uni(W->s) + off);
        const bf16_t* gain = (const bf16_t*)(uni(W->gain) + off);
        bool ok = true;   // of this wave
        if (kind == PH_O) {
            timed(ph, EV_ATT_START);
            u64* aev = M.dbg && l == 1 ? M.dbg + (size_t)(4 * M.L + 1) * kEvSlots + (size_t)ncta * 32 + ((size_t)blockIdx.x * 5 + 4) * 8 : nullptr;
            if (aev && tid == 0) { as_global(aev)[0] = wall_clock64(); as_global(aev)[4] = 0; as_global(aev)[5] = 0; }
            if (!attention_phase_tagged<kSoloWaves, HD, G, kAttnModeOf<WD>, true>(M, KV, pos_lds, share_lds, 1, l, lds + Lds::kImg, tag_of(tag_base, l, TAG_QKV),
                                                                                         tag_of(tag_base, l, TAG_ATT), sl + (u32)l, n_ctas, vote, ok, aev)) {
                leave();
                return;
            }
            if (aev && tid == 0) as_global(aev)[6] = wall_clock64();
            timed(ph, EV_ATT_END);
        }
        if (rows <= 0) {
            if (!wave_all(ok)) *failed = 1;
            continue;
        }
        timed(ph, EV_H_START);
        const int nit = wave < nu ? (nu - wave + kSoloWaves - 1) / kSoloWaves : 0;   // units of this wave
        constexpr int IPP = kSoloPassCols / kUCols<WD>;                               // units per pass
        const int npass = (nit + IPP - 1) / IPP;
        const bool normed = kind == PH_QKV || kind == PH_GU || kind == PH_LM;
        const cword_t* src = kind == PH_O ? M.cattn_o : kind == PH_GU ? M.cx2 : kind == PH_DOWN ? M.ch : M.cx;
        const u32 cnt = sl + (u32)l - (kind == PH_QKV || kind == PH_LM ? 1u : 0u);
        lds_u8* sc = (lds_u8*)(lds + Lds::kScale) + (ph & 1) * kSoloScaleRows * 2;
        if constexpr (WD == W_INT8) {
            if (rows <= kSoloScaleRows)
                for (int i = tid; i < rows; i += kSoloThreads) *(__attribute__((address_space(3))) f16_t*)(sc + 2 * i) = as_global(wscale)[r0 + i];
        }
        u32x4 gw[kSoloPasses];   // gains of the wave's columns (normalised inputs have at most kSoloPasses passes)
        SoloWords X;
        X.undefined();
#pragma unroll
        for (int s = 0; s < kSoloPasses; s++) asm volatile("" : "=v"(gw[s]));   // (defined in every phase: else it would be kept alive from one to the next)
        if (normed) {
#pragma unroll
            for (int s = 0; s < kSoloPasses; s++) gw[s] = *as_global((const u32x4*)(gain + min(SoloWords::col_of<WD>(s, wave, lane), K - 8)));
        }
        float ss = 0.f;
        for (int p = 0, left = rows; left > 0; p++, left -= 16 * T) {
            lds_float* part = red + buf * kSoloWaves * kSoloPanelRows;   // the waves' sums
            part[wave * kSoloPanelRows + lane] = 0.f;
            if (lane < kSoloPanelRows - 64) part[wave * kSoloPanelRows + 64 + lane] = 0.f;
            // columns of pass s (words in X.w[i]) as operands into slot i of the area
            auto operands = [&](int s, int i) {
                const bool there = SoloWords::col_of<WD>(s, wave, lane) < K;
                float t[8];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    t[2 * j] = there ? cvalue(X.w[i][j].x) : 0.f;
                    t[2 * j + 1] = there ? cvalue(X.w[i][j].y) : 0.f;
                }
                if (normed) {
                    const u32 gv[4] = {gw[i].x, gw[i].y, gw[i].z, gw[i].w};
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        ss = fmaf(t[2 * j], t[2 * j], ss); ss = fmaf(t[2 * j + 1], t[2 * j + 1], ss);
                        t[2 * j] *= bf_lo(gv[j]); t[2 * j + 1] *= bf_hi(gv[j]);
                    }
                }
                solo_operands<WD>(area, i, lane, t);
            };
            if (p == 0 && npass > 0) {
                if (kind == PH_QKV && l == 0) X.embed<WD>(erow, K, npass, wave, lane);
                else ok = X.wait<WD>(src, cnt, K, 0, npass > kSoloPasses ? 1 : npass, wave, lane) && ok;
                timed(ph, EV_SYNCED);
                if (feed.bounded) {   // (measurement switch) the phase's tiles are requested only now
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    slot = feed.ring;
                    feed.begin(M, tab, ph);
                    feed.fill(M, tab);
                }
                operands(0, 0);
                if (npass == kSoloPasses) operands(1, 1);
            }
            // inputs of more passes than the area holds (output and down projections, one panel): pass by pass
            const bool many = npass > kSoloPasses;
            const u32 mail = (u32)(size_t)(area + kSoloPassBytes);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, K * 4, 0x00020000);
            for (int s = 0, ns = many ? npass : 1; s < ns; s++) {
                if (s > 0) {   // (between its words' request and here there were at least IPP tiles)
                    if (!X.land<WD, IPP * R::kLoads>(mail, cnt, K, s, wave, lane)) ok = X.wait<WD>(src, cnt, K, s, 1, wave, lane) && ok;
                    operands(s, 0);
                }
                if (s + 1 < ns) SoloWords::send<WD>(rs, mail, s + 1, wave, lane);
                solo_run<WD>(feed, M, tab, slot, area, lane, many ? min(nit - s * IPP, IPP) : nit, T,
                             part + wave * kSoloPanelRows);
            }
            timed(ph, p == 0 ? 4 : 8);
            if (p == 0 && M.dbg && l == 1 && lane == 0 && kind < 4) as_global(M.dbg)[(size_t)(4 * M.L + 1) * kEvSlots + (blockIdx.x * kSoloWaves + wave) * 4 + kind] = wall_clock64();
            if (p == 0 && normed) {
                ss = wave_sum_uniform(ss);
                if (lane == 0) rms[(ph >> 1 & 1) * kSoloWaves + wave] = ss;
            }
            if (!wave_all(ok)) *failed = 1;
            wg_barrier_lds();
            timed(ph, p == 0 ? 5 : 9);
            if (__builtin_amdgcn_readfirstlane(*failed)) {
                if (tid == 0) atomicCAS(M.status, 0, -55 - 10 * ph);
                leave();
                return;
            }
            const int r = 16 * T * p + tid;   // row of the workgroup
            if (tid < min(left, 16 * T)) {
                const int row = r0 + r;
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < kSoloWaves; w++) v += part[w * kSoloPanelRows + tid];
                if (normed) {
                    float q = 0.f;
#pragma unroll
                    for (int w = 0; w < kSoloWaves; w++) q += rms[(ph >> 1 & 1) * kSoloWaves + w];
                    v *= rsqrtf(q / (float)K + M.eps);
                }
                if constexpr (WD == W_INT8)
                    v *= f16_to_f(rows <= kSoloScaleRows ? *(__attribute__((address_space(3))) f16_t*)(sc + 2 * r) : as_global(wscale)[row]);
                const float other = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));   // the neighbouring row of the pair
                if (kind == PH_QKV) {
                    const int half = HD / 2, nq = M.Hq * HD, nk = M.Hkv * HD, at = pos_lds[0];
                    const u32 tag = tag_of(tag_base, l, TAG_QKV);
                    if (row < nq + nk) {   // rows 2 i, 2 i + 1 of a head: elements i, i + hd / 2
                        const bool isq = row < nq;
                        const int e = isq ? row : row - nq, head = e / HD, i = (e % HD) / 2, dim = i + (e & 1) * half;
                        const float2 cs = rope[i];
                        const float y = (e & 1) ? v * cs.x + other * cs.y : v * cs.x - other * cs.y;
                        if (isq) tst(M.tq + head * HD + dim, y, tag);
                        else {
                            const bf16_t h = f_to_bf(y);
                            tst(M.tkvcur + head * HD + dim, bf_to_f(h), tag);
                            if (at >= 0) as_global(KV.plane(M, l, 0, head, 0))[(size_t)at * HD + dim] = h;
                        }
                    } else {
                        const int e = row - nq - nk, head = e / HD, dim = e % HD;
                        const bf16_t h = f_to_bf(v);
                        tst(M.tkvcur + (M.Hkv + head) * HD + dim, bf_to_f(h), tag);
                        if (at >= 0) as_global(KV.plane(M, l, 0, head, 1))[(size_t)at * HD + dim] = h;
                    }
                } else if (kind == PH_GU) {   // rows 2 f, 2 f + 1: gate and up of unit f
                    if (!(tid & 1)) cst1(M.ch + (row >> 1), v / (1.0f + expf(-v)) * other, sl + (u32)l);
                } else if (kind == PH_LM) {
                    if (pos_lds[0] >= 0) as_global(logits)[row] = v;   // (no logits for a sequence that sits the step out)
                } else {
                    const float x = xres[r] + v;
                    xres[r] = x;
                    cst1((kind == PH_O ? M.cx2 : M.cx) + row, x, sl + (u32)l);
                    if (ph == 4 * M.L - 1 && !lm_in_kernel) as_global(M.x)[row] = x;   // the LM head runs as launches of its own
                }
            }
            buf ^= 1;
        }
        timed(ph, EV_RUN_DONE);
    }
    leave();
    // the next step's counters: once every workgroup has read this step's
    if (blockIdx.x == 0 && tid == 0) {
        const u32 all = (steps_done + 1u) * (u32)ncta;
        for (int spins = 0; spins < kSpinLimit && (int)(xld_u32(M.stepctr + 2) - all) < 0; spins++) __builtin_amdgcn_s_sleep(1);
        xst_u32(M.stepctr + 1, 1u);
        xst_u32(M.stepctr, steps_done + 1u);
    }
}

}  // namespace ff
