// Implicit-GEMM convolution with an LDS-DMA pipeline (gfx950).
//
// Same GEMM as conv_bf16 (C[M][N] = A[M][K] * B[N][K]^T over the merged
// frames of several models, bf16 MFMA, fp32 accumulation, fused epilogue),
// organised for latency tolerance: each depth step of 32 or 64 is fetched by
// global_load_lds_dwordx4 straight into one of STAGES LDS buffers, so
// STAGES-1 steps are in flight while the MFMAs consume the oldest one (all
// STAGES where a step's fragments wait in registers) and no registers hold
// staged data. Each stage lives in its own __shared__
// array (the compiler then tracks which buffer an outstanding LDS-DMA
// writes and waits only where a read could alias it); the waits on the
// loads are explicit vmcnt counts, and workgroup syncs are bare s_barrier
// (a fenced barrier would drain every outstanding load).
//
// An LDS-DMA instruction writes 64 consecutive 16-byte slots per wave, so
// the layout is chosen through the addresses: slot p of a stage holds row
// p/4, 16-byte chunk (p%4) ^ ((row/2)%4) of that row. The swizzle puts the
// 16-byte fragment reads of 8 consecutive rows at the same chunk onto
// distinct banks.
//
// Requirements: Cin a multiple of 32 (a step is one filter tap and 32
// channels), input pixel stride a multiple of 8, depth per split a
// multiple of 32.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "conv_epi.h"
#include "kargs.h"
#include "kernels.h"

namespace gemel {

namespace {

typedef __attribute__((address_space(3))) unsigned char lds_u8;

// Calls f(std::integral_constant<int, i>) for i = 0 .. I-1 with a
// compile-time i, so that register arrays are indexed statically.
template <int I>
struct StaticFor {
    template <typename F>
    __device__ __forceinline__ static void run(F &&f) {
        StaticFor<I - 1>::run(f);
        f(std::integral_constant<int, I - 1>{});
    }
};
template <>
struct StaticFor<0> {
    template <typename F>
    __device__ __forceinline__ static void run(F &&) {}
};

// vmcnt-only wait: expcnt and lgkmcnt left at their maxima (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Waits until at most n steps of PER vm operations each are in flight, for a
// uniform n in 0 .. MAXN-1 (s_waitcnt takes an immediate, so one branch per
// count).
template <int PER, int MAXN>
__device__ __forceinline__ void wait_steps(int n) {
    StaticFor<MAXN>::run([&](auto c) __attribute__((always_inline)) {
        constexpr int i = decltype(c)::value;
        if (n == i) wait_vm<i * PER>();
    });
}

// lgkmcnt(0) only: vmcnt and expcnt left at their maxima (gfx9 encoding).
__device__ __forceinline__ void wait_lgkm0() {
    __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
}

}  // namespace

// MODE 1: the 2x2 stride-2 max pool fused (out_mode OUT_NHWC_POOL2);
// MODE 2: segments of different spatial sizes (ConvArgs::hetero). Separate
// instantiations, so that the plain kernels keep their code and registers.
// Waves per SIMD the kernel is compiled for: two where the LDS of two
// workgroups fits one CU and a workgroup has at most 4 waves (the register
// budget then allows both), else one.
template <int BM, int BN, int WM, int WN, int STAGES, int BK>
constexpr int dma_min_waves() {
    return WM * WN <= 4 && 2 * STAGES * (BM + BN) * BK * 2 <= 160 * 1024 ? 2 : 1;
}

template <int BM, int BN, int WM, int WN, int STAGES, int BK, int MODE>
__global__ __launch_bounds__(64 * WM *WN, (dma_min_waves<BM, BN, WM, WN, STAGES, BK>())) void conv_dma_kernel(
    const ConvArgs a) {
    constexpr int NW = WM * WN, NT = 64 * NW;
    static_assert(BK == 32 || BK == 64, "step depth");
    constexpr int CPR = BK / 8;                                 // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;                               // rows per DMA instruction
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / 16, FN = TN / 16;
    // 16-byte slots per stage; the rows of A are loaded by whole
    // instructions of the workgroup (rows beyond BM, which no fragment
    // reads, come from the zero page)
    constexpr int A_SLOTS = (BM * CPR + NT - 1) / NT * NT, B_SLOTS = BN * CPR;
    constexpr int AI = A_SLOTS / NT, BI = B_SLOTS / NT;        // DMA instructions per thread
    static_assert(AI * NT == A_SLOTS && BI * NT == B_SLOTS && AI >= 1 && BI >= 1, "tile/threads");
    constexpr int STAGE_BYTES = (A_SLOTS + B_SLOTS) * 16;
    constexpr int EPI_LD = TN + 4;                              // fp32 row pitch of a wave's staging
    static_assert(STAGES >= 2 && STAGES <= 4, "stages");
    static_assert(TN % 8 == 0 && 64 % (TN / 8) == 0 && TN <= 512,
                  "every epilogue item of a lane is the same 8-channel chunk of its wave's columns");
    constexpr int PER_STEP = AI + BI;                           // vm ops per thread per step
    // register double-buffered fragments (below): only where a second
    // fragment set fits beside the accumulators (512-thread workgroups have
    // 256 registers per lane). A stage's fragments are then in registers
    // before its MFMAs start, so every stage can be in flight.
    constexpr bool PIPE = STAGES == 4 && (NT <= 256 || FM * FN <= 16);
    constexpr int AHEAD = PIPE ? STAGES : STAGES - 1;           // steps requested before the depth loop
    // the phased loop (below, the 224 x 256 tile): its fragments and
    // accumulators take 176 of a lane's 256 registers, so it keeps the
    // loader's state small (256 rows did not fit: 40 to 100 bytes of scratch)
    constexpr bool PHASED = STAGES == 2 && BK == 64 && NT == 512 && FM == 7;
    __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGES > 2 ? STAGE_BYTES : 16];
    __shared__ __attribute__((aligned(1024))) unsigned char st3[STAGES > 3 ? STAGE_BYTES : 16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave - (wave / WN) * WN;
    const int tiles_n = (a.N + BN - 1) / BN;
    const int G = gridDim.x;
    const int t = (G & 7) == 0 ? (int)(blockIdx.x & 7) * (G >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    // the tile's rows [m_lo, min(m_lo + BM, m_end)), column tile tn and
    // weights. Grouped launches tile every segment on its own (a tile never
    // straddles two segments' weights; seg[s].t_start is its first tile).
    // Segment fields are gathered with selects over a static walk of the
    // table: indexing the argument block with a computed segment number
    // makes the compiler copy the whole block to scratch memory.
    int m_lo, m_end = a.M, tn, tiles;
    const void *wseg = a.w;
    if (a.grouped) {
        int ts = 0, ms = 0;
        bool past = false;
        for (int i = 0; i < a.nseg; ++i) {
            const int ti = a.seg[i].t_start, mi = a.seg[i].m_start;
            const void *wi = a.seg[i].w;
            const bool hit = t >= ti;
            if (!hit && !past) m_end = mi;   // the next segment's first row
            past = past || !hit;
            ts = hit ? ti : ts;
            ms = hit ? mi : ms;
            wseg = hit ? wi : wseg;
            tiles = ti + ((i + 1 < a.nseg ? a.seg[i + 1].m_start : a.M) - mi + BM - 1) / BM * tiles_n;
        }
        const int local = t - ts, tml = local / tiles_n;
        tn = local - tml * tiles_n;
        m_lo = ms + tml * BM;
    } else {
        tiles = ((a.M + BM - 1) / BM) * tiles_n;
        const int tm = t / tiles_n;
        tn = t - tm * tiles_n;
        m_lo = tm * BM;
    }
    if (t >= tiles) return;
    const int k_begin = blockIdx.y * a.k_per_split;
    const int k_end = min(a.K, k_begin + a.k_per_split);
    const int N = a.N, K = a.K;
    const int nk = (k_end - k_begin) / BK;

    // ---- DMA assignment: instruction i of this thread fills slot
    // (i*NW + wave)*64 + lane: row (i*NW + wave)*RPI + lane/CPR; the slot's
    // chunk position lane%CPR holds logical chunk (lane%CPR) ^ sw(row) ----
    auto sw = [](int row) __attribute__((always_inline)) { return (row >> 1) & (CPR - 1); };
    // weight rows beyond N read row 0 instead (their columns are never stored)
    // (PHASED: 32-bit byte offsets from the weights' base)
    const u16 *bbase[PHASED ? 1 : BI];
    uint32_t boff32[PHASED ? BI : 1];
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int rl = (i * NW + wave) * RPI + lane / CPR;
        const int gn = tn * BN + rl;
        if constexpr (PHASED)
            boff32[i] = ((uint32_t)(gn < N ? gn : 0) * (uint32_t)K + ((lane % CPR) ^ sw(rl)) * 8) * 2;
        else
            bbase[i] = (const u16 *)wseg + (size_t)(gn < N ? gn : 0) * K + ((lane % CPR) ^ sw(rl)) * 8;
    }
    int kb = k_begin;   // next step's depth of the weight loads
    auto issue_b = [&](unsigned char *stage) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const void *p;
            if constexpr (PHASED)
                p = (const char *)((const u16 *)wseg + kb) + boff32[i];
            else
                p = bbase[i] + kb;
            __builtin_amdgcn_global_load_lds(p, (lds_u8 *)(stage + A_SLOTS * 16 + (i * NW + wave) * 1024), 16, 0, 0);
        }
        kb += BK;
    };
    // the weights of the first two steps are requested before the input rows
    // are worked out: their addresses are few, and they often come from HBM,
    // whose latency then passes under the row arithmetic
    constexpr int EARLY = AHEAD < 2 ? AHEAD : 2;
    unsigned char *const stg[4] = {st0, st1, st2, st3};
    if constexpr (!PHASED) {
#pragma unroll
        for (int s = 0; s < EARLY; ++s)
            if (s < nk) issue_b(stg[s]);
    }
    const int HWo = a.Ho * a.Wo;
    const int H = a.H, W = a.W, in_cs = a.in_cs, Cin = a.Cin, kw = a.kw;
    const size_t frame_elems = (size_t)H * W * in_cs;
    const u16 *const zp = (const u16 *)a.zero;
    // segment of the tile's first and last row (wave-uniform, scalar loads):
    // rows of a tile inside one segment take its fields as uniform values;
    // per-row lookups only for a tile that straddles segments
    const int m_first = m_lo, m_last = min(m_end, m_first + BM) - 1;
    int s_first = 0, s_last = 0;
    for (int i = 1; i < a.nseg; ++i) {
        s_first += m_first >= a.seg[i].m_start ? 1 : 0;
        s_last += m_last >= a.seg[i].m_start ? 1 : 0;
    }
    const bool one_seg = s_first == s_last;
    const RowSeg useg = uni_seg(a, s_first);
    // (the walk out of the way of the usual path: every line of a kernel's
    // code that runs is fetched anew at most launches)
    auto seg_of = [&](int gm) __attribute__((always_inline)) {
        return __builtin_expect(one_seg, 1) ? useg : row_seg(a, gm);
    };

    // with the 2x2 max pool fused, rows run over the output in window
    // order: row 4g + 2dy + dx is pixel (2hp + dy, 2wp + dx) of pooled pixel g
    constexpr bool pool2 = MODE == 1;
    // with segments of different sizes, each row takes its segment's sizes
    // (and its frame within the segment from the rows before it)
    constexpr bool hetero = MODE == 2;
    static_assert(!PHASED || !hetero, "the phased loop walks one map size");
    const int Wp = a.Wo >> 1, HWp = HWo >> 2;
    const u16 *abase[AI];
    int ahi[AI], awi[AI], acq[AI];
    int aH[hetero ? AI : 1], aW[hetero ? AI : 1];
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        const int rl = (i * NW + wave) * RPI + lane / CPR;
        acq[i] = (lane % CPR) ^ sw(rl);
        const int gm = m_lo + rl;
        abase[i] = zp;
        ahi[i] = -(1 << 28);
        awi[i] = 0;
        if constexpr (hetero) {
            aH[i] = 0;
            aW[i] = 0;
        }
        const bool row_ok = gm < m_end && (A_SLOTS == BM * CPR || rl < BM);
        if (hetero && row_ok) {
            // the row's segment sizes: uniform in a tile inside one segment,
            // else gathered with scalar loads and selects like row_seg
            int sH = a.seg[s_first].H, sW = a.seg[s_first].W, sHo = a.seg[s_first].Ho, sWo = a.seg[s_first].Wo;
            if (!one_seg)
                for (int k = 1; k < a.nseg; ++k) {
                    const bool hit = gm >= a.seg[k].m_start;
                    sH = hit ? a.seg[k].H : sH;
                    sW = hit ? a.seg[k].W : sW;
                    sHo = hit ? a.seg[k].Ho : sHo;
                    sWo = hit ? a.seg[k].Wo : sWo;
                }
            const RowSeg sg = seg_of(gm);
            const int local = gm - sg.m_start, hw = sHo * sWo;
            const int fl = local / hw, pix = local - fl * hw, ho = pix / sWo;
            abase[i] = (const u16 *)sg.in + (size_t)fl * sH * sW * in_cs;
            ahi[i] = ho * a.stride - a.pad;
            awi[i] = (pix - ho * sWo) * a.stride - a.pad;
            aH[i] = sH;
            aW[i] = sW;
        } else if (row_ok) {
            int fr, ho, wo;
            // quotients by multiply-high (the launcher's magic numbers): a
            // per-lane integer division costs dozens of instructions
            auto qdiv = [&](int n, int q) __attribute__((always_inline)) {
                return (int)((__umulhi((uint32_t)n, a.dv_m[q]) + (uint32_t)n) >> a.dv_l[q]);
            };
            if constexpr (pool2) {
                const int g = gm >> 2;
                fr = qdiv(g, 0);
                const int pp = g - fr * HWp, hp = qdiv(pp, 1);
                ho = 2 * hp + ((gm >> 1) & 1);
                wo = 2 * (pp - hp * Wp) + (gm & 1);
            } else {
                fr = qdiv(gm, 0);
                const int pix = gm - fr * HWo;
                ho = qdiv(pix, 1);
                wo = pix - ho * a.Wo;
            }
            const RowSeg sg = seg_of(gm);
            abase[i] = (const u16 *)sg.in + (size_t)(fr - sg.f_start) * frame_elems;
            ahi[i] = ho * a.stride - a.pad;
            awi[i] = wo * a.stride - a.pad;
        }
    }
    // loader position (uniform): next step's tap (lr, ls) and channel base lc
    int lc, lr, ls;
    {
        const int rs = k_begin / Cin;
        lc = k_begin - rs * Cin;
        lr = rs / kw;
        ls = rs - lr * kw;
    }
    // each row's source for the current tap, the lane's chunk included: the
    // pixel, or the zero page where the tap falls outside the image (or the
    // row beyond M). Recomputed when the tap changes; a depth step only adds
    // the uniform channel offset (the zero page spans any row's channels).
    // (PHASED: the tap's pixel itself, moved by the taps' uniform distance,
    // and one bit per row for whether it lies in the image)
    const u16 *arow[AI];
    uint32_t inside = 0;
    if constexpr (PHASED) {
#pragma unroll
        for (int i = 0; i < AI; ++i)
            arow[i] = abase[i] + ((ptrdiff_t)(ahi[i] + lr) * W + awi[i] + ls) * in_cs + acq[i] * 8;
    }
    auto set_tap = [&]() __attribute__((always_inline)) {
        if constexpr (PHASED) inside = 0;
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            const int hi = ahi[i] + lr, wi = awi[i] + ls;
            const int Hr = hetero ? aH[hetero ? i : 0] : H, Wr = hetero ? aW[hetero ? i : 0] : W;
            const bool ok = (unsigned)hi < (unsigned)Hr && (unsigned)wi < (unsigned)Wr;
            if constexpr (PHASED)
                inside |= ok ? 1u << i : 0u;
            else
                arow[i] = (ok ? abase[i] + (size_t)(hi * Wr + wi) * in_cs : zp) + acq[i] * 8;
        }
    };
    set_tap();
    auto issue_a = [&](unsigned char *stage) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            const u16 *p = arow[i];
            if constexpr (PHASED) p = (inside >> i) & 1 ? p : zp;
            __builtin_amdgcn_global_load_lds((const void *)(p + lc), (lds_u8 *)(stage + (i * NW + wave) * 1024), 16, 0,
                                             0);
        }
        lc += BK;
        if (lc == Cin) {
            lc = 0;
            const bool wrap = ++ls == kw;
            if constexpr (PHASED) {
#pragma unroll
                for (int i = 0; i < AI; ++i) arow[i] += wrap ? (W - (kw - 1)) * in_cs : in_cs;
            }
            if (wrap) { ls = 0; ++lr; }
            set_tap();
        }
    };
    auto issue = [&](unsigned char *stage) __attribute__((always_inline)) {
        issue_a(stage);
        issue_b(stage);
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // fragment read offsets inside a stage (swizzled slots): a fragment row
    // is wave-tile row 16*i + lane%16 (a multiple of 16 plus lane%16), so
    // its swizzle depends on the lane only
    const int g = lane >> 4;
    const int swl = sw(lane & 15);
    int aoff[FM], boff[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) aoff[i] = (wm * TM + i * 16 + (lane & 15)) * CPR * 16;
#pragma unroll
    for (int j = 0; j < FN; ++j) boff[j] = A_SLOTS * 16 + (wn * TN + j * 16 + (lane & 15)) * CPR * 16;
    // fragments of one depth step in registers: H halves of 32
    constexpr int NH = BK / 32;
    typedef bf16x8 FragA[NH][FM];
    typedef bf16x8 FragB[NH][FN];
    auto read_frags = [&](const unsigned char *stage, FragA &fa, FragB &fb) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int pos = ((h * 4 + g) ^ swl) * 16;
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[h][j] = *(const bf16x8 *)(stage + boff[j] + pos);
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[h][i] = *(const bf16x8 *)(stage + aoff[i] + pos);
        }
    };
    auto mfmas = [&](const FragA &fa, const FragB &fb) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][j], acc[i][j], 0, 0, 0);
    };
    auto compute = [&](const unsigned char *stage) __attribute__((always_inline)) {
        FragA fa;
        FragB fb;
        read_frags(stage, fa, fb);
        mfmas(fa, fb);
    };

    // epilogue constants of this lane's 8 channels (every segment shares
    // one scale/shift pair), fetched ahead of the depth loop (PHASED: after
    // it, where the fragments' registers are free)
    const int my_gn = tn * BN + wn * TN + (lane % (TN / 8)) * 8;
    f32x4 sc0 = {1.f, 1.f, 1.f, 1.f}, sc1 = sc0, sh0 = {0.f, 0.f, 0.f, 0.f}, sh1 = sh0;
    auto load_affine = [&]() __attribute__((always_inline)) {
        if (a.k_splits <= 1 && my_gn < N) {
            const float *scl = useg.scale + my_gn, *shl = useg.shift + my_gn;
            sc0 = *(const f32x4 *)scl;
            sc1 = *(const f32x4 *)(scl + 4);
            sh0 = *(const f32x4 *)shl;
            sh1 = *(const f32x4 *)(shl + 4);
        }
    };
    if constexpr (!PHASED) load_affine();

    // the inputs of the first steps, and the weights beyond the early ones: a
    // step's loads are in flight in the order inputs, weights, but for the
    // early weights, which are older than everything here. Step 0 must then
    // land: behind its inputs, the second step's inputs and the whole steps
    // after it may fly (the waits of the loops below count whole steps
    // behind the one they need).
    auto prologue = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s)
            if (s < nk) {
                if (s < EARLY)
                    issue_a(stg[s]);
                else
                    issue(stg[s]);
            }
        if (AHEAD > 3 && nk > 3)
            wait_vm<AI + 2 * PER_STEP>();
        else if (AHEAD > 2 && nk > 2)
            wait_vm<AI + PER_STEP>();
        else if (AHEAD > 1 && nk > 1)
            wait_vm<AI>();
        else
            wait_vm<0>();
    };

    if constexpr (PHASED) {
        // Two stages of depth 64 and 8 waves (two per SIMD) of 7 x 4
        // fragments. A step is a row of phases (two halves of 32 depths x
        // groups of G0 fragment rows), and each phase reads the fragments of
        // the next one from LDS before its own MFMAs, so that the LDS reads
        // of a step (176 KB, about as many cycles as its MFMAs) run beside
        // them. The one barrier of a step stands before
        // its last phase: every wave has then read all of the step's stage
        // (its last fragments arrived) and its own loads of the next stage
        // have landed, so the stage is refilled for step s + 2 (a whole
        // step of time to land) and the next stage's first fragments are
        // read under the last phase's MFMAs.
        constexpr int G0 = (FM + 1) / 2;
        constexpr int NG = (FM + G0 - 1) / G0, NP = 2 * NG;
        bf16x8 fa[2][G0], fb[2][FN];
        // fragments of phase P (its B fragments with a half's first group)
        auto rd = [&](const unsigned char *stage, auto pc) __attribute__((always_inline)) {
            constexpr int P = decltype(pc)::value, h = P / NG, grp = P % NG;
            const int pos = ((h * 4 + g) ^ swl) * 16;
            if constexpr (grp == 0) {
#pragma unroll
                for (int j = 0; j < FN; ++j) fb[h][j] = *(const bf16x8 *)(stage + boff[j] + pos);
            }
            StaticFor<G0>::run([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                if constexpr (grp * G0 + i < FM) fa[P & 1][i] = *(const bf16x8 *)(stage + aoff[grp * G0 + i] + pos);
            });
        };
        auto mm = [&](auto pc) __attribute__((always_inline)) {
            constexpr int P = decltype(pc)::value, h = P / NG, grp = P % NG;
            StaticFor<G0>::run([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                if constexpr (grp * G0 + i < FM) {
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc[grp * G0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[P & 1][i], fb[h][j],
                                                                                       acc[grp * G0 + i][j], 0, 0, 0);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        // the phases of a step over stage cur; more: a next step exists (in
        // nxt), refill: one after it does
        auto do_step = [&](unsigned char *cur, unsigned char *nxt, bool more, bool refill) __attribute__((always_inline)) {
            StaticFor<NP - 1>::run([&](auto pc) __attribute__((always_inline)) {
                rd(cur, std::integral_constant<int, decltype(pc)::value + 1>{});
                mm(pc);
            });
            wait_lgkm0();
            if (more) {
                wait_vm<0>();
                __builtin_amdgcn_s_barrier();
                if (refill) issue(cur);
                __builtin_amdgcn_sched_barrier(0);
                rd(nxt, std::integral_constant<int, 0>{});
            }
            mm(std::integral_constant<int, NP - 1>{});
        };
        // a prologue of its own for the steady loop, without branches: the
        // compiler's waits then see one path into it (merged with the short
        // one, it drained every load at the top of the loop)
        int it = 0;
        if (nk >= 4) {
            issue(st0);
            issue(st1);
            wait_vm<PER_STEP>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            rd(st0, std::integral_constant<int, 0>{});
            do {
                do_step(st0, st1, true, true);
                do_step(st1, st0, true, true);
                it += 2;
            } while (it + 3 < nk);
        } else if (nk > 0) {
            issue(st0);
            if (nk > 1) issue(st1);
            wait_steps<PER_STEP, 2>(min(nk - 1, 1));
            __builtin_amdgcn_s_barrier();
            rd(st0, std::integral_constant<int, 0>{});
        }
        for (; it < nk; it += 2) {
            do_step(st0, st1, it + 1 < nk, it + 2 < nk);
            if (it + 1 < nk) do_step(st1, st0, it + 2 < nk, it + 3 < nk);
        }
    } else if constexpr (PIPE) {
        // Fragments double-buffered in registers: iteration it reads step
        // it+1's fragments from LDS, then issues step it's MFMAs from the
        // registers filled one iteration earlier, so the LDS reads overlap
        // the MFMAs. Step it's fragments have then left its stage: once
        // every wave has passed this iteration's barrier, the stage is
        // refilled for step it+STAGES, and STAGES-1 steps are in flight (a
        // small tile's step takes the latency of a load divided by the steps
        // in flight: LDS and MFMAs are idle for most of it). With STAGES-2
        // steps in flight before: M 3136, N 256, K 2304 13.9 -> 12.1 us, M 784,
        // N 512, K 2048 15.7 -> 12.7 us (weights from HBM).
        FragA fa[2];
        FragB fb[2];
        int base = 0;
        if (nk >= STAGES) {
            // the prologue without its branches: the compiler's waits then
            // see one path into the loop (merged with the short one, it
            // drained every load before the first step)
            issue_a(stg[0]);
            issue_a(stg[1]);
            issue(stg[2]);
            issue(stg[3]);
            wait_vm<AI + 2 * PER_STEP>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            read_frags(stg[0], fa[0], fb[0]);
            // steady state: every iteration of the group waits, issues the
            // DMA STAGES steps ahead and reads the next fragments (no
            // branches here either). The fragments read one iteration ago
            // (the operands of the MFMAs) have long arrived: waiting for
            // them before the barrier frees their stage, and keeps the
            // compiler from waiting for them after the next reads.
            if (base + 2 * STAGES <= nk) do {
#pragma unroll
                for (int s = 0; s < STAGES; ++s) {
                    wait_lgkm0();
                    wait_vm<(STAGES - 2) * PER_STEP>();
                    __builtin_amdgcn_s_barrier();
                    issue(stg[s]);
                    read_frags(stg[(s + 1) % STAGES], fa[(s + 1) & 1], fb[(s + 1) & 1]);
                    mfmas(fa[s & 1], fb[s & 1]);
                }
                base += STAGES;
            } while (base + 2 * STAGES <= nk);
        } else if (nk > 0) {
            prologue();
            __builtin_amdgcn_s_barrier();
            read_frags(stg[0], fa[0], fb[0]);
        }
        // the last groups, with the bounds checks
        for (; base < nk; base += STAGES) {
#pragma unroll
            for (int s = 0; s < STAGES; ++s) {
                const int it = base + s;
                if (it < nk) {
                    wait_lgkm0();   // on both paths: no read pending on the MFMAs' operands
                    if (it + 1 < nk) {
                        // step it+1 must have landed; the newer steps issued
                        // (up to it+STAGES-1, none beyond nk-1) may fly
                        wait_steps<PER_STEP, STAGES - 1>(min(nk - it - 2, STAGES - 2));
                        __builtin_amdgcn_s_barrier();
                        if (it + STAGES < nk) issue(stg[s]);
                        read_frags(stg[(s + 1) % STAGES], fa[(s + 1) & 1], fb[(s + 1) & 1]);
                    }
                    mfmas(fa[s & 1], fb[s & 1]);
                }
            }
        }
    } else {
        prologue();
        // main loop, unrolled by STAGES so that every buffer index is static
        for (int base = 0; base < nk; base += STAGES) {
#pragma unroll
            for (int s = 0; s < STAGES; ++s) {
                const int it = base + s;
                if (it < nk) {
                    // step it must have landed; the newer steps issued (up
                    // to it+STAGES-2, none beyond nk-1) may still fly
                    wait_steps<PER_STEP, STAGES - 1>(min(nk - it - 1, STAGES - 2));
                    __builtin_amdgcn_s_barrier();
                    if (it + STAGES - 1 < nk) issue(stg[(s + STAGES - 1) % STAGES]);
                    compute(stg[s]);
                }
            }
        }
    }

    // ---- epilogue: each wave stages PG passes of 16 rows of its tile at a
    // time in its share of the stage buffers. Only the accumulator dump is
    // unrolled per pass; the store code exists once (a kernel larger than
    // the instruction cache pays for its cold misses on every launch).
    constexpr int WPS = (NW + STAGES - 1) / STAGES;             // waves per stage buffer
    constexpr int PASS_FLOATS = 16 * EPI_LD;
    constexpr int GMAX = STAGE_BYTES / (WPS * PASS_FLOATS * 4);
    static_assert(GMAX >= 1, "a 16-row pass must fit a wave's share of a stage buffer");
    constexpr int PG = (GMAX >= 4 && FM % 4 == 0) ? 4 : (GMAX >= 2 && FM % 2 == 0) ? 2 : 1;
    constexpr int NGRP = FM / PG;
    constexpr int CHW = TN / 8;                                 // 8-channel chunks per wave row
    constexpr int ITEMS = PG * 16 * CHW / 64;                    // (row, chunk) items per lane per group
    static_assert(ITEMS * 64 == PG * 16 * CHW, "items per lane");
    if constexpr (PHASED) load_affine();
    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    const int sidx = wave % STAGES;
    unsigned char *const sbuf = sidx == 0 ? st0 : sidx == 1 ? st1 : sidx == 2 ? st2 : st3;
    float *const ew = (float *)(sbuf + (wave / STAGES) * PG * PASS_FLOATS * 4);
    const int out_cs = a.out_cs;
    const __amdgpu_buffer_rsrc_t pr = partial_rsrc(a.partial, (uint32_t)a.k_splits * a.M * N * 4u);
    const int ch = lane % CHW;                                  // this lane's chunk in every item
    const int gn = my_gn;
    const bool col_ok = gn < N;
    const bool pre_res = a.has_res && a.k_splits <= 1;
    const bool planes = MODE == 0 && a.out_mode == OUT_NCHW_F32 && a.k_splits <= 1;
    const int ekind = epi_kind(a.act, a.has_res, a.res_mode, a.slope);
    const float s8[8] = {sc0[0], sc0[1], sc0[2], sc0[3], sc1[0], sc1[1], sc1[2], sc1[3]};
    const float h8[8] = {sh0[0], sh0[1], sh0[2], sh0[3], sh1[0], sh1[1], sh1[2], sh1[3]};
#pragma nounroll
    for (int grp = 0; grp < NGRP; ++grp) {
        const int row0 = m_lo + wm * TM + grp * PG * 16;
        // residuals of the group's items, loaded ahead of the staging
        u32x4 rv[ITEMS];
#pragma unroll
        for (int u = 0; u < ITEMS; ++u) {
            rv[u] = u32x4{0u, 0u, 0u, 0u};
            const int gm = row0 + (lane + u * 64) / CHW;
            if (pre_res && col_ok && gm < m_end) {
                const RowSeg sg = seg_of(gm);
                rv[u] = *(const u32x4 *)((const u16 *)sg.res + (size_t)(gm - sg.m_start) * out_cs + gn);
            }
        }
        StaticFor<NGRP>::run([&](auto gc) __attribute__((always_inline)) {
            constexpr int gi = decltype(gc)::value;
            if (grp == gi) {
                StaticFor<PG>::run([&](auto pc) __attribute__((always_inline)) {
                    constexpr int pp = decltype(pc)::value;
                    constexpr int i = gi * PG + pp;
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            ew[(pp * 16 + (lane >> 4) * 4 + v) * EPI_LD + j * 16 + (lane & 15)] = acc[i][j][v];
                });
            }
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the residual loads (and the previous group's stores) complete
        // here, once: with none pending, the compiler needs no wait between
        // the stores below (vmcnt counts loads and stores together, so a
        // wait for a load would also wait for every earlier store). Without
        // a residual too: a wait under a branch leaves it believing that
        // loads are pending, and it waited before each store instead.
        wait_vm<0>();
        if constexpr (pool2) {
            // pooled items (window, chunk): the window's 4 staged rows through
            // the epilogue, each rounded to bf16 as stored unfused, then their
            // max in window order (what the separate pool computes)
            constexpr int NPI = PG * 4 * CHW;
#pragma unroll
            for (int u = 0; u < (NPI + 63) / 64; ++u) {
                const int idx = lane + u * 64;
                const int pr = idx / CHW;
                const int gm = row0 + 4 * pr;
                if (idx >= NPI || !col_ok || gm >= m_end) continue;
                float mx[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) mx[j] = -INFINITY;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float *src = ew + (4 * pr + q) * EPI_LD + ch * 8;
                    const float4 v0 = *(const float4 *)src, v1 = *(const float4 *)(src + 4);
                    const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
                    float y[8];
                    epi8_f32(v, s8, h8, u32x4{0u, 0u, 0u, 0u}, ekind, 0, 0, a.act, a.slope, y);
#pragma unroll
                    for (int j = 0; j < 8; ++j) mx[j] = fmaxf(mx[j], bf2f(f2bf(y[j])));
                }
                const RowSeg sg = seg_of(gm);
                *(u32x4 *)((u16 *)sg.out + (size_t)((gm - sg.m_start) >> 2) * out_cs + gn) = pack8_bf16(mx);
            }
        } else {
#pragma unroll
        for (int u = 0; u < ITEMS; ++u) {
            const int rl = (lane + u * 64) / CHW;
            const int gm = row0 + rl;
            if (!col_ok || gm >= m_end) continue;
            const float *src = ew + rl * EPI_LD + ch * 8;
            const float4 v0 = *(const float4 *)src, v1 = *(const float4 *)(src + 4);
            if (a.k_splits > 1) {
                const uint32_t off = (uint32_t)((((int)blockIdx.y * a.M + gm) * N + gn) * 4u);
                store_partial4(pr, off, v0);
                store_partial4(pr, off + 16, v1);
                continue;
            }
            const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            const RowSeg sg = seg_of(gm);
            float y[8];
            epi8_f32(v, s8, h8, rv[u], ekind, a.has_res, a.res_mode, a.act, a.slope, y);
            if (planes) {   // back to the staging, for the pass below
                *(float4 *)(ew + rl * EPI_LD + ch * 8) = make_float4(y[0], y[1], y[2], y[3]);
                *(float4 *)(ew + rl * EPI_LD + ch * 8 + 4) = make_float4(y[4], y[5], y[6], y[7]);
            } else {
                store8_bf16((u16 *)sg.out, (size_t)(gm - sg.m_start) * out_cs + gn, y, a.out_pair);
            }
        }
        }
        if (planes) {
            // NCHW fp32 output: consecutive lanes take consecutive rows
            // (pixels), so that a store writes up to 256 contiguous bytes of
            // a channel plane (8 channels of a pixel per lane, 4 bytes each
            // in 8 planes, before: 27.4 -> 16.0 us on M 12544, N 512, K 128)
            constexpr int R = PG * 16, CPL = 64 / R;   // rows, and channel quads side by side
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int rl = lane % R, gm = row0 + rl;
            if (gm < m_end) {
                const RowSeg sg = seg_of(gm);
                const int lr_ = gm - sg.m_start;
                const int f = lr_ / HWo, pix = lr_ - f * HWo;
                int c = tn * BN + wn * TN + lane / R * 4;
                float *o = (float *)sg.out + ((size_t)f * a.cout + c) * HWo + pix;
                const float *y = ew + rl * EPI_LD + lane / R * 4;
                // (unrolled as far as the large tiles' accumulators leave registers)
#pragma unroll FM * FN > 16 ? 1 : 4
                for (int q = 0; q < TN / 4 / CPL; ++q) {
                    const float4 v = *(const float4 *)y;
                    if (c < a.cout) o[0] = v.x;
                    if (c + 1 < a.cout) o[HWo] = v.y;
                    if (c + 2 < a.cout) o[2 * (size_t)HWo] = v.z;
                    if (c + 3 < a.cout) o[3 * (size_t)HWo] = v.w;
                    c += 4 * CPL;
                    y += 4 * CPL;
                    o += 4 * CPL * (size_t)HWo;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (a.k_splits > 1 && a.counters)
        splitk_fixup<64 * WM * WN>(a, t, m_lo, min(BM, m_end - m_lo), tn * BN, BN, (int *)st2);
    if (a.pf) {
        // the next conv's weights into L2 and the memory-side cache: the
        // workgroups share them out in 1 KB wave loads into a stage buffer
        // no longer read (after every wave's epilogue)
        __builtin_amdgcn_s_barrier();
        const uint64_t stride = (uint64_t)gridDim.x * gridDim.y * NW * 1024u;
        for (uint64_t off = (((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * NW + wave) * 1024u + lane * 16u;
             off + 16u <= a.pf_bytes; off += stride)
            __builtin_amdgcn_global_load_lds((const void *)((const char *)a.pf + off),
                                             (lds_u8 *)(st0 + wave * 1024), 16, 0, 0);
        wait_vm<0>();
    }
}

bool conv_dma_supported(const ConvArgs &a) {
    // a row outside the image reads the zero page at its channel offset
    return a.Cin % 32 == 0 && a.in_cs % 8 == 0 && a.K % 32 == 0 && a.k_per_split % 32 == 0 && a.zero &&
           (a.uni_affine || a.grouped) && (long)a.in_cs * 2 + 128 <= GEMEL_ZERO_PAGE_BYTES;
}
bool conv_dma_supported(const ConvArgs &a, int tile) {
    if (!conv_dma_supported(a)) return false;
    if (tile_dma_depth(tile) == 64) return a.Cin % 64 == 0 && a.k_per_split % 64 == 0;
    return true;
}

hipError_t launch_conv_dma(const ConvArgs &a, int tile, const Sink &sk) {
    if (!conv_dma_supported(a, tile) || a.M <= 0 || a.N <= 0 || a.N % 8 || a.nseg < 1 || a.nseg > GEMEL_MAX_SEG)
        return hipErrorInvalidValue;
    if (a.K != a.kh * a.kw * a.Cin || a.out_cs < a.N || a.seg[0].m_start != 0) return hipErrorInvalidValue;
    if (a.k_splits > 1 && !a.partial) return hipErrorInvalidValue;
    // fused 2x2 pool: whole windows, no split-K, no residual
    if (a.out_mode == OUT_NHWC_POOL2 &&
        (a.k_splits > 1 || a.has_res || (a.Ho & 1) || (a.Wo & 1) || a.Ho <= 0 || a.Wo <= 0))
        return hipErrorInvalidValue;
    if (a.k_splits > 1 && (long)a.k_splits * a.M * a.N * 4 > 0x7fffffffL) return hipErrorInvalidValue;
    if ((long)a.k_per_split * a.k_splits < a.K) return hipErrorInvalidValue;
    // bf16 pairs: internal NHWC output, both halves inside the pixel
    if (a.out_pair && (a.out_mode != OUT_NHWC || a.out_pair < a.N || a.out_pair % 8 || a.out_cs < a.out_pair + a.N))
        return hipErrorInvalidValue;
    // mixed sizes: NHWC output, no fused pool; each segment whole frames of
    // its own size, the rows of the segments back to back
    if (a.hetero && a.out_mode != OUT_NHWC) return hipErrorInvalidValue;
    if (a.grouped && a.hetero) return hipErrorInvalidValue;
    for (int i = 0; i < a.nseg; ++i) {
        const ConvSeg &s = a.seg[i];
        if (!s.in || !s.scale || !s.shift) return hipErrorInvalidValue;
        if (a.grouped && (!s.w || (i && s.m_start <= a.seg[i - 1].m_start))) return hipErrorInvalidValue;
        if ((a.k_splits <= 1 || a.counters) && !s.out) return hipErrorInvalidValue;
        if (a.has_res && !s.res) return hipErrorInvalidValue;
        if (!a.hetero) {
            if (s.m_start != s.f_start * a.Ho * a.Wo) return hipErrorInvalidValue;
            continue;
        }
        const long rows = (i + 1 < a.nseg ? a.seg[i + 1].m_start : a.M) - (long)s.m_start;
        if (s.H <= 0 || s.W <= 0 || s.Ho <= 0 || s.Wo <= 0 || rows <= 0 || rows % ((long)s.Ho * s.Wo))
            return hipErrorInvalidValue;
    }
    int bm = conv_tile_bm(tile), bn = conv_tile_bn(tile);
    if (!bm) return hipErrorInvalidValue;
    // the 256 x 256 tile of depth 64 has one workgroup on a CU: 224 rows
    // where that fills the CUs' last turn better (49 * 2^k rows, the usual
    // batches of 224-pixel frames, are 196 tiles of 256 rows on 256 CUs, or
    // 224 of 224 rows: M 50176, N 256, K 2304 takes 58-61 us instead of
    // 63-66 us, K 1152 38.5 instead of 44 us, 1.0 and 0.77 PFLOP/s); not with
    // segments of several map sizes, whose row walk leaves that tile no
    // registers
    const int mode = a.out_mode == OUT_NHWC_POOL2 ? 1 : a.hetero ? 2 : 0;
    bool rows224 = false;
    // (its weights are addressed with 32-bit byte offsets)
    if (tile == TILE_DMA64_256x256 && (long)a.N * a.K * 2 > 0xffffffffL) tile = TILE_DMA_256x256;
    if (tile == TILE_DMA64_256x256 && !a.grouped && !a.hetero && a.k_splits == 1) {
        auto turns = [&](long rows) { return ((a.M + rows - 1) / rows * ((a.N + 255) / 256) + 255) / 256 * rows; };
        rows224 = turns(224) < turns(256);
    }
    if (rows224) bm = 224;
    // grouped: each segment tiled on its own, from tile seg[s].t_start
    ConvArgs b = a;
    long tiles = 0;
    if (a.grouped) {
        for (int i = 0; i < a.nseg; ++i) {
            const long rows = (i + 1 < a.nseg ? a.seg[i + 1].m_start : a.M) - (long)a.seg[i].m_start;
            b.seg[i].t_start = (int32_t)tiles;
            tiles += (rows + bm - 1) / bm * ((a.N + bn - 1) / bn);
        }
    } else {
        tiles = (long)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn);
    }
    if (tiles != conv_tiles(a, bm, bn)) return hipErrorInvalidValue;
    const long blocks = tiles >= 8 ? (tiles + 7) / 8 * 8 : tiles;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    // magic numbers of the row decomposition (exact for rows below 2^31:
    // m = floor(2^32 (2^l - d) / d) + 1 with l = ceil(log2 d))
    {
        const bool pool = a.out_mode == OUT_NHWC_POOL2;
        const long d[2] = {pool ? (long)(a.Ho / 2) * (a.Wo / 2) : (long)a.Ho * a.Wo, pool ? a.Wo / 2 : a.Wo};
        for (int q = 0; q < 2; ++q) {
            if (d[q] <= 0) {
                b.dv_m[q] = 1;
                b.dv_l[q] = 0;
                continue;
            }
            int l = 0;
            while ((1L << l) < d[q]) ++l;
            b.dv_m[q] = (uint32_t)(((uint64_t)1 << 32) * (uint64_t)((1L << l) - d[q]) / (uint64_t)d[q] + 1);
            b.dv_l[q] = l;
        }
    }
    dim3 grid((unsigned)blocks, (unsigned)a.k_splits);
    hipError_t e = hipErrorInvalidValue;
#define GEMEL_DMA_CASE(T, BM_, BN_, WM_, WN_, ST_, BK_, NT_)                                                  \
    case T:                                                                                                   \
        e = submit(sk,                                                                                        \
                   mode == 1   ? reinterpret_cast<const void *>(&conv_dma_kernel<BM_, BN_, WM_, WN_, ST_, BK_, 1>) \
                   : mode == 2 ? reinterpret_cast<const void *>(&conv_dma_kernel<BM_, BN_, WM_, WN_, ST_, BK_, 2>) \
                               : reinterpret_cast<const void *>(&conv_dma_kernel<BM_, BN_, WM_, WN_, ST_, BK_, 0>), \
                   grid, dim3(NT_), b);                                                                       \
        break;
    switch (rows224 ? TILE_COUNT : tile) {
    case TILE_COUNT:
        e = submit(sk,
                   mode == 1 ? reinterpret_cast<const void *>(&conv_dma_kernel<224, 256, 2, 4, 2, 64, 1>)
                             : reinterpret_cast<const void *>(&conv_dma_kernel<224, 256, 2, 4, 2, 64, 0>),
                   grid, dim3(512), b);
        break;
        GEMEL_DMA_CASE(TILE_DMA_256x256, 256, 256, 2, 4, 4, 32, 512)
        GEMEL_DMA_CASE(TILE_DMA_256x128, 256, 128, 2, 2, 4, 32, 256)
        GEMEL_DMA_CASE(TILE_DMA_128x128, 128, 128, 2, 2, 4, 32, 256)
        GEMEL_DMA_CASE(TILE_DMA_128x64, 128, 64, 2, 1, 4, 32, 128)
        GEMEL_DMA_CASE(TILE_DMA_64x64, 64, 64, 2, 2, 4, 32, 256)
        GEMEL_DMA_CASE(TILE_DMA64_64x64, 64, 64, 2, 2, 4, 64, 256)
        GEMEL_DMA_CASE(TILE_DMA64_256x256, 256, 256, 2, 4, 2, 64, 512)
        GEMEL_DMA_CASE(TILE_DMA64_256x128, 256, 128, 2, 2, 3, 64, 256)
        GEMEL_DMA_CASE(TILE_DMA64_128x128, 128, 128, 2, 2, 2, 64, 256)
        GEMEL_DMA_CASE(TILE_DMA64_128x64, 128, 64, 2, 1, 3, 64, 128)
        GEMEL_DMA_CASE(TILE_DMA_256x128W8, 256, 128, 4, 2, 4, 32, 512)
        GEMEL_DMA_CASE(TILE_DMA_128x256W8, 128, 256, 2, 4, 4, 32, 512)
        GEMEL_DMA_CASE(TILE_DMA_256x64, 256, 64, 4, 1, 4, 32, 256)
        GEMEL_DMA_CASE(TILE_DMA_64x256, 64, 256, 1, 4, 4, 32, 256)
    default: break;
    }
#undef GEMEL_DMA_CASE
    return e;
}

}  // namespace gemel
