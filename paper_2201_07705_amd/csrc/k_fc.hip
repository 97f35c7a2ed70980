// Fully connected layers for small frame counts (M <= 64 frames).
//
// An FC layer at a few frames is a weight-streaming problem: every weight
// byte is read once and used M times, far below the MFMA ridge point, so
// the kernel is organised for HBM bandwidth. Each wave owns 16 output
// neurons and a slice of K. It streams its 16 weight rows through a ring of
// LDS buffers of its own, by direct global-to-LDS loads of 256 contiguous
// bytes per row, the steps ahead in flight while the oldest is read (no
// barrier in the depth loop: a wave waits for its own loads only), and
// v_mfma_f32_16x16x32_bf16 does the multiply-adds (weights as the 16-row A
// operand, up to 16 frames as the 16-column B operand). K is split over
// blockIdx.y so that enough waves are in flight to saturate HBM; partial
// sums go to a [splits][M][N] fp32 buffer and the last split of each column
// of 64 neurons to finish reduces them and applies bias, activation and the
// store (or, without arrival counters, fc_reduce does). With one split the
// epilogue is applied directly.
//
// Measured against loads into registers inside per-lane bounds checks (which
// the compiler waited for step by step), one layer alone, its weights in the
// memory-side cache, at 1 / 8 / 16 / 64 frames: 25088 -> 4096 (205 MB) 35.0 /
// 42.0 / 51.3 / 207 us before, 32.7 / 33.7 / 44.4 / 177 here; 4096 -> 1000 8.8
// / 11.5 / 14.1 / 31.6 before, 6.5 / 7.6 / 9.0 / 24.4 here; 2048 -> 20 7.2 / 9.1
// / 11.8 / 22.2 before, 5.1 / 5.8 / 7.5 / 15.0 here.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kargs.h"
#include "kernels.h"
#include "splitk.h"

namespace gemel {

typedef unsigned short u16;
typedef __attribute__((address_space(3))) unsigned char fc_lds_u8;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float fc_bf2f(u16 h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ u16 fc_f2bf(float f) { return __builtin_bit_cast(u16, (__bf16)f); }
__device__ __forceinline__ float fc_act(float y, int act, float slope) {
    const float relu = fmaxf(y, 0.f);
    const float leaky = y > 0.f ? y : y * slope;
    return act == 1 ? relu : act == 2 ? leaky : y;
}

// Fields of the segment that holds launch frame f (the last one with f_start
// <= f) by a select walk: the table lives in the argument block, which is
// read with scalar loads; indexing it with a per-lane number makes every
// field a dependent global load.
struct FcRow {
    const void *in;
    void *out;
    const float *scale, *shift;
    int f_start;
};
__device__ __forceinline__ FcRow fc_row(const FcArgs &a, int f) {
    FcRow r{a.seg[0].in, a.seg[0].out, a.seg[0].scale, a.seg[0].shift, 0};
    for (int i = 1; i < a.nseg; ++i) {
        const bool hit = f >= a.seg[i].f_start;
        r.in = hit ? a.seg[i].in : r.in;
        r.out = hit ? a.seg[i].out : r.out;
        r.scale = hit ? a.seg[i].scale : r.scale;
        r.shift = hit ? a.seg[i].shift : r.shift;
        r.f_start = hit ? a.seg[i].f_start : r.f_start;
    }
    return r;
}

__device__ __forceinline__ void fc_store(const FcArgs &a, int f, int n, float acc) {
    const FcRow sg = fc_row(a, f);
    const int lf = f - sg.f_start;
    const float y = fc_act(acc * sg.scale[n] + sg.shift[n], a.act, a.slope);
    if (a.out_mode == OUT_NHWC) {
        ((u16 *)sg.out)[(size_t)lf * a.out_cs + n] = fc_f2bf(y);
    } else if (n < a.cout) {
        ((float *)sg.out)[(size_t)lf * a.cout + n] = y;
    }
}

// vmcnt only: expcnt and lgkmcnt left at their maxima (gfx9 encoding).
template <int N>
__device__ __forceinline__ void fc_wait_vm() {
    static_assert(N >= 0 && N < 16, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(N | (0x7 << 4) | (0xF << 8));
}
__device__ __forceinline__ void fc_wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4)); }

// Depth of a ring step, and the 1 KB loads a wave makes for it (16 rows of
// 256 bytes).
constexpr int FC_KS = 128, FC_WI = 16 * FC_KS * 2 / 1024;

// MB: frame blocks of 16. DEEP: the input slice of 64 KB and four ring
// buffers (one workgroup on a CU); else a slice of 28 KB and three, so that
// two workgroups fit a CU. At 16 frames fc 25088 -> 4096 (16 splits of 1664)
// takes 44.4 us DEEP; 33 splits of 768, whose slices fit the small form, took
// 46.6.
template <int MB, bool DEEP>
__global__ __launch_bounds__(256) void fc_bf16_kernel(const FcArgs a) {
    constexpr int COLS = 64;   // neurons of a workgroup, 16 per wave
    constexpr int NST = DEEP ? 4 : 3;
    __shared__ __attribute__((aligned(1024))) unsigned char r0[4 * FC_WI * 1024], r1[4 * FC_WI * 1024],
        r2[4 * FC_WI * 1024], r3[NST > 3 ? 4 * FC_WI * 1024 : 16];
    __shared__ __attribute__((aligned(16))) u16 xs[DEEP ? FC_X_ELEMS : FC_X_SMALL];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n0 = blockIdx.x * COLS + wave * 16;
    const int k_begin = blockIdx.y * a.k_per_split;
    const int k_end = min(a.K, k_begin + a.k_per_split);
    const int g = lane >> 4, l16 = lane & 15;
    // frames [f0, f1) of this grid slice and their weights: every frame of
    // the launch, or (grouped) segment blockIdx.z alone
    const void *wsrc = a.w;
    int f0 = 0, f1 = a.M;
    if (a.grouped) {
        const int z = blockIdx.z;
        for (int i = 0; i < a.nseg; ++i) {
            wsrc = i == z ? a.seg[i].w : wsrc;
            f0 = i == z ? a.seg[i].f_start : f0;
            f1 = i == z + 1 ? a.seg[i].f_start : f1;
        }
    }
    const int mz = f1 - f0;
    // load i of a step fills slots i * 64 + lane of the wave's buffer: row
    // 4 i + lane / 16, whose 16-byte position lane % 16 holds chunk
    // (lane % 16) ^ row (so that one chunk of 16 rows spans all banks). Rows
    // beyond N read row N - 1 (never stored), chunks beyond k_end the last
    // one of the slice (masked where they are used).
    const u16 *wrow[FC_WI];
    int wch[FC_WI];
#pragma unroll
    for (int i = 0; i < FC_WI; ++i) {
        const int row = 4 * i + g;
        wrow[i] = (const u16 *)wsrc + (size_t)min(n0 + row, a.N - 1) * a.K;
        wch[i] = (l16 ^ row) * 8;
    }
    auto issue = [&](unsigned char *buf, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FC_WI; ++i)
            __builtin_amdgcn_global_load_lds((const void *)(wrow[i] + min(k + wch[i], k_end - 8)),
                                             (fc_lds_u8 *)(buf + (wave * FC_WI + i) * 1024), 16, 0, 0);
    };
    unsigned char *const ring[4] = {r0, r1, r2, r3};
    const int kn = k_end - k_begin;
    const int steps = (kn + FC_KS - 1) / FC_KS;
    // steps past the last one read its chunks again (into a buffer whose
    // reads are over), so that the loop below has no branch around a load
    const int k_last = k_begin + (steps - 1) * FC_KS;
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) issue(ring[s], min(k_begin + s * FC_KS, k_last));
    // the workgroup's slice of the inputs, [k_begin, k_end) x frames, staged
    // in LDS once: every wave reads it, and from LDS its reads need no wait
    // on a global round trip inside the depth loop. With MP frames staged
    // (M rounded up to a power of two up to 16, else 16 per frame block),
    // chunk c (8 elements) of frame f sits in 16-byte slot c * MP + f, so
    // the frames of a fragment are contiguous (no bank conflicts; lanes of
    // frames beyond MP read a staged frame again, for output columns that
    // are never stored). The slots are filled by direct global-to-LDS loads
    // (each wave instruction writes 64 consecutive slots), all in flight at
    // once; staged frames beyond M repeat frame M - 1.
    const int MP = mz > 16 ? 16 * MB : mz > 8 ? 16 : mz > 4 ? 8 : mz > 2 ? 4 : mz;
    {
        const int slots = (kn / 8) * MP;
        for (int s0 = wave * 64; s0 < slots; s0 += 256) {
            const int sl = min(s0 + lane, slots - 1);
            const int c = sl / MP, f = f0 + min(sl - c * MP, mz - 1);
            const FcRow r = fc_row(a, f);
            __builtin_amdgcn_global_load_lds(
                (const void *)((const u16 *)r.in + (size_t)(f - r.f_start) * a.K + k_begin + c * 8),
                (fc_lds_u8 *)(xs + s0 * 8), 16, 0, 0);
        }
        fc_wait_vm<0>();
    }
    __syncthreads();
    f32x4 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    constexpr int WJ = FC_KS / 32;
    auto step = [&](const unsigned char *buf, int k, bool tail) __attribute__((always_inline)) {
        uint4 wv[WJ];
#pragma unroll
        for (int j = 0; j < WJ; ++j)
            wv[j] = *(const uint4 *)(buf + wave * FC_WI * 1024 + (l16 * 16 + ((j * 4 + g) ^ l16)) * 16);
        uint4 xv[MB][WJ];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int fr = mb * 16 + l16;
            const u16 *xr = xs + (fr < MP ? fr : (fr & (MP - 1))) * 8;
#pragma unroll
            for (int j = 0; j < WJ; ++j)
                xv[mb][j] = *(const uint4 *)(xr + ((min(k + j * 32 + g * 8, k_end - 8) - k_begin) >> 3) * MP * 8);
        }
        if (tail) {
#pragma unroll
            for (int j = 0; j < WJ; ++j)
                if (k + j * 32 + g * 8 >= k_end) {
                    wv[j] = make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) xv[mb][j] = make_uint4(0, 0, 0, 0);
                }
        }
#pragma unroll
        for (int j = 0; j < WJ; ++j)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wv[j]),
                                                                  __builtin_bit_cast(bf16x8, xv[mb][j]), acc[mb], 0, 0, 0);
    };
    if (n0 < a.N) {
        auto turn = [&](int s, int k, bool tail) __attribute__((always_inline)) {
            // step s has landed; the NST - 2 newer ones may fly. The
            // refilled buffer was read in the step before.
            fc_wait_vm<(NST - 2) * FC_WI>();
            fc_wait_lgkm0();
            issue(ring[(s + NST - 1) % NST], min(k + (NST - 1) * FC_KS, k_last));
            __builtin_amdgcn_sched_barrier(0);
            step(ring[s], k, tail);
        };
        // whole turns of the ring first, with no branch between the loads
        // (the compiler's waits then see one path), then the last steps
        const int full = kn / FC_KS;   // whole steps
        int it = 0;
        for (; it + NST <= full; it += NST) {
#pragma unroll
            for (int s = 0; s < NST; ++s) turn(s, k_begin + (it + s) * FC_KS, false);
        }
#pragma unroll
        for (int s = 0; s < NST; ++s)
            if (it + s < steps) turn(s, k_begin + (it + s) * FC_KS, it + s >= full);
        fc_wait_vm<0>();
    }
    // D[neuron = n0 + 4 g + v][frame = mb*16 + lane%16]
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int f = f0 + mb * 16 + l16;
        if (f >= f1) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int n = n0 + g * 4 + v;
            if (n >= a.N) continue;
            if (a.k_splits > 1)
                store_partial1(a.partial + ((size_t)blockIdx.y * a.M + f) * a.N + n, acc[mb][v]);
            else
                fc_store(a, f, n, acc[mb][v]);
        }
    }
    // fused split-K reduction: the last split of this column of neurons
    // sums the partials in split order, as fc_reduce does
    if (a.k_splits > 1 && a.counters) {
        __shared__ int flag;
        if (!splitk_arrive(a.counters + (a.grouped ? blockIdx.z * gridDim.x : 0) + blockIdx.x, a.k_splits, &flag))
            return;
        // two items per thread, eight splits per batch of loads (at clamped
        // addresses: a load inside a branch is waited for at its end)
        const size_t split_elems = (size_t)a.M * a.N;
        for (int i0 = threadIdx.x; i0 < mz * COLS; i0 += 2 * 256) {
            float sum[2] = {0.f, 0.f};
            int f[2], n[2];
            const float *base[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int item = min(i0 + u * 256, mz * COLS - 1);
                f[u] = f0 + item / COLS;
                n[u] = blockIdx.x * COLS + item % COLS;
                base[u] = a.partial + (size_t)f[u] * a.N + min(n[u], a.N - 1);
            }
            for (int sp0 = 0; sp0 < a.k_splits; sp0 += 8) {
                float p[2][8];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        p[u][q] = load_partial1(base[u] + min(sp0 + q, a.k_splits - 1) * split_elems);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int q = 0; q < 8; ++q) sum[u] += sp0 + q < a.k_splits ? p[u][q] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (i0 + u * 256 < mz * COLS && n[u] < a.N) fc_store(a, f[u], n[u], sum[u]);
        }
    }
}

__global__ __launch_bounds__(256) void fc_reduce_kernel(const FcArgs a) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)a.M * a.N) return;
    const int f = (int)(idx / a.N), n = (int)(idx - (long)f * a.N);
    float acc = 0.f;
    for (int s = 0; s < a.k_splits; ++s) acc += a.partial[((size_t)s * a.M + f) * a.N + n];
    fc_store(a, f, n, acc);
}

static bool fc_args_ok(const FcArgs &a) {
    if (a.M <= 0 || a.N <= 0 || a.K <= 0 || a.nseg < 1 || a.nseg > GEMEL_MAX_SEG) return false;
    if (a.N % 8 || a.K % 8 || a.k_splits < 1 || a.k_per_split <= 0) return false;
    if ((long)a.k_splits * a.k_per_split < a.K) return false;
    if (a.out_mode == OUT_NHWC && a.out_cs < a.N) return false;
    if (a.out_mode == OUT_NCHW_F32 && a.cout > a.N) return false;
    if (a.seg[0].f_start != 0) return false;
    for (int i = 0; i < a.nseg; ++i)
        if (!a.seg[i].in || !a.seg[i].out || !a.seg[i].scale || !a.seg[i].shift) return false;
    if (a.k_splits > 1 && !a.partial) return false;
    if (a.grouped)
        for (int i = 0; i < a.nseg; ++i)
            if (!a.seg[i].w || (i > 0 && a.seg[i].f_start <= a.seg[i - 1].f_start)) return false;
    return true;
}

// Frames of the largest grid slice: the whole launch, or (grouped) the
// largest segment.
static int fc_slice_frames(const FcArgs &a) {
    if (!a.grouped) return a.M;
    int m = 0;
    for (int i = 0; i < a.nseg; ++i) m = std::max(m, (i + 1 < a.nseg ? a.seg[i + 1].f_start : a.M) - a.seg[i].f_start);
    return m;
}

hipError_t launch_fc_bf16(const FcArgs &a, const Sink &sk) {
    if (!fc_args_ok(a) || (a.k_splits > 1 && a.k_per_split % 128)) return hipErrorInvalidValue;
    const int ms = fc_slice_frames(a);
    if (ms < 1 || ms > 64) return hipErrorInvalidValue;
    const int64_t slice = fc_slice_elems(ms, std::min(a.K, a.k_per_split));
    if (slice > FC_X_ELEMS) return hipErrorInvalidValue;
    dim3 grid((unsigned)((a.N + 63) / 64), (unsigned)a.k_splits, (unsigned)(a.grouped ? a.nseg : 1)), block(256);
    const int mb = (ms + 15) / 16;
    const void *t[4] = {reinterpret_cast<const void *>(&fc_bf16_kernel<1, true>),
                        reinterpret_cast<const void *>(&fc_bf16_kernel<2, true>),
                        reinterpret_cast<const void *>(&fc_bf16_kernel<3, true>),
                        reinterpret_cast<const void *>(&fc_bf16_kernel<4, true>)};
    const void *fn = mb == 1 && slice <= FC_X_SMALL ? reinterpret_cast<const void *>(&fc_bf16_kernel<1, false>) : t[mb - 1];
    return submit(sk, fn, grid, block, a);
}

hipError_t launch_fc_reduce(const FcArgs &a, const Sink &sk) {
    if (!fc_args_ok(a) || a.k_splits < 2) return hipErrorInvalidValue;
    const long n = (long)a.M * a.N;
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
    return submit(sk, reinterpret_cast<const void *>(&fc_reduce_kernel), grid, block, a);
}

}  // namespace gemel
