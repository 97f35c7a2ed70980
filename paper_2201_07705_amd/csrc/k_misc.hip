// Memory-bound layout, pooling and routing kernels (NHWC, physical channel
// counts multiple of 8). Every thread moves 8 channels (16 bytes of bf16)
// so that loads and stores are full-width and coalesced along C; one launch
// covers all models of a node, blockIdx.y selecting the model's segment.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kargs.h"
#include "kernels.h"

namespace gemel {

typedef unsigned short u16;

__device__ __forceinline__ float m_bf2f(u16 h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ u16 m_f2bf(float f) { return __builtin_bit_cast(u16, (__bf16)f); }

__device__ __forceinline__ void load8(const u16 *p, float *v) {
    const uint4 x = *(const uint4 *)p;
    const u16 *h = (const u16 *)&x;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = m_bf2f(h[j]);
}
__device__ __forceinline__ void load8(const float *p, float *v) {
    const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void store8(u16 *p, const float *v) {
    uint4 x;
    u16 *h = (u16 *)&x;
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = m_f2bf(v[j]);
    *(uint4 *)p = x;
}
__device__ __forceinline__ void store8(float *p, const float *v) {
    *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
    *(float4 *)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
// exact copies (no conversion) of 8 elements
__device__ __forceinline__ void copy8(u16 *d, const u16 *s) { *(uint4 *)d = *(const uint4 *)s; }
__device__ __forceinline__ void copy8(float *d, const float *s) {
    *(float4 *)d = *(const float4 *)s;
    *(float4 *)(d + 4) = *(const float4 *)(s + 4);
}

// This workgroup's number in its segment: x and z of the grid together, as a
// launch holds fewer than 2^32 threads along x (frame_launch).
__device__ __forceinline__ uint32_t wg_number() { return blockIdx.z * gridDim.x + blockIdx.x; }

// Caller frames NCHW f32 -> NHWC, channels zero-padded to Co, for images
// (Co = 8): bound by HBM latency and bytes (12 or 16 read for 16 or 32
// written a pixel), so a thread has the loads of PX pixels in flight, 256
// apart, and every store instruction writes whole lines. CL: the channel
// count, or 8 for any (up to 8, those beyond it read again and dropped). The
// loads are unconditional, at clamped addresses: a load inside a branch is
// waited for at the branch's end.
// Grid: x, z = frames * ceil(hw / (256 * PX)), y = segment.
template <typename T, int PX, int CL>
__global__ __launch_bounds__(256) void pack_image_kernel(const EwArgs a) {
    const EwSeg &sg = a.seg[blockIdx.y];
    const long hw = (long)a.H * a.W;
    const uint32_t wg = wg_number(), per = (uint32_t)((hw + 256 * PX - 1) / (256 * PX));
    const int f = (int)(wg / per);
    const long p0 = (long)(wg - f * per) * 256 * PX + threadIdx.x;
    if (f >= sg.frames) return;
    const float *src = (const float *)sg.in0 + (size_t)f * a.c_logical * hw;
    T *dst = (T *)sg.out + (size_t)f * hw * 8;
    float v[PX][8];
#pragma unroll
    for (int q = 0; q < PX; ++q) {
        const long p = min(p0 + q * 256, hw - 1);
#pragma unroll
        for (int j = 0; j < CL; ++j) v[q][j] = src[(size_t)(CL == 8 ? min(j, a.c_logical - 1) : j) * hw + p];
    }
#pragma unroll
    for (int q = 0; q < PX; ++q) {
        const long p = p0 + q * 256;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[q][j] = j < CL && j < a.c_logical ? v[q][j] : 0.f;
        if (p < hw) store8(dst + (size_t)p * 8, v[q]);
    }
}

// 16-byte chunks of a 64-pixel x 64-channel tile in LDS, the chunk position
// swizzled by the pixel: both one chunk of consecutive pixels and the
// consecutive chunks of one pixel then fall on distinct banks.
template <typename T>
struct TransTile {
    static constexpr int EPC = 16 / (int)sizeof(T);   // elements per chunk
    static constexpr int CH = 64 / EPC;                // chunks per pixel
    static constexpr int CPW = CH / 4;                 // chunks per wave
    static constexpr int RPI = 256 / CH;               // pixels the workgroup covers per row pass
    static __device__ __forceinline__ int slot(int px, int ch) { return px * CH + (ch ^ (px & (CH - 1))); }
    static __device__ __forceinline__ uint4 chunk(const float *v) {
        if constexpr (sizeof(T) == 2) {
            auto two = [&](int j) { return (uint32_t)m_f2bf(v[j]) | ((uint32_t)m_f2bf(v[j + 1]) << 16); };
            return make_uint4(two(0), two(2), two(4), two(6));
        } else {
            return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
        }
    }
    static __device__ __forceinline__ float elem(const uint4 &x, int j) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
        if constexpr (sizeof(T) == 2)
            return __uint_as_float((j & 1) ? (w[j >> 1] & 0xffff0000u) : (w[j >> 1] << 16));
        else
            return __uint_as_float(w[j]);
    }
};

// The same for more than 8 channels: a 64-pixel x 64-channel tile turned in
// LDS. Reads are 256 bytes of one channel plane per wave, 16 in flight per
// thread; writes are 64 channels of a pixel (128 bytes of bf16). One thread
// per pixel walking all channels (the form before) left the chip idle: 8
// frames of 1024 x 14 x 14 took 286 us on 8 workgroups, 4.4 us here; 16
// frames of 256 x 56 x 56 72 us, 14 us here (5.5 TB/s).
// Grid: x, z = frames * ceil(hw / 64) * ceil(Co / 64), y = segment.
template <typename T>
__global__ __launch_bounds__(256) void pack_tile_kernel(const EwArgs a) {
    using TT = TransTile<T>;
    __shared__ uint4 lds[64 * TT::CH];
    const EwSeg &sg = a.seg[blockIdx.y];
    const long hw = (long)a.H * a.W;
    const uint32_t wg = wg_number(), per = (uint32_t)((hw + 63) / 64), cb = (uint32_t)(a.Co + 63) / 64;
    const uint32_t tile = wg / cb;
    const int c0 = (int)(wg - tile * cb) * 64, f = (int)(tile / per);
    const long p0 = (long)(tile - f * per) * 64;
    if (f >= sg.frames) return;   // uniform: before the barrier
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float *src = (const float *)sg.in0 + (size_t)f * a.c_logical * hw + min(p0 + lane, hw - 1);
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = src[(size_t)min(c0 + wave * 16 + j, a.c_logical - 1) * hw];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = c0 + wave * 16 + j < a.c_logical ? v[j] : 0.f;
#pragma unroll
    for (int q = 0; q < TT::CPW; ++q) {
        lds[TT::slot(lane, wave * TT::CPW + q)] = TT::chunk(v + q * TT::EPC);
    }
    __syncthreads();
    const int ch = threadIdx.x % TT::CH;
    if (c0 + ch * TT::EPC >= a.Co) return;
    T *dst = (T *)sg.out + ((size_t)f * hw + p0) * a.Co + c0 + ch * TT::EPC;
#pragma unroll
    for (int q = 0; q < 64 / TT::RPI; ++q) {
        const int px = threadIdx.x / TT::CH + q * TT::RPI;
        if (p0 + px < hw) *(uint4 *)(dst + (size_t)px * a.Co) = lds[TT::slot(px, ch)];
    }
}

// Grid of ceil(items / 256) workgroups per frame (items up to 2^32 - 256):
// this thread's frame and its item of the frame (32-bit divisions, the
// frame's by scalars). False for threads beyond either.
__device__ __forceinline__ bool frame_item(uint32_t items, int frames, uint32_t &f, uint32_t &idx) {
    const uint32_t wg = wg_number(), per = (items + 255) / 256;
    f = wg / per;
    idx = (wg - f * per) * 256 + threadIdx.x;
    return (int)f < frames && idx < items;
}

// Max pool, window k, stride, pad: out-of-range taps are skipped (= -inf).
// K > 0: the window size at compile time; taps beyond the border read the
// nearest pixel of the window instead (its maximum is the same), so that
// all K * K loads are in flight at once (8 frames of 64 x 112 x 112, 3x3
// stride 2: 7.3 -> 5.4 us).
template <typename T, int K>
__global__ __launch_bounds__(256) void maxpool_kernel(const EwArgs a) {
    const EwSeg &sg = a.seg[blockIdx.y];
    const uint32_t ch = (uint32_t)a.C / 8, items = (uint32_t)a.Ho * a.Wo * ch;
    uint32_t f, idx;
    if (!frame_item(items, sg.frames, f, idx)) return;
    const uint32_t px = idx / ch, row = px / (uint32_t)a.Wo;
    const int cc = (int)(idx - px * ch), wo = (int)(px - row * a.Wo), ho = (int)row;
    const T *in = (const T *)sg.in0 + (size_t)f * a.H * a.W * a.C + cc * 8;
    const int h0 = ho * a.stride - a.pad, w0 = wo * a.stride - a.pad;
    float m[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) m[j] = -INFINITY;
    if constexpr (K > 0) {
        const T *p[K];
        size_t wi[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            p[i] = in + (size_t)min(max(h0 + i, 0), a.H - 1) * a.W * a.C;
            wi[i] = (size_t)min(max(w0 + i, 0), a.W - 1) * a.C;
        }
#pragma unroll
        for (int i = 0; i < K; ++i)
#pragma unroll
            for (int q = 0; q < K; ++q) {
                float v[8];
                load8(p[i] + wi[q], v);
#pragma unroll
                for (int j = 0; j < 8; ++j) m[j] = fmaxf(m[j], v[j]);
            }
    } else {
        for (int i = 0; i < a.k; ++i) {
            const int hi = h0 + i;
            if (hi < 0 || hi >= a.H) continue;
            for (int q = 0; q < a.k; ++q) {
                const int wi = w0 + q;
                if (wi < 0 || wi >= a.W) continue;
                float v[8];
                load8(in + ((size_t)hi * a.W + wi) * a.C, v);
#pragma unroll
                for (int j = 0; j < 8; ++j) m[j] = fmaxf(m[j], v[j]);
            }
        }
    }
    store8((T *)sg.out + ((size_t)f * items + idx) * 8, m);
}

// Global average pool: [f][H][W][C] -> [f][C], fp32 sums in one order whatever
// the map's size and the launch: group g of 4 adds pixels g, g + 4, ... one
// after the other, then the groups are added in order. Bound by the latency of
// that chain's loads, so a workgroup takes CW = 4 or 16 8-channel chunks of one
// frame and all its threads load a tile of 512 or 64 pixels into LDS, the next
// tile in flight while a thread per group and channel pair adds (pixels beyond
// the map are zeros: the sums are never -0, so adding 0 leaves them alone).
// 8 frames of 7 x 7 x 2048 bf16 4.3 us, 16 x 16 x 32 float32 4.2, 48 x 48 x 32
// bf16 9.8 (a wave's lanes loading as they add, in the same order: 6.1, 9.7 and
// 146 us; 64 groups of pixels, in another: 4.4, 4.3 and 5.9).
// Grid: x, z = frames * ceil(chunks / CW), y = segment.
template <typename T, int CW>
__global__ __launch_bounds__(256) void avgpool_kernel(const EwArgs a) {
    constexpr int LP = 256 / CW, U = CW > 8 ? 4 : 8, P = LP * U;   // pixels of a load of the workgroup, and of a tile
    constexpr int Q = (int)sizeof(T) / 2;             // 16-byte pieces of a chunk
    constexpr int E = CW > 8 ? 2 : 1;                 // channels a thread adds
    constexpr int AT = CW * 8 / E;                    // such threads per group
    __shared__ uint4 tile[P * CW * Q];
    __shared__ float part[4][CW * 8];
    const EwSeg &sg = a.seg[blockIdx.y];
    const int ch = a.C / 8, cblocks = (ch + CW - 1) / CW;
    const int wg = (int)wg_number(), f = wg / cblocks;
    if (f >= sg.frames) return;   // uniform: before the barriers
    const int t = threadIdx.x;
    const int cl = t % CW, pl = t / CW, c0 = (wg - f * cblocks) * CW;
    const int c = t % AT, g = t / AT;
    const long hw = (long)a.H * a.W;
    const T *in = (const T *)sg.in0 + (size_t)f * hw * a.C + min(c0 + cl, ch - 1) * 8;
    uint4 v[U][Q];
    auto load = [&](long p0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const uint4 *src = (const uint4 *)(in + (size_t)min(p0 + q * LP + pl, hw - 1) * a.C);
#pragma unroll
            for (int i = 0; i < Q; ++i) v[q][i] = src[i];
        }
    };
    float s[E] = {};
    // 16 pixels of this thread's group and channels, from pixel b of the tile
    auto add16 = [&](int b) __attribute__((always_inline)) {
        float x[16][E];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int at = (b + 4 * i + g) * AT + c;
            if constexpr (sizeof(T) == 2 && E == 2) {
                const uint32_t w = ((const uint32_t *)tile)[at];
                x[i][0] = __uint_as_float(w << 16);
                x[i][1] = __uint_as_float(w & 0xffff0000u);
            } else if constexpr (E == 2) {
                const float2 w = ((const float2 *)tile)[at];
                x[i][0] = w.x;
                x[i][1] = w.y;
            } else if constexpr (sizeof(T) == 2) {
                x[i][0] = m_bf2f(((const u16 *)tile)[at]);
            } else {
                x[i][0] = ((const float *)tile)[at];
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int e = 0; e < E; ++e) s[e] += x[i][e];
    };
    load(0);
    for (long p0 = 0; p0 < hw; p0 += P) {
        if (p0) __syncthreads();   // the tile before has been added
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const bool ok = p0 + q * LP + pl < hw;
#pragma unroll
            for (int i = 0; i < Q; ++i)
                tile[((q * LP + pl) * CW + cl) * Q + i] = ok ? v[q][i] : make_uint4(0, 0, 0, 0);
        }
        __syncthreads();
        if (p0 + P < hw) load(p0 + P);
        if (g < 4) {
            if constexpr (P == 64) {
                add16(0);
            } else if (p0 + P <= hw) {
#pragma unroll
                for (int b = 0; b < P; b += 64) add16(b);
            } else {
                for (int b = 0; b < hw - p0; b += 64) add16(b);
            }
        }
    }
    if (g < 4) {
#pragma unroll
        for (int e = 0; e < E; ++e) part[g][c * E + e] = s[e];
    }
    __syncthreads();
    if (t < CW * 8 && c0 * 8 + t < a.C) {
        const float m = (part[0][t] + part[1][t] + part[2][t] + part[3][t]) * (1.0f / (float)hw);
        T *o = (T *)sg.out + (size_t)f * a.C + c0 * 8 + t;
        if constexpr (sizeof(T) == 2)
            *o = m_f2bf(m);
        else
            *o = m;
    }
}

// Nearest-neighbour 2x upsample.
template <typename T>
__global__ __launch_bounds__(256) void upsample2x_kernel(const EwArgs a) {
    const EwSeg &sg = a.seg[blockIdx.y];
    const uint32_t ch = (uint32_t)a.C / 8, items = (uint32_t)a.Ho * a.Wo * ch;
    uint32_t f, idx;
    if (!frame_item(items, sg.frames, f, idx)) return;
    const uint32_t px = idx / ch, ho = px / (uint32_t)a.Wo;
    const uint32_t cc = idx - px * ch, wo = px - ho * a.Wo;
    const T *in = (const T *)sg.in0 + (((size_t)f * a.H + ho / 2) * a.W + wo / 2) * a.C + cc * 8;
    copy8((T *)sg.out + ((size_t)f * items + idx) * 8, in);
}

// Channel concat [in0 (C), in1 (C1)] -> out (C + C1), same H x W.
template <typename T>
__global__ __launch_bounds__(256) void concat_kernel(const EwArgs a) {
    const EwSeg &sg = a.seg[blockIdx.y];
    const uint32_t ch = (uint32_t)a.Co / 8, hw = (uint32_t)a.H * a.W, items = hw * ch;
    uint32_t f, idx;
    if (!frame_item(items, sg.frames, f, idx)) return;
    const uint32_t px = idx / ch;
    const int c = (int)(idx - px * ch) * 8;
    const size_t p = (size_t)f * hw + px;
    const T *src = c < a.C ? (const T *)sg.in0 + p * a.C + c : (const T *)sg.in1 + p * a.C1 + (c - a.C);
    copy8((T *)sg.out + ((size_t)f * items + idx) * 8, src);
}

// Internal NHWC (C physical) -> caller NCHW f32 with c_logical channels: the
// pack tile's transpose the other way round. Reads are 64 channels of a
// pixel, writes 256 bytes of one channel plane per wave (8 x 64 x 56 x 56
// from bf16: 5.0 us; a thread per pixel and 8 channels, reading 16 bytes of
// each line, 6.1 us).
// Grid: x, z = frames * ceil(hw / 64) * ceil(c_logical / 64), y = segment.
template <typename T>
__global__ __launch_bounds__(256) void export_kernel(const EwArgs a) {
    using TT = TransTile<T>;
    __shared__ uint4 lds[64 * TT::CH];
    const EwSeg &sg = a.seg[blockIdx.y];
    const long hw = (long)a.H * a.W;
    const uint32_t wg = wg_number(), per = (uint32_t)((hw + 63) / 64), cb = (uint32_t)(a.c_logical + 63) / 64;
    const uint32_t tile = wg / cb;
    const int c0 = (int)(wg - tile * cb) * 64, f = (int)(tile / per);
    const long p0 = (long)(tile - f * per) * 64;
    if (f >= sg.frames) return;   // uniform: before the barrier
    const int ch = threadIdx.x % TT::CH, px0 = threadIdx.x / TT::CH;
    const T *src = (const T *)sg.in0 + ((size_t)f * hw + p0) * a.C + min(c0 + ch * TT::EPC, a.C - TT::EPC);
    uint4 x[64 / TT::RPI];
#pragma unroll
    for (int q = 0; q < 64 / TT::RPI; ++q) x[q] = *(const uint4 *)(src + (size_t)min((long)(px0 + q * TT::RPI), hw - 1 - p0) * a.C);
#pragma unroll
    for (int q = 0; q < 64 / TT::RPI; ++q) lds[TT::slot(px0 + q * TT::RPI, ch)] = x[q];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (p0 + lane >= hw) return;
    float *o = (float *)sg.out + (size_t)f * a.c_logical * hw + p0 + lane;
#pragma unroll
    for (int q = 0; q < TT::CPW; ++q) {
        const int cq = wave * TT::CPW + q;
        const uint4 v = lds[TT::slot(lane, cq)];
#pragma unroll
        for (int j = 0; j < TT::EPC; ++j) {
            const int c = c0 + cq * TT::EPC + j;
            if (c < a.c_logical) o[(size_t)c * hw] = TT::elem(v, j);
        }
    }
}

// A launcher with nothing to launch (no frames): the sink's timing events,
// if any, are recorded on its stream where the kernel would have run, so
// that they bound an empty interval instead of staying unrecorded.
static hipError_t submit_nothing(const Sink &sk) {
    if (sk.graph) return hipSuccess;
    if (sk.ev_start) {
        const hipError_t e = hipEventRecord(sk.ev_start, sk.stream);
        if (e != hipSuccess) return e;
    }
    return sk.ev_stop ? hipEventRecord(sk.ev_stop, sk.stream) : hipSuccess;
}

static bool ew_ok(const EwArgs &a, bool need_in1) {
    if (a.nseg < 1 || a.nseg > GEMEL_MAX_SEG || a.max_frames < 0) return false;
    for (int i = 0; i < a.nseg; ++i) {
        if (a.seg[i].frames < 0 || a.seg[i].frames > a.max_frames) return false;
        if (!a.seg[i].in0 || !a.seg[i].out || (need_in1 && !a.seg[i].in1)) return false;
    }
    return true;
}

// A grid of `blocks` workgroups per frame in x, one segment in y; more than
// 2^23 of them (2^31 threads) go on in z.
static hipError_t frame_launch(const void *kern, long blocks, const EwArgs &a, const Sink &sk) {
    if (blocks > 0x7fffffffL || blocks * a.max_frames > 0x7fffffffL) return hipErrorInvalidValue;
    const long n = blocks * a.max_frames, x = std::min(n, 1L << 23);
    if (n <= 0) return submit_nothing(sk);
    return submit(sk, kern, dim3((unsigned)x, (unsigned)a.nseg, (unsigned)((n + x - 1) / x)), dim3(256), a);
}
// One thread per item of a frame (frame_item).
static hipError_t item_launch(const void *kern, long items, const EwArgs &a, const Sink &sk) {
    return items > 0xffffff00L ? hipErrorInvalidValue : frame_launch(kern, (items + 255) / 256, a, sk);
}

template <typename T, int PX>
static const void *pack_image_of(int c) {
    return c == 3   ? reinterpret_cast<const void *>(&pack_image_kernel<T, PX, 3>)
           : c == 1 ? reinterpret_cast<const void *>(&pack_image_kernel<T, PX, 1>)
                    : reinterpret_cast<const void *>(&pack_image_kernel<T, PX, 8>);
}

hipError_t launch_pack(const EwArgs &a, bool bf16, const Sink &sk) {
    if (!ew_ok(a, false) || a.Co % 8 || a.c_logical > a.Co || a.c_logical <= 0) return hipErrorInvalidValue;
    const long hw = (long)a.H * a.W;
    if (a.Co == 8) {
        // 4 pixels a thread where that still leaves four workgroups per CU
        const bool wide = (hw + 1023) / 1024 * a.max_frames * a.nseg >= 1024;
        const long px = wide ? 1024 : 256;
        const void *k = bf16 ? (wide ? pack_image_of<u16, 4>(a.c_logical) : pack_image_of<u16, 1>(a.c_logical))
                             : (wide ? pack_image_of<float, 4>(a.c_logical) : pack_image_of<float, 1>(a.c_logical));
        return frame_launch(k, (hw + px - 1) / px, a, sk);
    }
    const void *k = bf16 ? reinterpret_cast<const void *>(&pack_tile_kernel<u16>)
                         : reinterpret_cast<const void *>(&pack_tile_kernel<float>);
    return frame_launch(k, (hw + 63) / 64 * ((a.Co + 63) / 64), a, sk);
}

template <typename T>
static const void *maxpool_of(int k) {
    return k == 2   ? reinterpret_cast<const void *>(&maxpool_kernel<T, 2>)
           : k == 3 ? reinterpret_cast<const void *>(&maxpool_kernel<T, 3>)
                    : reinterpret_cast<const void *>(&maxpool_kernel<T, 0>);
}

hipError_t launch_maxpool(const EwArgs &a, bool bf16, const Sink &sk) {
    // pad < k: every window holds a pixel (what the clamped taps rely on)
    if (!ew_ok(a, false) || a.C % 8 || a.k <= 0 || a.stride <= 0 || a.pad >= a.k) return hipErrorInvalidValue;
    if (a.Ho != (a.H + 2 * a.pad - a.k) / a.stride + 1 || a.Wo != (a.W + 2 * a.pad - a.k) / a.stride + 1)
        return hipErrorInvalidValue;
    return item_launch(bf16 ? maxpool_of<u16>(a.k) : maxpool_of<float>(a.k), (long)a.Ho * a.Wo * (a.C / 8), a, sk);
}

hipError_t launch_avgpool(const EwArgs &a, bool bf16, const Sink &sk) {
    if (!ew_ok(a, false) || a.C % 8 || a.H <= 0 || a.W <= 0) return hipErrorInvalidValue;
    const int cw = a.C / 8 <= 4 ? 4 : 16;
    const void *k = cw == 4 ? (bf16 ? reinterpret_cast<const void *>(&avgpool_kernel<u16, 4>)
                                    : reinterpret_cast<const void *>(&avgpool_kernel<float, 4>))
                            : (bf16 ? reinterpret_cast<const void *>(&avgpool_kernel<u16, 16>)
                                    : reinterpret_cast<const void *>(&avgpool_kernel<float, 16>));
    return frame_launch(k, (a.C / 8 + cw - 1) / cw, a, sk);
}

hipError_t launch_upsample2x(const EwArgs &a, bool bf16, const Sink &sk) {
    if (!ew_ok(a, false) || a.C % 8 || a.Ho != 2 * a.H || a.Wo != 2 * a.W) return hipErrorInvalidValue;
    const void *k = bf16 ? reinterpret_cast<const void *>(&upsample2x_kernel<u16>)
                         : reinterpret_cast<const void *>(&upsample2x_kernel<float>);
    return item_launch(k, (long)a.Ho * a.Wo * (a.C / 8), a, sk);
}

hipError_t launch_concat(const EwArgs &a, bool bf16, const Sink &sk) {
    if (!ew_ok(a, true) || a.C % 8 || a.C1 % 8 || a.Co != a.C + a.C1) return hipErrorInvalidValue;
    const void *k = bf16 ? reinterpret_cast<const void *>(&concat_kernel<u16>)
                         : reinterpret_cast<const void *>(&concat_kernel<float>);
    return item_launch(k, (long)a.H * a.W * (a.Co / 8), a, sk);
}

hipError_t launch_export(const EwArgs &a, bool bf16, const Sink &sk) {
    if (!ew_ok(a, false) || a.C % 8 || a.c_logical > a.C || a.c_logical <= 0) return hipErrorInvalidValue;
    const long hw = (long)a.H * a.W;
    const void *k = bf16 ? reinterpret_cast<const void *>(&export_kernel<u16>)
                         : reinterpret_cast<const void *>(&export_kernel<float>);
    return frame_launch(k, (hw + 63) / 64 * ((a.c_logical + 63) / 64), a, sk);
}

}  // namespace gemel
