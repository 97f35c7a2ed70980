// float32 convolution (and FC, as a 1x1 conv on a 1x1 map) on the fp32
// matrix cores: C[M][N] = A[M][K] * W[N][K]^T with v_mfma_f32_16x16x4_f32,
// fp32 operands and accumulation throughout.
//
// The fp32 MFMA is slow enough (32 cycles for 16x16x4) that operands need no
// LDS tiles: a wave's 32 x 32 tile takes 4 16-byte loads per lane for 16
// MFMAs, about half of what the L2 can feed a CU. A load gives 4 adjacent
// lanes 64 contiguous bytes of one row (a load in the MFMA's own layout, 16
// rows on 16 adjacent lanes, costs the address unit 64 separate accesses and
// ran the kernel at 40 TFLOP/s), and lane permutes then move each lane's 4
// depths to the MFMA's row l % 16, depth group l / 16: MFMA e of a 16-deep
// chunk multiplies the depths {e, 4 + e, 8 + e, 12 + e} of both operands (any
// order of the depths is a correct sum as long as both sides use it). Waves
// share nothing in the depth loop; the loads of one or two chunks are in
// flight per wave.
//
// float32 rounds are small (a few frames), so what bounds them is the number
// of waves and the serial depth of each. A workgroup therefore splits the
// depth over KW waves of the same tile and adds their accumulators in LDS;
// the launcher takes the smallest KW from 4 on that gives the chip two waves
// per SIMD. The order of the sums does not follow KW, which depends on the
// launch's rows: the depth is cut into up to 16 parts by K alone
// (f32_parts_log2), each summed on its own, and the parts are added in pairs,
// pairs of pairs and so on, inside a wave (the sums that wait in LDS) and then
// over the waves. A frame's results are the same bits in a round of any size,
// alone or merged with other models.
//
// One thread per output element with a serial fma chain (the form before)
// ran two ResNet-18 at 2 x 2 frames in 20.5 ms, 0.7 TFLOP/s; this form in 0.38
// ms, 45-50 TFLOP/s on the 3x3 convs of 0.9 GFLOP (the address unit and the
// permutes, not the MFMAs, are then the busiest).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "conv_epi.h"
#include "kargs.h"
#include "kernels.h"

namespace gemel {

// Parts of the depth: a power of two up to 16, each of at least two 32-deep
// chunks where there is more than one.
__host__ __device__ inline int f32_parts_log2(int K) {
    const int chunks = (K + 31) / 32;
    int lg = 0;
    while (lg < 4 && chunks >= 4 << lg) ++lg;
    return lg;
}

// FM x FN fragments of 16 pixels x 16 channels per wave; KW waves along the
// depth, MW pixel tiles per workgroup. KW is the number of parts, or 4 or 8 of
// up to 16.
template <int FM, int FN, int KW, int MW>
__global__ __launch_bounds__(64 * KW *MW, FM *FN == 4 ? 4 : 5) void conv_f32_mfma_kernel(const ConvArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // waves w, w + 4, ... share a SIMD: theirs are adjacent stretches of the
    // depth, so that a remainder of chunks falls on all SIMDs alike (36 chunks
    // over 16 waves: 8.3 us otherwise, 7.6 so)
    const int ks = KW >= 8 ? (wave & 3) * (KW / 4) + (wave >> 2) : wave / MW, mw = wave % MW;
    const int slot = ks * MW + mw;
    const int g = lane >> 4, l16 = lane & 15;
    const int tiles_n = (a.N + 16 * FN - 1) / (16 * FN);
    // consecutive tiles (the same pixels, other channels) on one XCD
    const int G = gridDim.x;
    const int t = (G & 7) == 0 ? (int)(blockIdx.x & 7) * (G >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int tm = t / tiles_n, tn = t - tm * tiles_n;
    const int m0 = (tm * MW + mw) * 16 * FM, n0 = tn * 16 * FN;
    if (m0 >= a.M && KW == 1) return;
    const int HWo = a.Ho * a.Wo;
    // part i of 1 << lg holds chunks [i * chunks >> lg, (i + 1) * chunks >> lg);
    // this wave takes `parts` of them from part0 on
    const int chunks = (a.K + 31) / 32, lg = f32_parts_log2(a.K);
    const int parts = (1 << lg) / KW, part0 = ks * parts;
    const int c0 = part0 * chunks >> lg, c1 = (part0 + parts) * chunks >> lg;
    const int k_end = min(a.K, c1 * 32);
    const float *const zp = (const float *)a.zero;

    // this lane loads depths 4 * (lane % 4) .. + 3 of row lane / 4 of each
    // fragment. Pixels (rows beyond M read zeros and are never stored)
    const float *xbase[FM];
    int hi0[FM], wi0[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int gm = m0 + 16 * i + (lane >> 2);
        xbase[i] = zp;
        hi0[i] = -(1 << 28);
        wi0[i] = 0;
        if (gm < a.M) {
            const RowSeg sg = row_seg(a, gm);
            const int lr = gm - sg.m_start;
            const int fr = lr / HWo, pix = lr - fr * HWo, ho = pix / a.Wo;
            xbase[i] = (const float *)sg.in + (size_t)fr * a.H * a.W * a.in_cs;
            hi0[i] = ho * a.stride - a.pad;
            wi0[i] = (pix - ho * a.Wo) * a.stride - a.pad;
        }
    }
    // weight rows (rows beyond N read row 0: their columns are never stored)
    const float *wrow[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int n = n0 + 16 * j + (lane >> 2);
        wrow[j] = (const float *)a.w + (size_t)(n < a.N ? n : 0) * a.K;
    }
    // this lane's next 4 depths: k, and its tap (r, s) and channel c. Cin and
    // K are multiples of 8 and k of 4, so the 4 depths are of one tap.
    int k = c0 * 32 + (lane & 3) * 4, c, r, s;
    {
        const int rs = k / a.Cin;
        c = k - rs * a.Cin;
        r = rs / a.kw;
        s = rs - r * a.kw;
    }
    f32x4 xv[2][FM][2], wv[2][FN][2];
    auto load = [&](int q) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool in = k < k_end;
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const int hi = hi0[i] + r, wi = wi0[i] + s;
                const bool ok = in && (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W;
                xv[q][i][h] = *(const f32x4 *)(ok ? xbase[i] + (size_t)(hi * a.W + wi) * a.in_cs + c : zp);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) wv[q][j][h] = *(const f32x4 *)(in ? wrow[j] + k : zp);
            k += 16;
            c += 16;
            while (c >= a.Cin) {
                c -= a.Cin;
                if (++s == a.kw) {
                    s = 0;
                    ++r;
                }
            }
        }
    };
    // the MFMA's lane (g, l16) takes what lane 4 * l16 + g loaded
    const int from = (4 * l16 + g) * 4;
    auto perm = [&](const f32x4 &v) __attribute__((always_inline)) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(v[e])));
        return o;
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mfmas = [&](int q) __attribute__((always_inline)) {
        f32x4 x[FM][2], w[FN][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < FN; ++j) w[j][h] = perm(wv[q][j][h]);
#pragma unroll
            for (int i = 0; i < FM; ++i) x[i][h] = perm(xv[q][i][h]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(w[j][e >> 2][e & 3], x[i][e >> 2][e & 3], acc[i][j], 0, 0, 0);
    };
    // a part ends with chunk cc: sums of 1 and 2 parts wait in this wave's LDS
    // slots (in registers they cost a wave per SIMD) and are joined like the
    // digits of a binary counter. The last part's sum stays in acc.
    constexpr int LEVELS = KW == 4 ? 2 : KW == 8 ? 1 : 0;
    __shared__ f32x4 lds[KW > 1 ? KW * MW : 1][LEVELS > 1 ? LEVELS : 1][KW > 1 ? FM * FN : 1][64];
    int part = 0, next = (part0 + 1) * chunks >> lg;
    auto fold = [&](int cc) __attribute__((always_inline)) {
        if constexpr (LEVELS > 0) {
            if (cc + 1 != next) return;
            auto join = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[i][j] = lds[slot][b][i * FN + j][lane] + acc[i][j];
            };
            auto keep = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) lds[slot][b][i * FN + j][lane] = acc[i][j];
            };
            if (part & 1) join(0);
            if (LEVELS > 1 && (part & 3) == 3) join(1);
            if (++part == parts) return;
            if (part & 1)
                keep(0);
            else
                keep(LEVELS - 1);
            next = (part0 + part + 1) * chunks >> lg;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // two chunks per iteration with no branch around a load (the compiler's
    // waits then leave the newer chunk's loads in flight), the last ones apart:
    // loads past a wave's depth would take address cycles from the others
    load(0);
    load(1);
    int cc = c0;
    for (; cc + 3 < c1; cc += 2) {
        mfmas(0);
        load(0);
        fold(cc);
        mfmas(1);
        load(1);
        fold(cc + 1);
    }
    if (cc < c1) {
        mfmas(0);
        if (cc + 2 < c1) load(0);
        fold(cc);
    }
    if (cc + 1 < c1) {
        mfmas(1);
        fold(cc + 1);
    }
    if (cc + 2 < c1) {
        mfmas(0);
        fold(cc + 2);
    }

    // ---- epilogue: lane (g, l16) of fragment (i, j) holds channels
    // n0 + 16 j + 4 g .. + 3 of pixel m0 + 16 i + l16 ----
    auto finish = [&](int gm, int n, f32x4 v) __attribute__((always_inline)) {
        if (gm >= a.M || n >= a.N) return;
        const RowSeg sg = row_seg(a, gm);
        const int lr = gm - sg.m_start;
        const f32x4 sc = *(const f32x4 *)(sg.scale + n), sh = *(const f32x4 *)(sg.shift + n);
        f32x4 rv = {0.f, 0.f, 0.f, 0.f};
        if (a.has_res) rv = *(const f32x4 *)((const float *)sg.res + (size_t)lr * a.out_cs + n);
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = epi(v[e] * sc[e] + sh[e], rv[e], a.has_res, a.res_mode, a.act, a.slope);
        if (a.out_mode == OUT_NHWC) {
            *(f32x4 *)((float *)sg.out + (size_t)lr * a.out_cs + n) = y;
        } else {
            const int f = lr / HWo, pix = lr - f * HWo;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < a.cout) ((float *)sg.out)[((size_t)f * a.cout + n + e) * HWo + pix] = y[e];
        }
    };
    if constexpr (KW == 1) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) finish(m0 + 16 * i + l16, n0 + 16 * j + 4 * g, acc[i][j]);
    } else {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) lds[slot][0][i * FN + j][lane] = acc[i][j];
        __syncthreads();
        constexpr int ITEMS = MW * FM * FN * 64;
        for (int it = threadIdx.x; it < ITEMS; it += 64 * KW * MW) {
            const int ln = it & 63, f = (it >> 6) % (FM * FN), mt = (it >> 6) / (FM * FN);
            f32x4 v[KW];
#pragma unroll
            for (int q = 0; q < KW; ++q) v[q] = lds[q * MW + mt][0][f][ln];
#pragma unroll
            for (int w = 1; w < KW; w *= 2)
#pragma unroll
                for (int q = 0; q < KW; q += 2 * w) v[q] += v[q + w];
            finish((tm * MW + mt) * 16 * FM + 16 * (f / FN) + (ln & 15), n0 + 16 * (f % FN) + 4 * (ln >> 4), v[0]);
        }
    }
}

template <int FM, int FN>
static hipError_t launch_f32(const ConvArgs &a, const Sink &sk) {
    const long tm = (a.M + 16 * FM - 1) / (16 * FM), tn = (a.N + 16 * FN - 1) / (16 * FN);
    // every part its own wave up to 4 (12 frames of 56 x 56 x 64 through two 3x3
    // convs each of 2 blocks: 188 us with 4 waves, 207 with 1 and 2); beyond
    // that as many as give each of the 1024 SIMDs two waves
    const int parts = 1 << f32_parts_log2(a.K);
    int kw = std::min(parts, 4);
    while (kw < parts && tm * tn * kw < 2048) kw *= 2;
    const int mw = kw == 1 ? 4 : kw == 2 ? 2 : 1;
    const long tiles = (tm + mw - 1) / mw * tn, blocks = tiles >= 8 ? (tiles + 7) / 8 * 8 : tiles;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    const void *fn = kw == 1   ? reinterpret_cast<const void *>(&conv_f32_mfma_kernel<FM, FN, 1, 4>)
                     : kw == 2 ? reinterpret_cast<const void *>(&conv_f32_mfma_kernel<FM, FN, 2, 2>)
                     : kw == 4 ? reinterpret_cast<const void *>(&conv_f32_mfma_kernel<FM, FN, 4, 1>)
                     : kw == 8 ? reinterpret_cast<const void *>(&conv_f32_mfma_kernel<FM, FN, 8, 1>)
                               : nullptr;
    // (2 x 2 fragments come in 256 tiles or more: at most 8 waves)
    if constexpr (FM * FN < 4) {
        if (kw == 16) fn = reinterpret_cast<const void *>(&conv_f32_mfma_kernel<FM, FN, 16, 1>);
    }
    if (!fn) return hipErrorInvalidValue;
    return submit(sk, fn, dim3((unsigned)blocks), dim3(64 * kw * mw), a);
}

// Fragments per wave: 2 x 2 (operand bytes per MFMA fall with both); one
// row of pixels where 2 x 2 gives fewer workgroups than CUs (or there are no
// more than 16 pixels), one row of channels where there are no more than 16.
hipError_t launch_conv_f32_mfma(const ConvArgs &a, const Sink &sk) {
    const long wgs = (long)((a.M + 31) / 32) * ((a.N + 31) / 32);
    if (a.N <= 16 && a.M > 16) return launch_f32<2, 1>(a, sk);
    return a.M <= 16 || wgs < 256 ? launch_f32<1, 2>(a, sk) : launch_f32<2, 2>(a, sk);
}

}  // namespace gemel
