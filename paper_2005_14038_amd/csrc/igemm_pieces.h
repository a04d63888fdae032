// Shared by the fp32 contractions on bf16 pieces (igemm_split.hip,
// igemm_planes.hip): the split of a value and the way back to fp32 MFMAs where
// a sum holds a NaN.
#pragma once
#include "igemm_common.h"

namespace hp {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two floats as bf16 (nearest even), the first in the low half
__device__ __forceinline__ unsigned cvt2(float a, float b) {
    const floatx2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// the three pieces of four consecutive elements, 8 bytes each
__device__ __forceinline__ void split4(const float (&x)[4], uint2& h, uint2& m, uint2& l) {
    unsigned p[3][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        float a = x[2 * e], b = x[2 * e + 1];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            p[q][e] = cvt2(a, b);
            a -= __uint_as_float(p[q][e] << 16);             // exact
            b -= __uint_as_float(p[q][e] & 0xFFFF0000u);
        }
    }
    h = make_uint2(p[0][0], p[0][1]);
    m = make_uint2(p[1][0], p[1][1]);
    l = make_uint2(p[2][0], p[2][1]);
}

// One element of the operands at linear reduction index k, zero outside the
// problem or in the padding (plain index arithmetic: recompute only).
template <int OP>
__device__ __forceinline__ float elem_a(const KArgs& args, long row, long k) {
    const ConvGeo& g = args.g;
    if (row >= args.M || k < 0) return 0.f;
    if constexpr (OP == OP_WGRAD) {
        return args.b[k * g.K + row];
    } else {
        const int CC = OP == OP_FWD ? g.C : g.K;
        const int c = (int)(k % CC), rs = (int)(k / CC), r = rs / g.S, s = rs % g.S;
        if constexpr (OP == OP_FWD) {
            const int q = (int)(row % g.Q), p = (int)(row / g.Q % g.P);
            const long n = row / g.Q / g.P;
            const int h = p * g.st - g.pad + r, w = q * g.st - g.pad + s;
            if ((unsigned)h >= (unsigned)g.H || (unsigned)w >= (unsigned)g.W) return 0.f;
            return args.a[((n * g.H + h) * g.W + w) * g.C + c];
        } else {
            const int w = (int)(row % g.W), h = (int)(row / g.W % g.H);
            const long n = row / g.W / g.H;
            const int tp = h + g.pad - r, tq = w + g.pad - s;
            if (tp < 0 || tq < 0 || tp % g.st || tq % g.st) return 0.f;
            const int p = tp / g.st, q = tq / g.st;
            if (p >= g.P || q >= g.Q) return 0.f;
            return args.a[((n * g.P + p) * g.Q + q) * g.K + c];
        }
    }
}

template <int OP>
__device__ __forceinline__ float elem_b(const KArgs& args, long col, long k) {
    const ConvGeo& g = args.g;
    if (col >= args.Ncols || k < 0) return 0.f;
    if constexpr (OP == OP_FWD) {
        return args.b[col * args.Kred + k];
    } else if constexpr (OP == OP_DGRAD) {
        const long kc = k % g.K, rs = k / g.K;
        return args.b[(kc * g.R * g.S + rs) * g.C + col];
    } else {
        if ((args.epi & EPI_BIASCOL) && col == args.Ncols - 1) return 1.f;
        const int c = (int)(col % g.C), rs = (int)(col / g.C), r = rs / g.S, s = rs % g.S;
        const int q = (int)(k % g.Q), p = (int)(k / g.Q % g.P);
        const long n = k / g.Q / g.P;
        const int h = p * g.st - g.pad + r, w = q * g.st - g.pad + s;
        if ((unsigned)h >= (unsigned)g.H || (unsigned)w >= (unsigned)g.W) return 0.f;
        return args.a[((n * g.H + h) * g.W + w) * g.C + c];
    }
}

// acc += low, the block's sum (SCALED: (acc + low low_scale) 2^ex); NaN in it (an infinite or NaN operand, or a sum
// past the largest float): computed again with fp32 MFMAs.  The reduction runs
// over the work item's tiles of BK, tap-inner where the caller's does.
template <int OP, int BK, int TM, int TN, bool SCALED = false>
__device__ __forceinline__ void sum_or_recompute(const KArgs& args, const Work& wk,
                                                 floatx16 (&acc)[TM][TN],
                                                 const floatx16 (&low)[TM][TN], bool tap_inner,
                                                 int wm, int wn, int lane,
                                                 float low_scale = 1.f, int ex = 0) {
    const ConvGeo& g = args.g;
    const int lr = lane & 31, lk = lane >> 5;
    const int tbeg = (int)(wk.kbeg / BK);
    const int ktiles = (int)((wk.kend - wk.kbeg + BK - 1) / BK);
    const int CCH = (OP == OP_FWD) ? g.C : g.K;
    const int RSN = g.R * g.S;
    float chk = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (SCALED)
                    acc[i][j][v] = ldexpf(fmaf(low[i][j][v], low_scale, acc[i][j][v]), ex);
                else
                    acc[i][j][v] += low[i][j][v];
                chk += acc[i][j][v];
            }
    if (!__any(chk != chk)) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
#pragma unroll 1
    for (int e = 0; e < ktiles * BK; e += 2) {
        const int T = tbeg + e / BK;
        long k;
        if (tap_inner) {
            k = (long)(T % RSN) * CCH + (T / RSN) * BK + e % BK + lk;
        } else {
            k = wk.kbeg + e + lk;
            if (k >= wk.kend) k = -1;
        }
        float av[TM], bv[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) av[i] = elem_a<OP>(args, wk.m0 + wm + 32 * i + lr, k);
#pragma unroll
        for (int j = 0; j < TN; ++j) bv[j] = elem_b<OP>(args, wk.n0 + wn + 32 * j + lr, k);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] =
                    __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
}

}  // namespace

}  // namespace hp
