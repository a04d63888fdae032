// fp32 convolutions on operands whose f16 pieces lie in memory (gfx950).
//
// igemm_split.hip's six bf16 products per fp32 product run at 1150 TFLOP/s
// (56x56x256, batch 32: 0.61 ms a contraction), which is what a large bf16
// matrix product reaches here (1200): only fewer products are faster.  Two f16
// pieces hold 24 bits as well: h = f16(x), l = f16((x - h) 2^11), x = h + l 2^-11
// to 2^-24 of x, and with three products
//
//   x y = h h' + (h l' + l h') 2^-11
//
// the one left out is below 2^-24 of x y.  What f16 lacks is range: each
// tensor is scaled by the power of two that brings its largest finite magnitude
// to [2^14, 2^15).  h is a normal number down to 2^-29 of that largest value and
// below it the error stays under 2^-50 of it (l's scale keeps it clear of f16's
// smallest numbers).  h h' has an accumulator of its own, the two small products
// share a second one.  An infinite or NaN operand makes l NaN, and a wave whose
// block's sum holds a NaN computes it again with fp32 MFMAs.
//
// Splitting while staging would cost as many vector instructions as the matrix
// cores have clocks, so a pass over each operand writes its planes, in the
// value's own layout, after a pass that finds its largest magnitude (16 bytes
// of traffic per value in all), and the contraction copies 16-byte groups of
// the planes straight into LDS.  Against 64 bits (56x56x256, normal operands):
// MEASURED_ERR
//
// Tile: 256 x 128 outputs, eight waves of 64 x 64 (128 accumulator registers a
// lane, so two waves per SIMD), k tile 32.  Both operands' plane tiles are 48
// KB, two stages of the 160 KB of LDS, one workgroup per CU.  The loads of tile
// kt+1 are issued when tile kt begins and have its 48 MFMAs per SIMD to land.
#include <algorithm>

#include "igemm_pieces.h"

namespace hp {

namespace {

constexpr int PL_BK = 32, PL_WAVES = 8, PL_ROW = 2 * PL_BK;

// this wave's loads into LDS and reads from it are done, and so are all others'
__device__ __forceinline__ void publish() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// the power of two that brings a tensor's largest finite magnitude (its bits)
// into [2^14, 2^15)
__device__ __forceinline__ int scale_exp(unsigned amax) {
    const int e = (int)(amax >> 23) - 127;
    return 14 - (e > -112 ? e : -112);
}

__device__ __forceinline__ float scale_of(unsigned amax) {
    return __uint_as_float((unsigned)(scale_exp(amax) + 127) << 23);
}

// a scaled value's pieces
__device__ __forceinline__ void split2(float x, _Float16& h, _Float16& l) {
    h = (_Float16)x;
    l = (_Float16)((x - (float)h) * 2048.f);              // the difference is exact
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const unsigned short* p, long plane,
                                                            int q, long elems) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(p + q * plane), (short)0,
                                             (int)(elems * 2), BUF_CFG);
}

__device__ __forceinline__ void zero_tiles(floatx16 (&a)[2][2], floatx16 (&b)[2][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) a[i][j][v] = b[i][j][v] = 0.f;
}

// the three piece products of one 16-deep step
__device__ __forceinline__ void mma3(const f16x8 (&a)[2][2], const f16x8 (&b)[2][2],
                                     floatx16 (&acc)[2][2], floatx16 (&low)[2][2]) {
    constexpr int pa[3] = {0, 0, 1}, pb[3] = {0, 1, 0};
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                floatx16& c = q ? low[i][j] : acc[i][j];
                c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[pa[q]][i], b[pb[q]][j], c, 0, 0, 0);
            }
}

// Forward and stride-1 data gradient: both operands have the reduction index
// contiguous (the data gradient reads transposed weights), the channel count is
// a multiple of the k tile, at most 32 taps (the bit masks).  LDS rows are 32 k
// of one plane, four 16-byte chunks exchanged by the row's number / 4 mod 4 so
// that 16 lanes' reads cover the 64 banks.
template <int OP>
__global__ void __launch_bounds__(64 * PL_WAVES, 2) igemm_planes_kernel(KArgs args) {
    static_assert(OP == OP_FWD || OP == OP_DGRAD, "k-major operands");
    constexpr int BM = kCfgs[6].bm, BN = kCfgs[6].bn, BK = PL_BK, ROW = PL_ROW;
    constexpr int LA = BM / 16 / PL_WAVES, LB = BN / 16 / PL_WAVES;
    constexpr int PLA = BM * ROW, PLB = BN * ROW, STAGE = 2 * (PLA + PLB);
    static_assert(LA * 16 * PL_WAVES == BM && LB * 16 * PL_WAVES == BN, "loads per wave");
    static_assert((BM / 64) * (BN / 64) == PL_WAVES, "waves");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];

    const ConvGeo& g = args.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = (wave / (BN / 64)) * 64;
    const int wn = (wave % (BN / 64)) * 64;
    const Work wk = decode_work<BM, BN>(args);
    const int ktiles = (int)((wk.kend - wk.kbeg) / BK);   // whole tiles by construction
    const int T0 = (int)(wk.kbeg / BK);
    const int IH = (OP == OP_FWD) ? g.H : g.P;
    const int IW = (OP == OP_FWD) ? g.W : g.Q;
    const int CC = (OP == OP_FWD) ? g.C : g.K;
    const int RSN = g.R * g.S;
    __amdgpu_buffer_rsrc_t rsA[2], rsB[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        rsA[q] = plane_rsrc(args.a16, args.a16s, q, (long)g.N * IH * IW * CC);
        rsB[q] = plane_rsrc(args.b16, args.b16s, q, args.Ncols * args.Kred);
    }

    // the chunk this lane loads: position lane % 4 of row (.. + lane / 4)
    const int kc = ((lane & 3) ^ ((lane >> 4) & 3)) * 8;
    // A rows: byte offset of the row's pixel at tap (0, 0) and chunk kc, and the
    // taps (bit r*S + s) whose pixel lies outside the image (all for rows past M)
    int a_off[LA];
    unsigned a_out[LA];
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const long m = wk.m0 + (wave * LA + j) * 16 + (lane >> 2);
        const bool row_ok = m < args.M;
        const int mm = row_ok ? (int)m : 0;
        const int OW = (OP == OP_FWD) ? g.Q : g.W, OH = (OP == OP_FWD) ? g.P : g.H;
        const int w = mm % OW, tt = mm / OW, h = tt % OH, n = tt / OH;
        const int h0 = (OP == OP_FWD) ? h * g.st - g.pad : h + g.pad;
        const int w0 = (OP == OP_FWD) ? w * g.st - g.pad : w + g.pad;
        unsigned out = 0;
        for (int r = 0; r < g.R; ++r)
            for (int s = 0; s < g.S; ++s) {
                const int hh = (OP == OP_FWD) ? h0 + r : h0 - r;
                const int ww = (OP == OP_FWD) ? w0 + s : w0 - s;
                if (!row_ok || (unsigned)hh >= (unsigned)IH || (unsigned)ww >= (unsigned)IW)
                    out |= 1u << (r * g.S + s);
            }
        a_out[j] = out;
        a_off[j] = (((n * IH + h0) * IW + w0) * CC + kc) * 2;
    }
    unsigned b_off[LB];
#pragma unroll
    for (int j = 0; j < LB; ++j) {
        const long n = wk.n0 + (wave * LB + j) * 16 + (lane >> 2);
        b_off[j] = n < args.Ncols ? (unsigned)((n * args.Kred + kc) * 2) : BUF_OOB;
    }

    // the next tile to load, in reduction order (chunk T / RS, tap T % RS)
    const int rs0 = T0 % RSN;
    int ic = (T0 / RSN) * BK, ir = rs0 / g.S, is = rs0 - ir * g.S, itap = rs0;
    auto issue = [&](unsigned char* S) __attribute__((always_inline)) {
        const int dr = (OP == OP_FWD) ? ir : -ir;
        const int ds = (OP == OP_FWD) ? is : -is;
        const int sk = ((dr * IW + ds) * CC + ic) * 2;
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            // a tap outside the image sets bit 31: past the end of any plane
            const unsigned vo = ((a_out[j] >> itap) << 31) | (unsigned)(a_off[j] + sk);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                buf_load16_lds(rsA[q], S + q * PLA + (wave * LA + j) * 1024, vo, 0u);
        }
        const unsigned kload = (unsigned)((itap * CC + ic) * 2);
#pragma unroll
        for (int j = 0; j < LB; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                buf_load16_lds(rsB[q], S + 2 * PLA + q * PLB + (wave * LB + j) * 1024, b_off[j],
                               kload);
        ++itap;
        if (++is == g.S) {
            is = 0;
            if (++ir == g.R) { ir = 0; itap = 0; ic += BK; }
        }
    };

    floatx16 acc[2][2], low[2][2];
    zero_tiles(acc, low);
    const int lr = lane & 31, lk = lane >> 5;
    const int rsw = (lr >> 2) & 3;       // chunk exchange of this lane's operand rows
    auto lds16 = [](const unsigned char* p) __attribute__((always_inline)) {
        return __builtin_bit_cast(f16x8, *reinterpret_cast<const uintx4*>(p));
    };
    auto compute = [&](const unsigned char* S) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ch = ((2 * h + lk) ^ rsw) * 16;
            const unsigned char* A = S + (wm + lr) * ROW + ch;
            const unsigned char* B = S + 2 * PLA + (wn + lr) * ROW + ch;
            f16x8 a[2][2], b[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[q][i] = lds16(A + q * PLA + 32 * i * ROW);
                    b[q][i] = lds16(B + q * PLB + 32 * i * ROW);
                }
            mma3(a, b, acc, low);
        }
    };

    if (ktiles > 0) issue(smem);
    for (int kt = 0, at = 0; kt < ktiles; ++kt, at ^= 1) {
        publish();
        if (kt + 1 < ktiles) issue(smem + (at ^ 1) * STAGE);
        compute(smem + at * STAGE);
    }
    __syncthreads();
    sum_or_recompute<OP, BK, 2, 2, true>(args, wk, acc, low, true, wm, wn, lane, 1.f / 2048.f,
                                         -scale_exp(*args.amax_a) - scale_exp(*args.amax_b));
    static_assert(2 * STAGE >= PL_WAVES * SLOT_FLOATS * (int)sizeof(float), "epilogue slots");
    write_tile_plain<BM, BN, 2, 2, true>(args, wk, acc, wm, wn, lane,
                                         reinterpret_cast<float*>(smem) + wave * SLOT_FLOATS);
}

// Weight gradient: the reduction index (the output pixel) is the memory row of
// both operands, read from LDS with transpose reads (see igemm_h16w_kernel).
// A stage holds, per plane, blocks of 32 pixels x 128 columns; a wave loads four
// rows of each with one instruction, so a lane has one pixel per k tile.  A
// row's 64-byte quarters are exchanged by its number mod 4: the four rows that
// 32 lanes of a transpose read take lie in disjoint quarters of the banks.
template <int BM, int BN>
__global__ void __launch_bounds__(64 * PL_WAVES, 2) igemm_planes_w_kernel(KArgs args) {
    constexpr int BK = PL_BK, SUB = BK * 256;             // bytes of a 128-column block
    constexpr int NA = BM / 128, NB = BN / 128;
    constexpr int PLA = NA * SUB, PLB = NB * SUB, STAGE = 2 * (PLA + PLB);
    static_assert((BM / 64) * (BN / 64) == PL_WAVES && BK == 4 * PL_WAVES, "waves");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];

    const ConvGeo& g = args.g;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = (wave / (BN / 64)) * 64;
    const int wn = (wave % (BN / 64)) * 64;
    const Work wk = decode_work<BM, BN>(args);
    const int ktiles = (int)((wk.kend - wk.kbeg + BK - 1) / BK);
    const int kend = (int)wk.kend;
    __amdgpu_buffer_rsrc_t rsD[2], rsX[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        rsX[q] = plane_rsrc(args.a16, args.a16s, q, (long)g.N * g.H * g.W * g.C);
        rsD[q] = plane_rsrc(args.b16, args.b16s, q, (long)g.N * g.P * g.Q * g.K);
    }
    const int row = 4 * wave + (lane >> 4);
    const int col = ((lane & 15) ^ ((lane >> 4) << 2)) * 8;
    bool a_ok[NA], b_ok[NB];
    int bc[NB], br[NB], bs[NB];
#pragma unroll
    for (int a = 0; a < NA; ++a) a_ok[a] = wk.m0 + 128 * a + col < args.M;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const long j = wk.n0 + 128 * b + col;             // one tap (C % 8 == 0)
        b_ok[b] = j < args.Ncols;
        const int jj = b_ok[b] ? (int)j : 0;
        bc[b] = jj % g.C;
        const int rs = jj / g.C;
        br[b] = rs / g.S - g.pad;
        bs[b] = rs % g.S - g.pad;
    }
    int pix = (int)wk.kbeg + row;                         // of the next tile to load
    auto issue = [&](unsigned char* S) __attribute__((always_inline)) {
        const bool in = pix < kend;
        const unsigned u = (unsigned)pix;
        const unsigned t2 = (unsigned)(((unsigned long long)u * args.mq) >> args.sq);
        const int q0 = (int)(u - t2 * (unsigned)g.Q) * g.st;
        const unsigned n = (unsigned)(((unsigned long long)t2 * args.mp) >> args.sp);
        const int p0 = (int)(t2 - n * (unsigned)g.P) * g.st;
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            const unsigned vo =
                in && a_ok[a] ? (unsigned)(pix * g.K + (int)wk.m0 + 128 * a + col) * 2u : BUF_OOB;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                buf_load16_lds(rsD[q], S + q * PLA + a * SUB + wave * 1024, vo, 0u);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int h = p0 + br[b], w = q0 + bs[b];
            const bool ok = in && b_ok[b] && (unsigned)h < (unsigned)g.H &&
                            (unsigned)w < (unsigned)g.W;
            const unsigned vo =
                ok ? (unsigned)((((int)n * g.H + h) * g.W + w) * g.C + bc[b]) * 2u : BUF_OOB;
#pragma unroll
            for (int q = 0; q < 2; ++q)
                buf_load16_lds(rsX[q], S + 2 * PLA + q * PLB + b * SUB + wave * 1024, vo, 0u);
        }
        pix += BK;
    };

    floatx16 acc[2][2], low[2][2];
    zero_tiles(acc, low);
    const int gq = lane >> 4, sl = lane & 15;
    const int rr = sl >> 2;                               // k row mod 4
    const int tr = (8 * (gq >> 1) + rr) * 256 + (2 * (gq & 1) + ((sl & 3) >> 1)) * 16 + (sl & 1) * 8;
    int oa[2], ob[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        oa[i] = (wm >> 7) * SUB + tr + (((((wm & 127) >> 5) + i) ^ rr) << 6);
        ob[i] = 2 * PLA + (wn >> 7) * SUB + tr + (((((wn & 127) >> 5) + i) ^ rr) << 6);
    }
    auto frag = [](const unsigned char* p) __attribute__((always_inline)) -> f16x8 {
        auto rd = [](const unsigned char* r) __attribute__((always_inline)) -> v4s {
            return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) v4s*)(
                    (__attribute__((address_space(3))) unsigned char*)(r)));
        };
        const v4s lo = rd(p), hi = rd(p + 4 * 256);
        return __builtin_bit_cast(f16x8,
                                  __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto compute = [&](const unsigned char* S) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f16x8 a[2][2], b[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[q][i] = frag(S + q * PLA + oa[i] + h * 16 * 256);
                    b[q][i] = frag(S + q * PLB + ob[i] + h * 16 * 256);
                }
            mma3(a, b, acc, low);
        }
    };

    if (ktiles > 0) issue(smem);
    for (int kt = 0, at = 0; kt < ktiles; ++kt, at ^= 1) {
        publish();
        if (kt + 1 < ktiles) issue(smem + (at ^ 1) * STAGE);
        compute(smem + at * STAGE);
    }
    __syncthreads();
    sum_or_recompute<OP_WGRAD, BK, 2, 2, true>(
        args, wk, acc, low, false, wm, wn, lane, 1.f / 2048.f,
        -scale_exp(*args.amax_a) - scale_exp(*args.amax_b));
    write_tile_plain<BM, BN, 2, 2, true>(args, wk, acc, wm, wn, lane,
                                         reinterpret_cast<float*>(smem) + wave * SLOT_FLOATS);
}

// The magnitude of a finite value as bits that order as integers; 0 for others.
__device__ __forceinline__ unsigned finite_bits(float x) {
    const unsigned u = __float_as_uint(x) & 0x7FFFFFFFu;
    return u < 0x7F800000u ? u : 0u;
}

__device__ __forceinline__ void block_max(unsigned m, unsigned* out) {
    __shared__ unsigned part[4];
#pragma unroll
    for (int o = 32; o; o >>= 1) {
        const unsigned v = __shfl_xor(m, o);
        m = m > v ? m : v;
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 1; i < 4; ++i) m = m > part[i] ? m : part[i];
        atomicMax(out, m);
    }
}

__global__ void __launch_bounds__(256) clear_kernel(unsigned* p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Both bound by memory: 4 bytes per value, then 8.
__global__ void __launch_bounds__(256) amax_kernel(const float* __restrict__ src, size_t n, int vec,
                                                   unsigned* out) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t n4 = vec ? n / 4 : 0;
    unsigned m = 0;
    for (size_t i = t; i < n4; i += stride) {
        const float4 v = reinterpret_cast<const float4*>(src)[i];
        m = max(max(m, max(finite_bits(v.x), finite_bits(v.y))),
                max(finite_bits(v.z), finite_bits(v.w)));
    }
    for (size_t i = 4 * n4 + t; i < n; i += stride) m = max(m, finite_bits(src[i]));
    block_max(m, out);
}

__global__ void __launch_bounds__(256) split_planes_kernel(const float* __restrict__ src,
                                                           _Float16* __restrict__ dst, size_t n,
                                                           int vec, const unsigned* amax) {
    typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
    const float sc = scale_of(*amax);
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t n4 = vec ? n / 4 : 0;
    for (size_t i = t; i < n4; i += stride) {
        const float4 v = reinterpret_cast<const float4*>(src)[i];
        const float x[4] = {v.x, v.y, v.z, v.w};
        f16x4 h, l;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            _Float16 a, b;
            split2(x[e] * sc, a, b);
            h[e] = a;
            l[e] = b;
        }
        *reinterpret_cast<f16x4*>(dst + 4 * i) = h;
        *reinterpret_cast<f16x4*>(dst + n + 4 * i) = l;
    }
    for (size_t i = 4 * n4 + t; i < n; i += stride) split2(src[i] * sc, dst[i], dst[n + i]);
}

// AMAX: the layers' largest magnitudes into amax[layer]; else the planes.
template <bool AMAX>
__global__ void __launch_bounds__(256) weights_kernel(const float* __restrict__ src,
                                                      _Float16* __restrict__ dst,
                                                      _Float16* __restrict__ dst_t, long plane,
                                                      const WpLayer* __restrict__ table,
                                                      int nlayers, unsigned* amax) {
    const int b = blockIdx.x;
    int at = 0;
    while (at + 1 < nlayers && table[at + 1].tile0 <= b) ++at;
    const WpLayer L = table[at];
    const int tkn = (L.K + WT_TILE - 1) / WT_TILE, tcn = (L.C + WT_TILE - 1) / WT_TILE;
    int tl = b - L.tile0;
    const int c0 = (tl % tcn) * WT_TILE;
    tl /= tcn;
    const int k0 = (tl % tkn) * WT_TILE;
    const int rs = tl / tkn;
    if constexpr (AMAX) {
        unsigned m = 0;
        for (int e = threadIdx.x; e < WT_TILE * WT_TILE; e += 256) {
            const int k = k0 + e / WT_TILE, c = c0 + e % WT_TILE;
            if (k < L.K && c < L.C)
                m = max(m, finite_bits(src[L.off + ((long)k * L.RS + rs) * L.C + c]));
        }
        block_max(m, amax + at);
    } else {
        __shared__ _Float16 tile[2][WT_TILE][WT_TILE + 2];
        const float sc = scale_of(amax[at]);
        for (int e = threadIdx.x; e < WT_TILE * WT_TILE; e += 256) {
            const int kk = e / WT_TILE, cc = e % WT_TILE;
            const int k = k0 + kk, c = c0 + cc;
            if (k >= L.K || c >= L.C) continue;
            const long i = ((long)k * L.RS + rs) * L.C + c;
            split2(src[L.off + i] * sc, tile[0][kk][cc], tile[1][kk][cc]);
            dst[L.dst + i] = tile[0][kk][cc];
            dst[plane + L.dst + i] = tile[1][kk][cc];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < WT_TILE * WT_TILE; e += 256) {
            const int cc = e / WT_TILE, kk = e % WT_TILE;
            const int k = k0 + kk, c = c0 + cc;
            if (k >= L.K || c >= L.C) continue;
            const long i = L.dst + ((long)c * L.RS + rs) * L.K + k;
            dst_t[i] = tile[0][kk][cc];
            dst_t[plane + i] = tile[1][kk][cc];
        }
    }
}

}  // namespace

KernelRef planes_kernel(int op, int cfg) {
    const void* fn;
    if (op == OP_FWD) fn = reinterpret_cast<const void*>(&igemm_planes_kernel<OP_FWD>);
    else if (op == OP_DGRAD) fn = reinterpret_cast<const void*>(&igemm_planes_kernel<OP_DGRAD>);
    else if (cfg == 7) fn = reinterpret_cast<const void*>(&igemm_planes_w_kernel<128, 256>);
    else fn = reinterpret_cast<const void*>(&igemm_planes_w_kernel<256, 128>);
    return {fn, 64 * PL_WAVES};
}

hipError_t launch_clear(unsigned* p, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(clear_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_split_planes(const float* src, uint16_t* dst, size_t n, unsigned* amax,
                               hipStream_t s) {
    if (n == 0) return hipSuccess;
    const int vec = (n & 3) == 0 && ((((uintptr_t)src) & 15) | (((uintptr_t)dst) & 7)) == 0;
    const size_t items = (vec ? n / 4 : n) / 256 + 1;
    const dim3 few((unsigned)std::min<size_t>(items, 2048)),
        many((unsigned)std::min<size_t>(items, 16384));
    hipLaunchKernelGGL(amax_kernel, few, dim3(256), 0, s, src, n, vec, amax);
    hipLaunchKernelGGL(split_planes_kernel, many, dim3(256), 0, s, src,
                       reinterpret_cast<_Float16*>(dst), n, vec, amax);
    return hipGetLastError();
}

hipError_t launch_split_weights(const float* src, uint16_t* dst, uint16_t* dst_t, long plane,
                                const WpLayer* table, int nlayers, int tiles, unsigned* amax,
                                hipStream_t s) {
    if (nlayers <= 0 || tiles <= 0) return hipSuccess;
    _Float16* d = reinterpret_cast<_Float16*>(dst);
    _Float16* dt = reinterpret_cast<_Float16*>(dst_t);
    hipLaunchKernelGGL(weights_kernel<true>, dim3(tiles), dim3(256), 0, s, src, d, dt, plane,
                       table, nlayers, amax);
    hipLaunchKernelGGL(weights_kernel<false>, dim3(tiles), dim3(256), 0, s, src, d, dt, plane,
                       table, nlayers, amax);
    return hipGetLastError();
}

}  // namespace hp
