// fp32 contractions on the bf16 matrix cores (gfx950): every fp32 operand is
// split into three bf16 pieces, x = h + m + l, as it is staged into LDS, and a
// product x y is the sum of the six piece products of at least 2^-18 of it:
//
//   h h' + (h m' + m h') + (m m' + h l' + l h')
//
// Three round-to-nearest pieces hold all 24 bits of an fp32 value; the three
// products left out (m l', l m', l l') are below 2^-25 of x y.  A bf16 MFMA
// multiplies 16 times as fast as an fp32 one, so six of them take 6/16 of the
// time.  The piece products are exact in fp32; what rounds is the addition to
// the accumulator, once per MFMA.  h h' has an accumulator of its own and the
// five small products share a second one, whose rounding is 2^-8 of the first
// one's: the sum then rounds once per 16 products (an fp32 MFMA chain rounds
// once per product or two).  Against 64 bits, 512 x 512 outputs, relu(normal)
// x normal operands, K = 576 / 2304 / 25088: 1.05e-7 / 2.3e-7 / 9.3e-7, fp32
// MFMAs 3.1e-7 / 6.1e-7 / 2.0e-6; one accumulator for all six 3.5e-7 / 7.0e-7 /
// 2.4e-6 (its low products are rounded down).
//
// Below 2^-110 the low pieces run into bf16's smallest exponent; an infinite
// operand splits into NaN pieces.  A wave whose block holds a NaN computes it
// again with fp32 MFMAs (recompute), so infinities and NaN come out as there.
#include "igemm_pieces.h"

namespace hp {

namespace {

constexpr int SBK = 16;                       // k tile

// Workgroup tile BM x BN, wave tile WM x WN.  LDS holds, per stage and
// operand, the h, m and l planes of a k tile: an operand whose reduction index
// is contiguous in memory as rows of 16 k (two 16-byte chunks, exchanged in
// every other group of 8 rows so that 16 lanes' reads cover the 64 banks), the
// others as rows of BM (BN) elements padded by 32, read with transpose reads
// (see igemm_h16w_kernel).  The loads of tile kt+2 are issued while tile kt is
// multiplied, the registers of tile kt+1 split and written to the other stage.
//
// FAST: a forward or stride-1 data-gradient contraction whose reduction
// channel count (C, or K) is a multiple of the k tile, with the tap-inner
// order and the unit stride fixed at compile time: no k tile crosses a tap,
// so the per-thread wrap of the channel index, the linear-order paths and the
// stride's division and exact-tap test drop out of the k loop (the data
// gradient's stride alone: VGG-19 +1.1 %, its first stage +1.3 %).  The tap
// index steps by selects and (r, s) follow from it by a multiply and shift,
// exact for at most 7 x 7 taps (the host's condition).  For a
// weight gradient: an output width Q that is a multiple of the k tile, so that
// no k tile (16 output pixels) crosses an output row and the pixel's image
// and row are the tile's.
template <int OP, int BM, int BN, int WM, int WN, bool FAST>
__global__ void __launch_bounds__(64 * (BM / WM) * (BN / WN), 2) igemm_split_kernel(KArgs args) {
    constexpr int BK = SBK;
    constexpr int NT = 64 * (BM / WM) * (BN / WN);
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr bool A_KMAJ = (OP != OP_WGRAD);
    constexpr bool B_KMAJ = (OP == OP_FWD);
    constexpr int PA = BM + 32, PB = BN + 32;             // m-major row pitch (elements)
    constexpr int PLA = (A_KMAJ ? BM * BK : BK * PA) * 2;  // plane sizes (bytes)
    constexpr int PLB = (B_KMAJ ? BN * BK : BK * PB) * 2;
    constexpr int STAGE = 3 * (PLA + PLB);
    constexpr int WAVES_N = BN / WN;
    constexpr int AV = BM * BK / 4 / NT, BV = BN * BK / 4 / NT;
    static_assert(AV >= 1 && BV >= 1 && (BM * BK / 4) % NT == 0 && (BN * BK / 4) % NT == 0,
                  "tile shape");
    constexpr int KVPR = BK / 4, AVPR = BM / 4, BVPR = BN / 4;
    static_assert(NT % AVPR == 0 && NT % BVPR == 0 && NT % KVPR == 0, "one column per thread");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];

    const ConvGeo& g = args.g;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = (wave / WAVES_N) * WM;
    const int wn = (wave % WAVES_N) * WN;

    const Work wk = decode_work<BM, BN>(args);
    const long m0 = wk.m0, n0 = wk.n0, kbeg = wk.kbeg, kend = wk.kend;
    const int ktiles = (int)((kend - kbeg + BK - 1) / BK);
    const int CCH = (OP == OP_FWD) ? g.C : g.K;
    const int RSN = g.R * g.S;
    const bool tap_inner = (OP != OP_WGRAD) && (FAST || ((CCH % BK == 0) && RSN > 1));
    const int tbeg = (int)(kbeg / BK), tend = (int)((kend + BK - 1) / BK);

    // ---- per-thread staging coordinates (as in igemm_kernel) ----
    int arow_base[AV], arow_h[AV], arow_w[AV];
    bool arow_ok[AV];
    int akv = 0;
    if constexpr (A_KMAJ) {
        akv = (t % KVPR) * 4;
#pragma unroll
        for (int i = 0; i < AV; ++i) {
            const long m = m0 + (t + i * NT) / KVPR;
            arow_ok[i] = m < args.M;
            const long mm = arow_ok[i] ? m : 0;
            if constexpr (OP == OP_FWD) {
                const int q = (int)(mm % g.Q); const long tt = mm / g.Q;
                const int p = (int)(tt % g.P); const int n = (int)(tt / g.P);
                arow_base[i] = n * g.H * g.W * g.C;
                arow_h[i] = p * g.st - g.pad;
                arow_w[i] = q * g.st - g.pad;
                if (FAST && !arow_ok[i]) arow_h[i] = -g.H - g.R;   // no tap in the image
            } else {
                const int w = (int)(mm % g.W); const long tt = mm / g.W;
                const int h = (int)(tt % g.H); const int n = (int)(tt / g.H);
                arow_base[i] = n * g.P * g.Q * g.K;
                arow_h[i] = h + g.pad;
                arow_w[i] = w + g.pad;
                if (FAST && !arow_ok[i]) arow_h[i] = -g.P - g.R;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < AV; ++i) {
            const long m = m0 + (t % AVPR) * 4;
            arow_ok[i] = m < args.M;
            arow_base[i] = (int)m;
            arow_h[i] = arow_w[i] = 0;
        }
    }
    int bcol_r = 0, bcol_s = 0, bcol_c = 0, bkv = 0;
    bool bcol_ok = true, bcol_ones = false;
    int brow_n[BV];
    bool brow_ok[BV];
    if constexpr (B_KMAJ) {
        bkv = (t % KVPR) * 4;
#pragma unroll
        for (int i = 0; i < BV; ++i) {
            const long n = n0 + (t + i * NT) / KVPR;
            brow_ok[i] = n < args.Ncols;
            brow_n[i] = brow_ok[i] ? (int)(n * args.Kred) : 0;
        }
    } else {
        const long col = n0 + (t % BVPR) * 4;
        bcol_ok = col < args.Ncols;
        if (OP == OP_WGRAD && (args.epi & EPI_BIASCOL) && col == args.Ncols - 1) {
            bcol_ones = true;      // the appended column of ones (bias gradient)
            bcol_ok = false;
        }
        const int cc = bcol_ok ? (int)col : 0;
        if constexpr (OP == OP_WGRAD) {
            bcol_c = cc % g.C;
            const int tt = cc / g.C;
            bcol_s = tt % g.S;
            bcol_r = tt / g.S;
        } else {
            bcol_c = cc;
        }
#pragma unroll
        for (int i = 0; i < BV; ++i) { brow_n[i] = 0; brow_ok[i] = true; }
    }
    // data gradient: tap (r, s) of channel c0 + kr is at a uniform base plus
    // this thread's constant when a k tile lies within one tap
    const int rsc = g.R * g.S * g.C;
    const bool dg_one_tap = (OP == OP_DGRAD) && (FAST || g.K % BK == 0);
    int b_thr[BV];
#pragma unroll
    for (int i = 0; i < BV; ++i) b_thr[i] = ((t + i * NT) / BVPR) * rsc + bcol_c;

    const long x_el = (long)g.N * g.H * g.W * g.C, dy_el = (long)g.N * g.P * g.Q * g.K;
    const long a_el = (OP == OP_DGRAD) ? dy_el : x_el;
    const long b_el = (OP == OP_WGRAD) ? dy_el : (long)g.K * g.R * g.S * g.C;
    const __amdgpu_buffer_rsrc_t rsa = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(args.a), (short)0, (int)(a_el * 4), BUF_CFG);
    const __amdgpu_buffer_rsrc_t rsb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(args.b), (short)0, (int)(b_el * 4), BUF_CFG);
    float areg[AV][4], breg[BV][4];
    bool bone[BV];
    auto ldb = [](__amdgpu_buffer_rsrc_t rs, bool ok, int off, float (&v)[4])
        __attribute__((always_inline)) {
        const uintx4 q = buf_load16(rs, ok ? (unsigned)off * 4u : BUF_OOB, 0u);
        v[0] = __uint_as_float(q[0]); v[1] = __uint_as_float(q[1]);
        v[2] = __uint_as_float(q[2]); v[3] = __uint_as_float(q[3]);
    };

    // uniform decomposition of the next tile to load, stepped tile by tile
    int nr = 0, ns = 0, nc = 0, ntap = 0, nq = 0, np = 0, nn = 0;
    const int magS = (256 + g.S - 1) / g.S;   // (t * magS) >> 8 = t / S for t < R*S <= 49
    if constexpr (OP == OP_FWD || OP == OP_DGRAD) {
        if (tap_inner) {
            ntap = tbeg % RSN;
            nc = (tbeg / RSN) * BK;
        } else {
            ntap = (int)kbeg / CCH;
            nc = (int)kbeg - ntap * CCH;
        }
        nr = ntap / g.S;
        ns = ntap - nr * g.S;
    } else {
        nq = (int)kbeg % g.Q;
        const int t0 = (int)kbeg / g.Q;
        np = t0 % g.P;
        nn = t0 / g.P;
    }

    auto gload = [&](int kt) __attribute__((always_inline)) {
        const int T = tbeg + kt;
        // FAST: the loads of tiles past the end read in-range or range-checked
        // offsets and are never staged
        const bool tin = FAST || T < tend;
        const int k0 = tap_inner ? (tin ? ntap * CCH + nc : 0) : (int)(kbeg + (long)kt * BK);
        const int kend_i = tap_inner ? (tin ? k0 + BK : 0) : (int)kend;
        if constexpr (OP == OP_FWD || OP == OP_DGRAD) {
            const int c0 = nc, r0 = nr, s0 = ns;
            if constexpr (FAST) {
                ntap = (ntap + 1 == RSN) ? 0 : ntap + 1;
                nc = (ntap == 0) ? nc + BK : nc;
                nr = (ntap * magS) >> 8;
                ns = ntap - nr * g.S;
            } else if (tap_inner) {
                ++ntap;
                if (++ns == g.S) {
                    ns = 0;
                    if (++nr == g.R) { nr = 0; ntap = 0; nc += BK; }
                }
            } else {
                nc += BK;
                while (nc >= CCH) { nc -= CCH; if (++ns == g.S) { ns = 0; ++nr; } }
            }
            int c = c0 + akv, r = r0, sx = s0;
            if constexpr (!FAST)
                while (c >= CCH) { c -= CCH; if (++sx == g.S) { sx = 0; ++r; } }
            const bool kin = FAST ? tin : k0 + akv < kend_i;
#pragma unroll
            for (int i = 0; i < AV; ++i) {
                if constexpr (OP == OP_FWD) {
                    const int h = arow_h[i] + r, w = arow_w[i] + sx;
                    const bool ok = (FAST || arow_ok[i]) && kin && (unsigned)h < (unsigned)g.H &&
                                    (unsigned)w < (unsigned)g.W;
                    ldb(rsa, ok, arow_base[i] + (h * g.W + w) * g.C + c, areg[i]);
                } else {
                    const int tp = arow_h[i] - r, tq = arow_w[i] - sx;
                    int p = tp, q = tq;
                    bool ok;
                    if constexpr (FAST) {
                        ok = kin && (unsigned)p < (unsigned)g.P && (unsigned)q < (unsigned)g.Q;
                    } else {
                        bool on_grid = true;
                        if (g.st != 1) {
                            p = tp / g.st;
                            q = tq / g.st;
                            on_grid = p * g.st == tp && q * g.st == tq;
                        }
                        ok = arow_ok[i] && kin && tp >= 0 && tq >= 0 && on_grid && p < g.P &&
                             q < g.Q;
                    }
                    ldb(rsa, ok, arow_base[i] + (p * g.Q + q) * g.K + c, areg[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < BV; ++i) {
                if constexpr (OP == OP_FWD) {
                    const int kk = k0 + bkv;
                    ldb(rsb, brow_ok[i] && kk < kend_i, brow_n[i] + kk, breg[i]);
                } else {
                    const int kr = (t + i * NT) / BVPR;
                    int off;
                    if (dg_one_tap) {
                        off = c0 * rsc + (r0 * g.S + s0) * g.C + b_thr[i];
                    } else {
                        int k = c0 + kr, r2 = r0, s2 = s0;
                        while (k >= CCH) { k -= CCH; if (++s2 == g.S) { s2 = 0; ++r2; } }
                        off = ((k * g.R + r2) * g.S + s2) * g.C + bcol_c;
                    }
                    ldb(rsb, bcol_ok && k0 + kr < kend_i, off, breg[i]);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < AV; ++i) {
                const int kk = k0 + (t + i * NT) / AVPR;
                ldb(rsb, arow_ok[i] && (FAST || kk < kend_i), kk * g.K + arow_base[i], areg[i]);
            }
            const bool px1 = !FAST && g.P * g.Q == 1;
            const int q0 = nq, p0 = np, n0i = nn;
            if constexpr (FAST) {
                nq += BK;
                if (nq == g.Q) { nq = 0; if (++np == g.P) { np = 0; ++nn; } }
            } else if (px1) {
                nn += BK;
            } else {
                nq += BK;
                while (nq >= g.Q) { nq -= g.Q; if (++np == g.P) { np = 0; ++nn; } }
            }
#pragma unroll
            for (int i = 0; i < BV; ++i) {
                const int kr = (t + i * NT) / BVPR;
                int q = q0 + kr, p = p0, n = n0i;
                if constexpr (!FAST) {
                    if (px1) {
                        q = 0;
                        n = n0i + kr;
                    } else {
                        while (q >= g.Q) { q -= g.Q; if (++p == g.P) { p = 0; ++n; } }
                    }
                }
                const bool kin = FAST || k0 + kr < kend_i;
                const int h = p * g.st - g.pad + bcol_r, w = q * g.st - g.pad + bcol_s;
                const bool ok = bcol_ok && kin && (unsigned)h < (unsigned)g.H &&
                                (unsigned)w < (unsigned)g.W;
                ldb(rsa, ok, ((n * g.H + h) * g.W + w) * g.C + bcol_c, breg[i]);
                bone[i] = bcol_ones && kin;
            }
        }
    };

    // this thread's write offsets within a plane
    int a_st[AV], b_st[BV];
#pragma unroll
    for (int i = 0; i < AV; ++i) {
        if constexpr (A_KMAJ) {
            const int row = (t + i * NT) / KVPR, kq = t % KVPR;
            a_st[i] = row * (2 * BK) + (((kq >> 1) ^ ((row >> 3) & 1)) << 4) + ((kq & 1) << 3);
        } else {
            a_st[i] = (((t + i * NT) / AVPR) * PA + (t % AVPR) * 4) * 2;
        }
    }
#pragma unroll
    for (int i = 0; i < BV; ++i) {
        if constexpr (B_KMAJ) {
            const int row = (t + i * NT) / KVPR, kq = t % KVPR;
            b_st[i] = row * (2 * BK) + (((kq >> 1) ^ ((row >> 3) & 1)) << 4) + ((kq & 1) << 3);
        } else {
            b_st[i] = (((t + i * NT) / BVPR) * PB + (t % BVPR) * 4) * 2;
        }
    }
    auto sstore = [&](unsigned char* S) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < AV; ++i) {
            uint2 h, m, l;
            split4(areg[i], h, m, l);
            *reinterpret_cast<uint2*>(S + a_st[i]) = h;
            *reinterpret_cast<uint2*>(S + PLA + a_st[i]) = m;
            *reinterpret_cast<uint2*>(S + 2 * PLA + a_st[i]) = l;
        }
        unsigned char* SB = S + 3 * PLA;
#pragma unroll
        for (int i = 0; i < BV; ++i) {
            if (OP == OP_WGRAD && bone[i]) {      // the rest of its vector was read as zeros
                breg[i][0] = 1.f;
            }
            uint2 h, m, l;
            split4(breg[i], h, m, l);
            *reinterpret_cast<uint2*>(SB + b_st[i]) = h;
            *reinterpret_cast<uint2*>(SB + PLB + b_st[i]) = m;
            *reinterpret_cast<uint2*>(SB + 2 * PLB + b_st[i]) = l;
        }
    };

    floatx16 acc[TM][TN], low[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;

    // operand fragments: lane (lr, lk) holds k = 8 lk .. 8 lk + 7 of row lr
    const int lr = lane & 31, lk = lane >> 5;
    const int gq = lane >> 4, sl = lane & 15;
    const int tr_row = 8 * (gq >> 1) + (sl >> 2);
    const int tr_col = 16 * (gq & 1) + 4 * (sl & 3);
    const int kch = (lk ^ ((lr >> 3) & 1)) << 4;
    const int a_fr = A_KMAJ ? (wm + lr) * (2 * BK) + kch : (tr_row * PA + wm + tr_col) * 2;
    const int b_fr = B_KMAJ ? (wn + lr) * (2 * BK) + kch : (tr_row * PB + wn + tr_col) * 2;
    auto tr_read = [](const unsigned char* p) __attribute__((always_inline)) -> v4s {
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) v4s*)(
                (__attribute__((address_space(3))) unsigned char*)(p)));
    };
    auto frag_a = [&](const unsigned char* S, int i) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (A_KMAJ) {
            return __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const uintx4*>(S + a_fr + 32 * i * (2 * BK)));
        } else {
            const v4s lo = tr_read(S + a_fr + 64 * i), hi = tr_read(S + a_fr + 64 * i + 8 * PA);
            return __builtin_bit_cast(
                bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    };
    auto frag_b = [&](const unsigned char* S, int j) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (B_KMAJ) {
            return __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const uintx4*>(S + b_fr + 32 * j * (2 * BK)));
        } else {
            const v4s lo = tr_read(S + b_fr + 64 * j), hi = tr_read(S + b_fr + 64 * j + 8 * PB);
            return __builtin_bit_cast(
                bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    };
    auto mma = [](const bf16x8 (&a)[TM], const bf16x8 (&b)[TN], floatx16 (&c)[TM][TN])
        __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], c[i][j], 0, 0, 0);
    };

    auto step = [&](int kt, int s) __attribute__((always_inline)) {
        const unsigned char* S = smem + s * STAGE;
        bf16x8 a[3][TM], b[3][TN];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[q][i] = frag_a(S + q * PLA, i);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[q][j] = frag_b(S + 3 * PLA + q * PLB, j);
        }
        if (kt + 1 < ktiles) sstore(smem + (s ^ 1) * STAGE);
        gload(kt + 2);
        __builtin_amdgcn_s_setprio(1);
        mma(a[0], b[0], acc);
        mma(a[0], b[1], low);
        mma(a[1], b[0], low);
        mma(a[1], b[1], low);
        mma(a[0], b[2], low);
        mma(a[2], b[0], low);
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
    };

    gload(0);
    if (ktiles > 0) sstore(smem);
    gload(1);
    __syncthreads();
    int kt = 0;
    for (; kt + 1 < ktiles; kt += 2) {
        step(kt, 0);
        step(kt + 1, 1);
    }
    if (kt < ktiles) step(kt, 0);

    sum_or_recompute<OP, BK, TM, TN>(args, wk, acc, low, tap_inner, wm, wn, lane);

    static_assert(2 * STAGE >= (NT / 64) * SLOT_FLOATS * (int)sizeof(float), "epilogue slots");
    write_tile<BM, BN, TM, TN, true>(args, wk, acc, wm, wn, lane,
                                     reinterpret_cast<float*>(smem) + wave * SLOT_FLOATS,
                                     reinterpret_cast<float*>(smem));
}

template <int OP, int BM, int BN, int WM, int WN>
KernelRef ref(bool fast) {
    const void* fn = fast ? reinterpret_cast<const void*>(&igemm_split_kernel<OP, BM, BN, WM, WN, true>)
                          : reinterpret_cast<const void*>(&igemm_split_kernel<OP, BM, BN, WM, WN, false>);
    return {fn, 64 * (BM / WM) * (BN / WN)};
}

template <int OP>
KernelRef ref_op(int cfg, bool fast) {
    switch (cfg) {
        case 1: return ref<OP, 128, 64, 32, 64>(fast);
        case 2: return ref<OP, 64, 256, 64, 64>(fast);
        case 3: return ref<OP, 64, 128, 32, 64>(fast);
        case 4: return ref<OP, 64, 64, 32, 32>(fast);
        default: return ref<OP, 128, 128, 64, 64>(fast);
    }
}

}  // namespace

KernelRef split_kernel(int op, int cfg, bool fast) {
    if (op == OP_FWD) return ref_op<OP_FWD>(cfg, fast);
    if (op == OP_DGRAD) return ref_op<OP_DGRAD>(cfg, fast);
    return ref_op<OP_WGRAD>(cfg, fast);
}

}  // namespace hp
