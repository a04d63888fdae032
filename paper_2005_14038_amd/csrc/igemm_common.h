// Shared by the contraction kernels' sources (igemm.hip, igemm_split.hip):
// tile configurations, kernel arguments, work assignment and epilogues.
#pragma once
#include <type_traits>

#include "kernels.h"

namespace hp {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

namespace {

// LDS row padding (floats).  Operands staged from k-major rows are written
// transposed, one float per store: a row length of 2 mod 32 spreads a wave's
// stores over distinct banks.  Operands staged as whole float4 rows need a
// row length that keeps 16-byte alignment.
constexpr int PAD_T = 2;
constexpr int PAD_V = 4;

// Tile configurations: workgroup tile BM x BN, reduction tile BK of the
// kernels that stage from fp32 and BKH of the kernels on bf16 operands in
// memory, wave tile WM x WN (a grid of (WM/32) x (WN/32) MFMA 32x32 tiles per
// wave); the workgroup has (BM/WM) * (BN/WN) waves.  BKH = 64 halves the
// barriers per MFMA; the 128x64 tile keeps 32, where the second register set
// of a 64-wide k tile would cost it occupancy.
struct TileCfg { int bm, bn, bk, wm, wn, bkh; };
// Waves of 32x64 (eight in the general tile, four in the 128x64 and 64x128
// ones) hide the staging latency better than fewer waves of 64x64, at the
// cost of more LDS reads per MFMA.
constexpr TileCfg kCfgs[] = {
    {128, 128, 16, 32, 64, 64},    // 0: general (8 waves)
    {128, 64, 16, 32, 64, 32},     // 1: narrow N (at most 64 output columns, 4 waves)
    {64, 256, 16, 64, 64, 32},     // 2: narrow M, N a multiple of 256 or large
    {64, 128, 16, 32, 64, 64},     // 3: narrow M otherwise (4 waves)
    {64, 64, 16, 32, 32, 64},      // 4: small M and N (4 waves of 32x32)
    {256, 128, 16, 128, 64, 32},   // 5: igemm_h16d_kernel (4 waves)
    {256, 128, 32, 64, 64, 32},    // 6: the plane kernels (igemm_planes.hip, 8 waves)
    {128, 256, 32, 64, 64, 32},    // 7: their weight gradient with 128 output rows (8 waves)
};

struct KArgs {
    ConvGeo g;
    const float* a;
    const float* b;
    float* out;
    const float* bias;
    const float* mask;
    float* bias_out;
    long M, Ncols, Kred;
    int tiles_m, tiles_n;
    int tfull;        // tiles computed whole, one per workgroup (the first tfull ids)
    int splits;       // every remaining tile is cut into `splits` reduction chunks
    int kchunk;       // reduction length of a chunk (multiple of the K tile)
    float* ws;        // partial tiles of the cut tiles: [tile - tfull][split][BM * BN]
    float* stats;     // optional column statistics per row tile (see Epilogue)
    int epi;
    const unsigned short* a16;   // bf16 copies of a and b (16-bit operand kernel only)
    const unsigned short* b16;
    // plane kernels: elements from one plane of a16 / b16 to the next, and the
    // largest magnitudes their scales follow from
    long a16s, b16s;
    const unsigned* amax_a;
    const unsigned* amax_b;
    // optional: every final output element is also written here rounded to
    // bf16 (nearest even), row-major like out (no bias-gradient column)
    unsigned short* out16;
    // weight gradient on bf16 operands: floor(i / Q) = (i * mq) >> sq and
    // floor(i / P) = (i * mp) >> sp for 0 <= i < 2^31
    unsigned mq, mp;
    int sq, sp;
};

// Destination of output element (row, col): the bias-gradient column of a
// weight gradient goes to bias_out[row]; everything else is row-major with
// the weight part's row length.
__device__ __forceinline__ float* out_ptr(float* out, float* bias_out, long row, long col,
                                          long Ncols, int epi) {
    if (epi & EPI_BIASCOL) {
        if (col == Ncols - 1) return bias_out + row;
        return out + row * (Ncols - 1) + col;
    }
    return out + row * Ncols + col;
}

__device__ __forceinline__ float epilogue(float v, long row, long col, long Ncols, int epi,
                                          const float* bias, const float* mask, const float* prev) {
    if (epi & EPI_BIAS) v += bias[col];
    if (epi & EPI_RELU) v = fmaxf(v, 0.f);
    if ((epi & EPI_MASK) && !(mask[row * Ncols + col] > 0.f)) v = 0.f;
    if (epi & EPI_ACCUM) v += *prev;
    return v;
}

__device__ __forceinline__ float round_bf16(float x) {
    unsigned u = __float_as_uint(x);
    u = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
    return __uint_as_float(u);
}

// Two floats rounded to bf16, packed low element first (LDS byte order).
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
    return (__float_as_uint(round_bf16(lo)) >> 16) | (__float_as_uint(round_bf16(hi)) & 0xFFFF0000u);
}

__device__ __forceinline__ unsigned short bf16_bits(float x) {
    return (unsigned short)(__float_as_uint(round_bf16(x)) >> 16);
}

// Work assignment.  The first `tfull` workgroups each compute one whole
// output tile (whole rounds of the resident workgroups); the rest cut each
// remaining tile's reduction into `splits` chunks, so that the last round is
// as full as the others, and leave partial tiles for the reduce kernels.
// XCD-aware: consecutive workgroup ids are dealt round-robin to the 8 XCDs;
// each XCD gets a contiguous run of whole tiles (n fastest), so tiles sharing
// A rows share that XCD's L2, and likewise a contiguous run of cut-tile items
// (chunk, tile), so tiles reducing over the same chunk share it.
struct Work {
    int tile, z;
    bool partial;
    long m0, n0, kbeg, kend;
};

template <int BM, int BN>
__device__ __forceinline__ Work decode_work(const KArgs& args) {
    Work w;
    int bid = blockIdx.x;
    w.z = 0;
    w.partial = bid >= args.tfull;
    if (!w.partial) {
        if ((args.tfull & 7) == 0) bid = (bid & 7) * (args.tfull >> 3) + (bid >> 3);
        w.tile = bid;
    } else {
        const int r = bid - args.tfull;
        const int ncut = args.tiles_m * args.tiles_n - args.tfull;
        if ((args.tfull & 7) == 0) {
            // the workgroups of one XCD (ids congruent mod 8) take a contiguous
            // run of (chunk, tile) items, tiles fastest: the cut tiles that
            // reduce over the same chunk (same dy rows, same image rows) share
            // that XCD's L2
            const int nparts = ncut * args.splits;
            const int x = r & 7, q = nparts >> 3, rem = nparts & 7;
            const int item = x * q + min(x, rem) + (r >> 3);
            w.z = item / ncut;
            w.tile = args.tfull + (item - w.z * ncut);
        } else {
            w.tile = args.tfull + r / args.splits;
            w.z = r - (w.tile - args.tfull) * args.splits;
        }
    }
    w.m0 = (long)(w.tile / args.tiles_n) * BM;
    w.n0 = (long)(w.tile % args.tiles_n) * BN;
    w.kbeg = w.partial ? (long)w.z * args.kchunk : 0;
    w.kend = w.partial ? min(w.kbeg + (long)args.kchunk, args.Kred) : args.Kred;
    return w;
}

// Writes a wave's accumulators: acc[i][j][v] holds
// out[m0 + wm + 32i + 8(v/4) + 4(lane/32) + v%4][n0 + wn + 32j + lane%32]
// (the output layout of the 32x32 MFMAs), through the epilogue, or raw into
// the workspace slot of a cut tile.  The epilogue's reads (the previous
// output to accumulate into, the ReLU mask) of one 32x32 tile are all issued
// before its stores: a store may alias a later read as far as the compiler
// knows, so interleaving them would serialise one memory latency per element.
constexpr int EPI_CHUNK = 8;     // outputs per lane whose epilogue reads are batched

template <int BM, int BN, int TM, int TN, bool FENCE = false>
__device__ __forceinline__ void store_tile(const KArgs& args, const Work& w,
                                           const floatx16 (&acc)[TM][TN], int wm, int wn,
                                           int lane) {
    const int lr = lane & 31, lk = lane >> 5;
    if (w.partial) {
        float* pslot = args.ws + ((long)(w.tile - args.tfull) * args.splits + w.z) * (BM * BN);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
                if constexpr (FENCE) __builtin_amdgcn_sched_barrier(0);   // one block at a time
            const int lcol = wn + 32 * j + lr;
            if (w.n0 + lcol >= args.Ncols) continue;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int lrow = wm + 32 * i + 8 * (v >> 2) + 4 * lk + (v & 3);
                    if (w.m0 + lrow < args.M) pslot[lrow * BN + lcol] = acc[i][j][v];
                }
        }
        return;
    }
    const int epi = args.epi;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const long col = w.n0 + wn + 32 * j + lr;
        if (col >= args.Ncols) continue;
        // output row stride and the address of (row0, col); the bias-gradient
        // column goes to bias_out[row]
        long ld = args.Ncols;
        float* cbase = args.out + col;
        if (epi & EPI_BIASCOL) {
            ld = args.Ncols - 1;
            cbase = args.out + col;
            if (col == args.Ncols - 1) { ld = 1; cbase = args.bias_out; }
        }
        const float bias = (epi & EPI_BIAS) ? args.bias[col] : 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if constexpr (FENCE) __builtin_amdgcn_sched_barrier(0);   // one block at a time
            const long row0 = w.m0 + wm + 32 * i + 4 * lk;
            // rows row0 + 8(v/4) + v%4 of this lane; those >= M are outside
            const int left = (int)min(args.M - row0, 32L);
            float* obase = cbase + row0 * ld;
            const float* mbase = (epi & EPI_MASK) ? args.mask + row0 * args.Ncols + col : nullptr;
            const int ldi = (int)ld, ldm = (int)args.Ncols;
#pragma unroll
            for (int v0 = 0; v0 < 16; v0 += EPI_CHUNK) {
                float prev[EPI_CHUNK], msk[EPI_CHUNK];
#pragma unroll
                for (int u = 0; u < EPI_CHUNK; ++u) {
                    const int r = 8 * ((v0 + u) >> 2) + ((v0 + u) & 3);
                    prev[u] = 0.f;
                    msk[u] = 1.f;
                    if (r < left) {
                        if (epi & EPI_ACCUM) prev[u] = obase[r * ldi];
                        if (epi & EPI_MASK) msk[u] = mbase[r * ldm];
                    }
                }
#pragma unroll
                for (int u = 0; u < EPI_CHUNK; ++u) {
                    const int r = 8 * ((v0 + u) >> 2) + ((v0 + u) & 3);
                    if (r >= left) continue;
                    float val = acc[i][j][v0 + u];
                    if (epi & EPI_BIAS) val += bias;
                    if (epi & EPI_RELU) val = fmaxf(val, 0.f);
                    if ((epi & EPI_MASK) && !(msk[u] > 0.f)) val = 0.f;
                    if (epi & EPI_ACCUM) val += prev[u];
                    obase[r * ldi] = val;
                    if (args.out16) args.out16[(row0 + r) * args.Ncols + col] = bf16_bits(val);
                }
            }
        }
    }
}

// The same writes through the wave's private 4 KB LDS slot (the k loop's
// buffers are free once its last barrier has passed): each 32x32 block is
// staged in LDS and read back with every lane holding 4 consecutive columns of
// one row (8 rows per pass, 4 passes, two at a time), so the epilogue's loads and stores are
// 16 bytes wide instead of 4.  Used when the output, the bias and the mask
// allow 16-byte access and there is no bias-gradient column; a group of 4
// columns that crosses the last column is written element by element.
constexpr int SLOT_FLOATS = 32 * 32;

template <int BM, int BN, int TM, int TN, bool FENCE = false>
__device__ __forceinline__ void store_tile_wide(const KArgs& args, const Work& w,
                                                const floatx16 (&acc)[TM][TN], int wm, int wn,
                                                int lane, float* slot) {
    const int lr = lane & 31, lk = lane >> 5;
    const int rq = lane >> 3, cq = (lane & 7) * 4;
    const int epi = args.epi;
    const long N = args.Ncols;
    float* pslot =
        w.partial ? args.ws + ((long)(w.tile - args.tfull) * args.splits + w.z) * (BM * BN)
                  : nullptr;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if constexpr (FENCE) __builtin_amdgcn_sched_barrier(0);   // one block at a time
#pragma unroll
            for (int v = 0; v < 16; ++v)
                slot[(8 * (v >> 2) + 4 * lk + (v & 3)) * 32 + lr] = acc[i][j][v];
            const int lcol = wn + 32 * j + cq;
            const long col = w.n0 + lcol;
            const bool full = col + 3 < N;
            float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!w.partial && (epi & EPI_BIAS) && col < N) {
                if (full) {
                    bias = *reinterpret_cast<const float4*>(args.bias + col);
                } else {
                    bias.x = args.bias[col];
                    if (col + 1 < N) bias.y = args.bias[col + 1];
                    if (col + 2 < N) bias.z = args.bias[col + 2];
                }
            }
            // two passes (rows 8q + rq) at a time: their epilogue reads first,
            // then the stores
#pragma unroll
            for (int q0 = 0; q0 < 4; q0 += 2) {
                float4 val[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    val[h] = *reinterpret_cast<const float4*>(slot + (8 * (q0 + h) + rq) * 32 + cq);
                if (w.partial) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int lrow = wm + 32 * i + 8 * (q0 + h) + rq;
                        if (w.m0 + lrow < args.M && col < N)
                            *reinterpret_cast<float4*>(pslot + lrow * BN + lcol) = val[h];
                    }
                    continue;
                }
                if (col >= N) continue;
                float4 prev[2], msk[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const long row = w.m0 + wm + 32 * i + 8 * (q0 + h) + rq;
                    prev[h] = make_float4(0.f, 0.f, 0.f, 0.f);
                    msk[h] = make_float4(1.f, 1.f, 1.f, 1.f);
                    if (row >= args.M) continue;
                    const long off = row * N + col;
                    if (full) {
                        if (epi & EPI_ACCUM) prev[h] = *reinterpret_cast<const float4*>(args.out + off);
                        if (epi & EPI_MASK) msk[h] = *reinterpret_cast<const float4*>(args.mask + off);
                    } else {
                        float* pp = &prev[h].x;
                        float* mm = &msk[h].x;
                        for (int e = 0; e < 4 && col + e < N; ++e) {
                            if (epi & EPI_ACCUM) pp[e] = args.out[off + e];
                            if (epi & EPI_MASK) mm[e] = args.mask[off + e];
                        }
                    }
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const long row = w.m0 + wm + 32 * i + 8 * (q0 + h) + rq;
                    if (row >= args.M) continue;
                    float o[4] = {val[h].x, val[h].y, val[h].z, val[h].w};
                    const float b4[4] = {bias.x, bias.y, bias.z, bias.w};
                    const float p4[4] = {prev[h].x, prev[h].y, prev[h].z, prev[h].w};
                    const float m4[4] = {msk[h].x, msk[h].y, msk[h].z, msk[h].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (epi & EPI_BIAS) o[e] += b4[e];
                        if (epi & EPI_RELU) o[e] = fmaxf(o[e], 0.f);
                        if ((epi & EPI_MASK) && !(m4[e] > 0.f)) o[e] = 0.f;
                        if (epi & EPI_ACCUM) o[e] += p4[e];
                    }
                    const long off = row * N + col;
                    if (full) {
                        *reinterpret_cast<float4*>(args.out + off) =
                            make_float4(o[0], o[1], o[2], o[3]);
                        if (args.out16) {
                            uint2 h;
                            h.x = pack_bf16(o[0], o[1]);
                            h.y = pack_bf16(o[2], o[3]);
                            *reinterpret_cast<uint2*>(args.out16 + off) = h;
                        }
                    } else {
                        for (int e = 0; e < 4 && col + e < N; ++e) {
                            args.out[off + e] = o[e];
                            if (args.out16) args.out16[off + e] = bf16_bits(o[e]);
                        }
                    }
                }
            }
        }
    }
}

// Column statistics of a whole tile for a following batch norm: the mean of
// each column over the tile's rows below M and the sum of squared deviations
// from it, two passes over the accumulators (values after the bias), lanes l
// and l + 32 combined by a shuffle, the waves along M through LDS in a fixed
// order.  Every thread of the workgroup takes part (barriers); lds holds at
// least (BM / WM + 1) * BN floats.
template <int BM, int BN, int TM, int TN>
__device__ __forceinline__ void tile_stats(const KArgs& args, const Work& w,
                                           const floatx16 (&acc)[TM][TN], int wm, int wn,
                                           int lane, float* lds) {
    constexpr int WAVES_M = BM / (32 * TM);
    const int lr = lane & 31, lk = lane >> 5;
    const int wave_m = wm / (32 * TM);
    const long rows = min((long)BM, args.M - w.m0);
    float* part = lds;                   // [WAVES_M][BN]
    float* mean = lds + WAVES_M * BN;    // [BN]
    const int t = threadIdx.x;
    const int nthreads = blockDim.x;
    float bias[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const long col = w.n0 + wn + 32 * j + lr;
        bias[j] = ((args.epi & EPI_BIAS) && col < args.Ncols) ? args.bias[col] : 0.f;
    }
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const float mu = pass ? mean[wn + 32 * j + lr] : 0.f;
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = wm + 32 * i + 8 * (v >> 2) + 4 * lk + (v & 3);
                    if (r < rows) {
                        const float d = acc[i][j][v] + bias[j] - mu;
                        sum += pass ? d * d : d;
                    }
                }
            sum += __shfl_xor(sum, 32);
            if (lk == 0) part[wave_m * BN + wn + 32 * j + lr] = sum;
        }
        __syncthreads();
        for (int c = t; c < BN; c += nthreads) {
            float s = 0.f;
            for (int m = 0; m < WAVES_M; ++m) s += part[m * BN + c];
            const long col = w.n0 + c;
            if (pass == 0) {
                mean[c] = rows > 0 ? s / (float)rows : 0.f;
            } else if (col < args.Ncols) {
                const long tm = w.m0 / BM;
                args.stats[tm * args.Ncols + col] = mean[c];
                args.stats[((long)args.tiles_m + tm) * args.Ncols + col] = s;
            }
        }
        __syncthreads();
    }
}

// Writes a wave's tile: the wide path when the kernel was built with it
// (WIDE) and its conditions hold (uniform).  The wide path costs registers,
// which the fp32 kernels on long reductions, where the epilogue is a small
// part of the time, keep for occupancy.
// The epilogue without column statistics: the wide path where the output, the
// bias, the mask and the workspace allow 16-byte access and there is no
// bias-gradient column, else the narrow one.
template <int BM, int BN, int TM, int TN, bool FENCE = false>
__device__ __forceinline__ void write_tile_plain(const KArgs& args, const Work& w,
                                                 const floatx16 (&acc)[TM][TN], int wm, int wn,
                                                 int lane, float* slot) {
    auto a16 = [](const void* p) { return (((uintptr_t)p) & 15) == 0; };
    const int epi = args.epi;
    const bool wide = !(epi & EPI_BIASCOL) && (args.Ncols & 3) == 0 && a16(args.out) &&
                      (!(epi & EPI_BIAS) || a16(args.bias)) &&
                      (!(epi & EPI_MASK) || a16(args.mask)) && a16(args.ws);
    if (wide)
        store_tile_wide<BM, BN, TM, TN, FENCE>(args, w, acc, wm, wn, lane, slot);
    else
        store_tile<BM, BN, TM, TN, FENCE>(args, w, acc, wm, wn, lane);
}

template <int BM, int BN, int TM, int TN, bool WIDE = true>
__device__ __forceinline__ void write_tile(const KArgs& args, const Work& w,
                                           const floatx16 (&acc)[TM][TN], int wm, int wn,
                                           int lane, float* slot, float* lds_all) {
    if constexpr (WIDE) {
        // column statistics of whole tiles (uniform per workgroup: it is either
        // whole or cut); the LDS slots are reused afterwards.  Built only into
        // the wide kernels, whose register budget already allows it.
        if (args.stats && !w.partial)
            tile_stats<BM, BN, TM, TN>(args, w, acc, wm, wn, lane, lds_all);
        write_tile_plain<BM, BN, TM, TN>(args, w, acc, wm, wn, lane, slot);
        return;
    }
    store_tile<BM, BN, TM, TN>(args, w, acc, wm, wn, lane);
}

// Raw buffer loads: the hardware's range check returns zeros for an offset at
// or past the end of the buffer, so an operand element that lies in the
// padding or outside the matrix is read with an offset of BUF_OOB instead of
// being masked.
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
constexpr unsigned BUF_OOB = 0x80000000u;      // buffer offset past any operand here
constexpr int BUF_CFG = 0x00020000;            // buffer descriptor word 3 (gfx9 family)

__device__ __forceinline__ uintx4 buf_load16(__amdgpu_buffer_rsrc_t rs, unsigned voff,
                                             unsigned soff) {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, 0);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// 16 bytes per lane from a buffer straight into LDS: lane l writes at lds + 16 l
// (the LDS byte address goes in M0, which must be uniform).  Written as
// assembly so that the compiler does not track these loads: the kernel waits
// for them itself (wait_vmcnt before the barrier that publishes a stage), and
// the compiler's own tracking, which cannot tell the stages apart across the
// loop's back edge, would wait for every load in flight before the next
// stage's LDS reads.  The memory clobber keeps LDS accesses on their side.
__device__ __forceinline__ void buf_load16_lds(__amdgpu_buffer_rsrc_t rs, void* lds, unsigned voff,
                                               unsigned soff) {
    const unsigned m0 = (unsigned)(size_t)(lds_ptr_t)lds;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(rs), "s"(soff)
                 : "memory", "m0");
}

// ---- operand gathers -------------------------------------------------------
// Each returns VW consecutive elements along the operand's contiguous axis
// (zero where the element lies outside the problem or in the padding).

template <int VW>
__device__ __forceinline__ void load_vec(const float* p, bool ok, float* v) {
    if constexpr (VW == 4) {
        if (ok) {
            float4 t = *reinterpret_cast<const float4*>(p);
            v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        } else {
            v[0] = v[1] = v[2] = v[3] = 0.f;
        }
    } else {
        v[0] = ok ? *p : 0.f;
    }
}

}  // namespace

struct KernelRef {
    const void* fn;
    int nt;
};

// The fp32 kernels on split operands (igemm_split.hip) for an operation and
// tile configuration (fast: igemm_split_kernel's FAST).
KernelRef split_kernel(int op, int cfg, bool fast);

// The fp32 kernels on operands whose pieces lie in memory (igemm_planes.hip).
KernelRef planes_kernel(int op, int cfg);

}  // namespace hp
