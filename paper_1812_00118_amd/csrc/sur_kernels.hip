// HIP kernels of the convolutional surrogate (gfx950, BF16 MFMA, FP32 accumulation).
//
// Activations are NHWC BF16; gradients FP32.  A 3x3 convolution with circular padding
//   out[p, o] = b[o] + sum_{tap, c} in[p + off(tap), c] w[o, tap, c],  off(tap) = (tap/3 - 1,
//   tap%3 - 1) in (y, x), is an implicit GEMM with M = pixels, N = Cout, K = 9 Cin; the
// K index runs over (tap, channel group of 8).  The same kernel computes the input
// gradient with the weights transposed and the taps mirrored.  The weight gradient is a
// GEMM over pixels (K = B H W) with the tiles transposed through LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "sur_internal.hpp"

namespace pfsur {

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// SiLU z sigmoid(z) and its derivative.  The sigmoid's reciprocal is the hardware
// v_rcp_f32 (1 ulp): the results are rounded to BF16 (or feed BF16 products) anyway, and
// an IEEE division would cost three times the instructions of the whole activation.
__device__ __forceinline__ float sigmoid(float z) {
    return __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}
__device__ __forceinline__ float silu(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float silu_grad(float z) {
    const float s = sigmoid(z);
    return s * (1.0f + z * (1.0f - s));
}

// Workgroup barrier over LDS traffic only: __syncthreads() also waits for the wave's global
// stores to be acknowledged
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// coordinate of a halo position from -1 on: positions past n, which no valid output uses,
// take that of n, so that the coordinate is in range for every n >= 1
__device__ __forceinline__ int halo(int v, int n) { return wrap(min(v, n), n); }

// 8 consecutive input channels at output-resolution pixel (b, y, x), through the layer's
// input mode (same resolution, 2x nearest upsampling, or 2x2 average pooling).  M is the
// mode when the caller fixes it at compile time, -1 to take g.mode.  Pixel indices fit
// 32 bits (at most 2^28 input pixels).
template <int M>
__device__ __forceinline__ bf16x8 gather8(const GatherP& g, int b, int y, int x, int c) {
    const int mode = M >= 0 ? M : g.mode;
    if (mode == MODE_UP) {
        y >>= 1;
        x >>= 1;
    }
    const int cc = g.c0 + c;
    if (mode != MODE_POOL) {
        const uint32_t pix = ((uint32_t)b * (uint32_t)g.Hin + (uint32_t)y) * (uint32_t)g.Win + (uint32_t)x;
        return *reinterpret_cast<const bf16x8*>(g.p + (size_t)pix * g.cs + cc);
    }
    const uint32_t pix =
        ((uint32_t)b * (uint32_t)g.Hin + 2u * (uint32_t)y) * (uint32_t)g.Win + 2u * (uint32_t)x;
    const __bf16* q = g.p + (size_t)pix * g.cs + cc;
    const size_t row = (size_t)g.Win * g.cs;
    const bf16x8 v0 = *reinterpret_cast<const bf16x8*>(q);
    const bf16x8 v1 = *reinterpret_cast<const bf16x8*>(q + g.cs);
    const bf16x8 v2 = *reinterpret_cast<const bf16x8*>(q + row);
    const bf16x8 v3 = *reinterpret_cast<const bf16x8*>(q + row + g.cs);
    bf16x8 r;
    for (int k = 0; k < 8; ++k)
        r[k] = (__bf16)(0.25f * ((((float)v0[k] + (float)v1[k]) + (float)v2[k]) + (float)v3[k]));
    return r;
}

// Staging of an E x E halo patch of 32 channels by a workgroup of 256 threads: a thread
// takes one (column, group of 8 channels) and every row of its own run of rows, so that a
// load's address is the one before it plus a row (the wrap is one compare), where addressing
// each 16-byte item by itself took 30 and more instructions.  Items lie row by row, column
// by column, 4 groups a pixel.
template <int E>
struct HaloCols {
    static constexpr int COLS = 4 * E;                    // (column, group) pairs
    static constexpr int RUNS = 256 / COLS;               // runs of rows side by side
    static constexpr int N = (E + RUNS - 1) / RUNS;       // rows (loads) per thread
    int col, row0;                                        // this thread's; row0 >= E: none
    __device__ __forceinline__ HaloCols()
        : col((int)threadIdx.x % COLS), row0((int)threadIdx.x / COLS * N) {}
    __device__ __forceinline__ bool has(int k) const { return row0 < RUNS * N && row0 + k < E; }
    // loads of the patch whose first row and column are y, x (from -1 on) of image b, at
    // channels c of the tensor g as it lies in memory; nothing past channel g.C
    __device__ __forceinline__ void load(const GatherP& g, int b, int y, int x, int c,
                                         bf16x8 (&r)[N]) const {
        const int cc = c + 8 * (col & 3);
        const size_t rowb = (size_t)g.Win * g.cs;
        const __bf16* p = g.p + (size_t)b * g.Hin * rowb +
                          (size_t)halo(x + (col >> 2), g.Win) * g.cs + g.c0 + cc;
        int yy = halo(min(y + row0, g.Hin), g.Hin);
        p += yy * rowb;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            r[k] = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
            if (has(k) && cc < g.C) r[k] = *reinterpret_cast<const bf16x8*>(p);
            ++yy;
            p += rowb;
            if (yy == g.Hin) {
                yy = 0;
                p -= (size_t)g.Hin * rowb;
            }
        }
    }
};

// ---------------------------------------------------------------------------
// Implicit-GEMM 3x3 convolution.  A workgroup of 4 waves covers 256 output pixels x 32
// output channels; a wave covers 64 pixels (4 MFMA row blocks) x 32 channels (2 column
// blocks) with v_mfma_f32_16x16x32_bf16, whose lane l holds A row l%16 / B column l%16
// with K elements 8(l/16)..8(l/16)+7, and C rows 4(l/16)..+3 of column l%16.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_conv3x3(ConvP a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = lane >> 4, r16 = lane & 15;
    const int P = a.B * a.H * a.W;
    const int p0 = blockIdx.x * 256 + wave * 64;
    const int co0 = blockIdx.y * 32;
    const int cg_per_tap = a.g.C >> 3;               // channel groups of 8 per tap
    const int nkg = 9 * cg_per_tap;
    // this lane's pixel in each of the 4 row blocks
    int pb[4], py[4], px[4];
    bool pv[4];
    for (int mb = 0; mb < 4; ++mb) {
        const int p = p0 + mb * 16 + r16;
        pv[mb] = p < P;
        const int pp = pv[mb] ? p : 0;
        px[mb] = pp % a.W;
        py[mb] = (pp / a.W) % a.H;
        pb[mb] = pp / (a.W * a.H);
    }
    f32x4 acc[4][2];
    for (int mb = 0; mb < 4; ++mb)
        for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero8 = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
    for (int s = 0; 4 * s < nkg; ++s) {
        const int kg = 4 * s + q;
        const bool kv = kg < nkg;
        const int tap = kv ? kg / cg_per_tap : 0;
        const int cg = kv ? kg - tap * cg_per_tap : 0;
        const int dy = tap / 3 - 1, dx = tap % 3 - 1;
        bf16x8 A[4], Bm[2];
        for (int mb = 0; mb < 4; ++mb)
            A[mb] = (kv && pv[mb]) ? gather8<-1>(a.g, pb[mb], wrap(py[mb] + dy, a.H), wrap(px[mb] + dx, a.W), cg * 8)
                                   : zero8;
        for (int nb = 0; nb < 2; ++nb) {
            const int co = co0 + nb * 16 + r16;
            Bm[nb] = (kv && co < a.Cout)
                         ? *reinterpret_cast<const bf16x8*>(a.w + (size_t)co * 9 * a.g.C + (size_t)kg * 8)
                         : zero8;
        }
        for (int mb = 0; mb < 4; ++mb)
            for (int nb = 0; nb < 2; ++nb)
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[mb], Bm[nb], acc[mb][nb], 0, 0, 0);
    }
    // epilogue
    for (int nb = 0; nb < 2; ++nb) {
        const int co = co0 + nb * 16 + r16;
        if (co >= a.Cout) continue;
        const float bias = a.bias ? a.bias[co] : 0.0f;
        for (int mb = 0; mb < 4; ++mb)
            for (int j = 0; j < 4; ++j) {
                const int p = p0 + mb * 16 + 4 * q + j;
                if (p >= P) continue;
                const float v = acc[mb][nb][j] + bias;
                if (a.zout) a.zout[(size_t)p * a.Cout + co] = (__bf16)v;
                if (a.out)
                    a.out[(size_t)p * a.out_cs + a.out_c0 + co] = (__bf16)(a.act ? silu(v) : v);
                if (a.fout) {
                    float* f = a.fout + (size_t)p * a.f_cs + a.f_c0 + co;
                    *f = v;
                }
            }
    }
}

// ---------------------------------------------------------------------------
// 16x16-pixel tiles of the first two layers (k_conv_first, k_conv_stem): wave w owns patch
// rows 4w..4w+3 as two 32-pixel blocks of two rows.
// ---------------------------------------------------------------------------
constexpr int TP = 16;                 // output patch edge
constexpr int HP = TP + 2;             // halo patch edge
constexpr int UPH = TP / 2 + 2;        // the same at half resolution (an upsampled input)
constexpr int APAD = 40;               // BF16 per staged pixel (32 channels + pad)
// Row pitch of the staged halo patch: HP pixels of APAD BF16 plus RPAD BF16, so that a
// row is 112 16-byte units (16 mod 32).  The 32 lanes of a B-operand read cover two patch
// rows of 16 pixels, and gfx950's LDS serves such a 16-byte read in 512-byte groups of
// 32 lanes: with rows HP * APAD apart, two lanes 14 pixels apart in the two rows meet in
// one bank (measured: 1/6 of the LDS cycles of a probe in this pattern were conflict
// stalls, for every APAD); with the pitch at 16 mod 32 units the second row's 16 units
// are exactly the ones the first row leaves free.
constexpr int RPAD = 176;
constexpr int ROWA = HP * APAD + RPAD; // BF16 per staged patch row

// Epilogues of a 16x16-pixel tile.  The MFMAs compute D[channel][pixel] (weights as the
// A operand), so lane l holds pixel l%32 of its 32-pixel row block and, for j = 0..15,
// channel 8(j/4) + 4(l/32) + j%4 of the 32-channel block.
//
// The bias comes from LDS (sBias, the workgroup's output channels, zeros without a bias): as
// per-lane loads from memory, each behind its own wait, it was the largest part of the
// epilogue of the row kernel below.
//
// values of row block mb, channel block nb: 4 runs of 4 channels
template <int NB, int MB>
__device__ __forceinline__ void tile_values(const f32x16 (&acc)[MB][NB], int mb, int nb, int g,
                                            const float* sBias, float (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(&sBias[nb * 32 + 8 * q + 4 * g]);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * q + e] = acc[mb][nb][4 * q + e] + b[e];
    }
}

// 16 values as BF16, through SiLU if act is set
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void to_bf16(const float (&v)[16], int act, bf16x4 (&o)[4]) {
    if (act) {
#pragma unroll
        for (int e = 0; e < 16; ++e) o[e >> 2][e & 3] = (__bf16)silu(v[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) o[e >> 2][e & 3] = (__bf16)v[e];
    }
}

// FP32 output of one pixel's 32-channel block
__device__ __forceinline__ void put_f32(const ConvP& a, size_t p, int cb, int g,
                                        const float (&v)[16]) {
    float* f = a.fout + p * a.f_cs + a.f_c0 + cb + 4 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(f + 8 * q) =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}

// Direct: each lane writes its runs of 4 consecutive channels as one 8-byte (BF16) or
// 16-byte (FP32) store.  Used for 32-channel tiles, where it measured as fast as the
// staged form without its extra barrier.
template <int NB>
__device__ __forceinline__ void tile_epilogue_direct(const ConvP& a, const f32x16 (&acc)[2][NB],
                                                     int b, int y0, int x0, int co0, int wave,
                                                     int l32, int g, const float* sBias) {
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const int y = y0 + 4 * wave + 2 * mb + (l32 >> 4), x = x0 + (l32 & 15);
        if (y >= a.H || x >= a.W) continue;
        const size_t p = ((size_t)b * a.H + y) * a.W + x;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int cb = co0 + nb * 32;
            if (cb >= a.Cout) break;
            float v[16];
            bf16x4 o[4];
            tile_values(acc, mb, nb, g, sBias, v);
            if (a.zout) {
                to_bf16(v, 0, o);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<bf16x4*>(a.zout + p * a.Cout + cb + 8 * q + 4 * g) = o[q];
            }
            if (a.out) {
                to_bf16(v, a.act, o);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<bf16x4*>(a.out + p * a.out_cs + a.out_c0 + cb + 8 * q +
                                               4 * g) = o[q];
            }
            if (a.fout) put_f32(a, p, cb, g, v);
        }
    }
}

// Staged (64-channel tiles, 8-12% faster there): the BF16 outputs go through LDS, one
// 32-channel block at a time, in the wave's own region of OROW BF16 per pixel (sO: 64
// OROW per wave): each lane writes its 4-channel runs, then reads back 16 bytes (8
// channels) of one pixel so that four consecutive lanes store one pixel's 64 contiguous
// bytes and a store instruction covers 16 pixels instead of 64 scattered 8-byte pieces.
// The FP32 output (input gradients) keeps direct 16-byte stores.  With pout set, the
// staged activations also give their 2x2 averages (the input of the next level's pooling
// layer), so that layer reads a compact quarter-size tensor at its own resolution.
constexpr int OROW = 40;   // BF16 per staged pixel: 32 channels + pad

// LDS accesses of one wave complete in order; the wait and the clobber keep the
// compiler from moving the read-back across the writes (and the next writes across it)
__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int NB>
__device__ __forceinline__ void tile_epilogue_staged(const ConvP& a, const f32x16 (&acc)[2][NB],
                                                     int b, int y0, int x0, int co0, int wave,
                                                     int l32, int g, const float* sBias,
                                                     __bf16* __restrict__ sO) {
    const int lane = l32 + 32 * g;
    __bf16* so = sO + wave * 64 * OROW;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int cb = co0 + nb * 32;            // first channel of the block
        if (cb >= a.Cout) break;
        float v[2][16];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) tile_values(acc, mb, nb, g, sBias, v[mb]);
        if (a.fout) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                const int y = y0 + 4 * wave + 2 * mb + (l32 >> 4), x = x0 + (l32 & 15);
                if (y < a.H && x < a.W) put_f32(a, ((size_t)b * a.H + y) * a.W + x, cb, g, v[mb]);
            }
        }
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            __bf16* dst = pass == 0 ? a.zout : a.out;
            if (!dst) continue;
            const int cs = pass == 0 ? a.Cout : a.out_cs;
            const int c0 = pass == 0 ? 0 : a.out_c0;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                bf16x4 o[4];
                to_bf16(v[mb], pass == 1 && a.act, o);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<bf16x4*>(&so[(mb * 32 + l32) * OROW + 8 * q + 4 * g]) = o[q];
            }
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = lane + 64 * k;                 // 16-byte item: pixel i/4
                const int px = i >> 2, grp = i & 3;
                const int mb = px >> 5, pl = px & 31;
                const int y = y0 + 4 * wave + 2 * mb + (pl >> 4), x = x0 + (pl & 15);
                const bf16x8 val = *reinterpret_cast<const bf16x8*>(&so[px * OROW + 8 * grp]);
                if (y < a.H && x < a.W) {
                    const size_t p = ((size_t)b * a.H + y) * a.W + x;
                    *reinterpret_cast<bf16x8*>(dst + p * cs + c0 + cb + 8 * grp) = val;
                }
            }
            if (pass == 1 && a.pout) {
                // 2x2 average of the stored activations for the next level's pooling
                // layer, added in the pooling gather's order: (y, x), (y, x+1), (y+1, x),
                // (y+1, x+1).  The wave's 4 x 16 pixels give 2 x 8 pooled pixels x 4
                // groups of 8 channels: one item per lane.
                const int pp = lane >> 2, grp = lane & 3;
                const int mb = pp >> 3, pc = pp & 7;
                const int base = mb * 32 + 2 * pc;               // staged pixel (y, x)
                const bf16x8 v00 = *reinterpret_cast<const bf16x8*>(&so[base * OROW + 8 * grp]);
                const bf16x8 v01 = *reinterpret_cast<const bf16x8*>(&so[(base + 1) * OROW + 8 * grp]);
                const bf16x8 v10 = *reinterpret_cast<const bf16x8*>(&so[(base + 16) * OROW + 8 * grp]);
                const bf16x8 v11 = *reinterpret_cast<const bf16x8*>(&so[(base + 17) * OROW + 8 * grp]);
                bf16x8 r;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    r[e] = (__bf16)(0.25f * ((((float)v00[e] + (float)v01[e]) + (float)v10[e]) +
                                             (float)v11[e]));
                const int y = y0 + 4 * wave + 2 * mb, x = x0 + 2 * pc;
                if (y + 1 < a.H && x + 1 < a.W) {
                    const size_t q = ((size_t)b * (a.H >> 1) + (y >> 1)) * (a.W >> 1) + (x >> 1);
                    *reinterpret_cast<bf16x8*>(a.pout + q * a.pout_cs + cb + 8 * grp) = r;
                }
            }
            wave_lds_sync();
        }
    }
}

// ---------------------------------------------------------------------------
// Implicit-GEMM 3x3 convolution for C and Cout multiples of 32.  A workgroup (4 waves)
// computes NCB blocks of 32 output channels x ROWS rows of 32 output pixels of one image;
// a wave one block x RW rows, on v_mfma_f32_32x32x16_bf16 with the weights as A (lane l: row
// l%32 = output channel, K elements 8(l/32)..+7) and a row of pixels as B (column l%32 =
// pixel, same K), so D[channel][pixel] has lane l on pixel l%32 with channels
// 8(j/4) + 4(l/32) + j%4.  The input channels go in chunks of 32:
//   pixels   the chunk's halo rows go from memory straight into LDS (wrap applied by the
//            addresses, an upsampled input at its own resolution), two chunks (or tiles)
//            ahead of the products, in three buffers with one barrier a chunk; 64 bytes a
//            pixel, its four 16-byte groups exchanged by the column's bits 1-2 so that 8
//            consecutive lanes' reads hit distinct banks.  With one chunk ahead, through
//            registers, the loads' latency was not covered: without any products the
//            network's layers took two thirds of their time.
//   weights  straight from memory (L2) into registers, 18 operands a chunk, used for all of
//            a wave's rows; with up to NW chunks (NW > 0) they stay there for all tiles, else
//            (NW = 0) the next chunk's replace them as their tap row is done.
// An input row's 6 operands are read from LDS once and serve the three output rows that use
// it: (RW + 2) 6 reads for 18 RW products (4 rows: one read per two products), where taking
// weights and pixels both from LDS for 64 pixels x 64 channels needed one read per product
// and left the kernel bound by LDS (72 KB a chunk and wave, the LDS as busy as the matrix
// cores at their peak).  The products of an output are added in the order chunk, tap,
// channel half, whatever RW.
// Measured in the 256x256 U-Net against 64 x 64 blocks with both operands in LDS: batch 1,
// all layers, 248 -> 117 us; batch 32, 128x128 pixels 64 -> 64 channels 67 -> 54 us (715
// TFLOP/s), 64x64 pixels 256 -> 128 channels 96 -> 79 us (980 TFLOP/s), 256x256 pixels 64 ->
// 32 channels 143 -> 114 us (3.5 TB/s of unique bytes).  What is left: the matrix cores in
// the deep layers, and memory with them in the 256x256 ones, whose workgroups' products and
// transfers overlap in part only.
// ---------------------------------------------------------------------------
constexpr int RPX = 32;                // output pixels of a row tile

// Epilogues (of a wave's rows, acc[r]: row r).  EPI_OUT: zout, out, pout and fout, as given;
// EPI_HEAD: the 1x1 head; EPI_BWD + BWD_*: the backward pass's.
enum { EPI_OUT = 0, EPI_HEAD = 1, EPI_BWD = 2 };

// where a wave's rows lie: image b, rows y.. , this lane's column x; the output channels from
// cb on
struct RowTile {
    int b, y, x, cb;
};

// 32 pixels x 32 channels of BF16 (row staged in so as RPX x OROW) to dst[p * cs + c], 16
// bytes a lane: four consecutive lanes store one pixel's 64 bytes
__device__ __forceinline__ void put_row(const ConvP& a, const RowTile& t, int r, int lane, int l32,
                                        const __bf16* so, __bf16* dst, int cs, int c) {
    if (t.y + r >= a.H) return;
    const size_t p0 = ((size_t)t.b * a.H + t.y + r) * a.W + (t.x - l32);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int px = (lane >> 2) + 16 * k, grp = lane & 3;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(&so[px * OROW + 8 * grp]);
        if (t.x - l32 + px < a.W)
            *reinterpret_cast<bf16x8*>(dst + (p0 + px) * cs + c + 8 * grp) = v;
    }
}

__device__ __forceinline__ void stage_row(__bf16* so, int l32, int g, const bf16x4 (&o)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<bf16x4*>(&so[l32 * OROW + 8 * q + 4 * g]) = o[q];
}

// Outputs.  With pout set, the stored activations of two rows also give their 2x2 averages
// (the input of the next level's pooling layer), so that layer reads a compact quarter-size
// tensor at its own resolution.
template <int RW>
__device__ __forceinline__ void rows_out(const ConvP& a, const f32x16 (&acc)[RW][1],
                                         const RowTile& t, int lane, int l32, int g,
                                         const float* sBias, __bf16* so) {
    float top[16];                               // of a pooled pair of rows
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        float v[16];
        bf16x4 o[4];
        tile_values(acc, r, 0, g, sBias, v);
        if (a.fout && t.y + r < a.H && t.x < a.W)
            put_f32(a, ((size_t)t.b * a.H + t.y + r) * a.W + t.x, t.cb, g, v);
        if (a.zout) {
            to_bf16(v, 0, o);
            stage_row(so, l32, g, o);
            wave_lds_sync();
            put_row(a, t, r, lane, l32, so, a.zout, a.Cout, t.cb);
            wave_lds_sync();
        }
        if (a.out) {
            to_bf16(v, a.act, o);
            stage_row(so, l32, g, o);
            wave_lds_sync();
            put_row(a, t, r, lane, l32, so, a.out, a.out_cs, a.out_c0 + t.cb);
            wave_lds_sync();
            if (RW > 1 && a.pout) {
                // the 2x2 averages, added in the pooling gather's order: (y, x), (y, x+1),
                // (y+1, x), (y+1, x+1); x + 1 is lane l ^ 1's
                float m[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float w = (float)o[e >> 2][e & 3], x1 = __shfl_xor(w, 1);
                    m[e] = (r & 1) ? 0.25f * ((top[e] + w) + x1) : w + x1;
                }
                if (r & 1) {
                    to_bf16(m, 0, o);
                    if (!(l32 & 1)) stage_row(so, l32 >> 1, g, o);
                    wave_lds_sync();
                    const int pc = lane >> 2, grp = lane & 3, x = t.x - l32 + 2 * pc;
                    const bf16x8 u = *reinterpret_cast<const bf16x8*>(&so[pc * OROW + 8 * grp]);
                    if (x + 1 < a.W && t.y + r < a.H) {
                        const size_t q = ((size_t)t.b * (a.H >> 1) + ((t.y + r) >> 1)) * (a.W >> 1) + (x >> 1);
                        *reinterpret_cast<bf16x8*>(a.pout + q * a.pout_cs + t.cb + 8 * grp) = u;
                    }
                    wave_lds_sync();
                } else {
#pragma unroll
                    for (int e = 0; e < 16; ++e) top[e] = m[e];
                }
            }
        }
    }
}

// Partial sums of the 1x1 head over the 16 channels 8q + 4g + e (q, e = 0..3) of one
// pixel, in that order.  A head output is (half(g = 0) + half(g = 1)) + b: the order
// k_head_train uses and the one the fused epilogue gets, where lanes l and l + 32 of a wave
// hold the two halves of a pixel's 32 channels.
__device__ __forceinline__ void head_half(const float (&v)[16], int g, const float* wh,
                                          float (&p)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                p[k] = fmaf(v[4 * q + e], wh[k * 32 + 8 * q + 4 * g + e], p[k]);
}

// The last 32-channel layer at inference: its activations (rounded to BF16, as they would be
// stored) go straight into the 1x1 head; the layer's activation tensor is never written.  sH
// holds the head's weights and biases.
template <int RW>
__device__ __forceinline__ void rows_head(const ConvP& a, const f32x16 (&acc)[RW][1],
                                          const RowTile& t, int g, const float* sBias,
                                          const float* sH) {
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        float v[16];
        bf16x4 b[4];
        tile_values(acc, r, 0, g, sBias, v);
        to_bf16(v, a.act, b);
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = (float)b[e >> 2][e & 3];
        float p[4], o[4];
        head_half(v, g, sH, p);
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = __shfl_xor(p[k], 32);
        if (g == 0 && t.y + r < a.H && t.x < a.W) {
            const size_t px = ((size_t)t.b * a.H + t.y + r) * a.W + t.x;
            reinterpret_cast<float4*>(a.head_out)[px] =
                make_float4((p[0] + o[0]) + sH[128], (p[1] + o[1]) + sH[129],
                            (p[2] + o[2]) + sH[130], (p[3] + o[3]) + sH[131]);
        }
    }
}

// The backward pass: a layer's input gradient goes straight into the dz of the layer that
// produced the input, dz = (gradient of its activation) silu'(z), rounded to BF16 once, so
// that the FP32 gradients (4 and more bytes a value, written and read again) stay in
// registers.  Each gradient is formed as by separate passes, in the same order.
//   BWD_SAME  the producer is at the same resolution.  Channels below a.dz_c0 belong to a
//             skip connection, whose gradient gets a second part later: stored to a.fout.
//   BWD_UP    the input was upsampled: the 2x2 sum of the gradient, at half resolution.
//   BWD_POOL  the input was pooled: a quarter of the gradient on each of four pixels at
//             double resolution, added to the skip connection's in a.fout.
// (Gradients of 16 samples of 256x256: 725 us of element-wise kernels before, none now.)
__device__ __forceinline__ void load_z(const __bf16* z, int g, bf16x4 (&zq)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) zq[q] = *reinterpret_cast<const bf16x4*>(z + 8 * q + 4 * g);
}
__device__ __forceinline__ void silu_bwd(float (&v)[16], const bf16x4 (&zq)[4]) {
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] *= silu_grad((float)zq[e >> 2][e & 3]);
}

template <int RW, int BWD>
__device__ __forceinline__ void rows_bwd(const ConvP& a, const f32x16 (&acc)[RW][1],
                                         const RowTile& t, int lane, int l32, int g, __bf16* so) {
    const int cd = t.cb - a.dz_c0;               // channel of dz
    if constexpr (BWD == BWD_SAME) {
        if (cd < 0) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if (t.y + r < a.H && t.x < a.W) {
                    float v[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) v[e] = acc[r][0][e];
                    put_f32(a, ((size_t)t.b * a.H + t.y + r) * a.W + t.x, t.cb, g, v);
                }
            return;
        }
    }
    // What a row needs from memory is asked for before the stores of those before it (all of
    // it at once, or for a pooled input the next pixel's): row by row, each waited for its own
    // loads and for the stores before them (256x256, 16 images: the first pooling layer's
    // 105 -> 90 us, the backward layers together 5% less).
    const int xc = min(t.x, a.W - 1);
    if constexpr (BWD == BWD_SAME) {
        bf16x4 z[RW][4];
#pragma unroll
        for (int r = 0; r < RW; ++r)
            load_z(a.zin + (((size_t)t.b * a.H + min(t.y + r, a.H - 1)) * a.W + xc) * a.dz_cs + cd, g, z[r]);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            float v[16];
            bf16x4 o[4];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = acc[r][0][e];
            silu_bwd(v, z[r]);
            to_bf16(v, 0, o);
            stage_row(so, l32, g, o);
            wave_lds_sync();
            put_row(a, t, r, lane, l32, so, a.dz, a.dz_cs, cd);
            wave_lds_sync();
        }
    } else if constexpr (BWD == BWD_UP) {
        bf16x4 z[RW / 2 + 1][4];
        auto half = [&](int r) {
            return ((size_t)t.b * (a.H >> 1) + (min(t.y + r, a.H - 1) >> 1)) * (a.W >> 1) + (xc >> 1);
        };
#pragma unroll
        for (int r = 0; r < RW; r += 2) load_z(a.zin + half(r) * a.dz_cs + cd, g, z[r / 2]);
#pragma unroll
        for (int r = 0; r < RW; r += 2) {        // a block's rows are r and r + 1, its lanes l, l^1
            float v[16];
            bf16x4 o[4];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float u = acc[r][0][e], w = acc[r + (RW > 1)][0][e];
                v[e] = ((u + __shfl_xor(u, 1)) + w) + __shfl_xor(w, 1);
            }
            silu_bwd(v, z[r / 2]);
            to_bf16(v, 0, o);
            if (t.y + r < a.H && t.x < a.W && !(t.x & 1)) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<bf16x4*>(a.dz + half(r) * a.dz_cs + cd + 8 * q + 4 * g) = o[q];
            }
        }
    } else {
        bf16x4 z[2][4];
        f32x4 f[2][4];
        auto pixel = [&](int s) {
            return ((size_t)t.b * 2 * a.H + 2 * min(t.y + (s >> 2), a.H - 1) + (s >> 1 & 1)) * 2 * a.W +
                   2 * xc + (s & 1);
        };
        auto load = [&](int s) {
            const float* sk = a.fout + pixel(s) * a.f_cs + a.f_c0 + t.cb + 4 * g;
#pragma unroll
            for (int q = 0; q < 4; ++q) f[s & 1][q] = *reinterpret_cast<const f32x4*>(sk + 8 * q);
            load_z(a.zin + pixel(s) * a.dz_cs + cd, g, z[s & 1]);
        };
        load(0);
#pragma unroll
        for (int s = 0; s < 4 * RW; ++s) {
            const int r = s >> 2;
            if (s + 1 < 4 * RW) load(s + 1);
            float u[16];
            bf16x4 o[4];
#pragma unroll
            for (int e = 0; e < 16; ++e) u[e] = fmaf(0.25f, acc[r][0][e], f[s & 1][e >> 2][e & 3]);
            silu_bwd(u, z[s & 1]);
            to_bf16(u, 0, o);
            if (t.y + r < a.H && t.x < a.W) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<bf16x4*>(a.dz + pixel(s) * a.dz_cs + cd + 8 * q + 4 * g) = o[q];
            }
        }
    }
}

template <int NCB, int RW, int NW, int MODE, int EPI, bool BIG>
__global__ void __launch_bounds__(256, 2) k_conv_rows(ConvP a, int tiles_per_wg) {
    constexpr int RG = 4 / NCB, ROWS = RG * RW;               // row groups, rows of a tile
    constexpr int XR = MODE == MODE_UP ? ROWS / 2 + 2 : ROWS + 2;
    constexpr int XC = MODE == MODE_UP ? RPX / 2 + 2 : RPX + 2;
    constexpr int ITEMS = XR * XC * 4, NI = (ITEMS + 255) / 256;   // 16-byte items
    constexpr int BUF = (ITEMS + 63) / 64 * 64 * 8;           // whole waves of items, in BF16
    static_assert(MODE != MODE_UP || ROWS % 2 == 0, "whole rows of the upsampled input");
    static_assert(EPI != EPI_BWD + BWD_UP || RW % 2 == 0, "a 2x2 block's rows are in one wave");
    static_assert(XC * 64 % 128 == 0, "a row's first pixel starts a line of banks");
    // One object: with several, the compiler marks which one an access is to, and has every
    // read of the pixels wait for all loads to LDS in flight, the latest included
    struct Shared {
        __bf16 a[3 * BUF], o[4][RPX * OROW];
        float bias[32 * NCB], head[EPI == EPI_HEAD ? 4 * 32 + 4 : 1];
    };
    __shared__ __align__(16) Shared sh;
    __bf16* const sA = sh.a;
    float *const sBias = sh.bias, *const sH = sh.head;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __bf16* const sO = sh.o[wave];
    const int l32 = lane & 31, g = lane >> 5;
    const int wcb = wave % NCB, rg = wave / NCB;              // the wave's channel block, rows
    const int cb0 = blockIdx.y * 32 * NCB, cb = cb0 + 32 * wcb;
    if (threadIdx.x < 32 * NCB) sBias[threadIdx.x] = a.bias ? a.bias[cb0 + threadIdx.x] : 0.0f;
    if constexpr (EPI == EPI_HEAD)
        for (int i = threadIdx.x; i < 4 * 32 + 4; i += 256)
            sH[i] = i < 128 ? a.head_w[i] : a.head_b[i - 128];
    const int tx_n = (a.W + RPX - 1) / RPX, ty_n = (a.H + ROWS - 1) / ROWS;
    const int ntile = a.B * tx_n * ty_n;
    // a contiguous run of tiles per XCD (workgroups go round the 8 of them), so that the halos
    // that neighbouring tiles share are read from memory once and then from that XCD's L2
    const int xcd = blockIdx.x % 8, xq = gridDim.x / 8, xr = gridDim.x % 8;
    const int t_beg = (xcd * xq + min(xcd, xr) + (int)blockIdx.x / 8) * tiles_per_wg;
    const int t_end = min(ntile, t_beg + tiles_per_wg);
    if (t_beg >= t_end) return;
    const int nchunk = NW > 0 ? NW : a.g.C / 32;
    auto tile_at = [&](int t, int& b, int& y0, int& x0) {      // down the columns
        const int ty = t % ty_n;
        t /= ty_n;
        const int tx = t % tx_n;
        b = t / tx_n;
        x0 = tx * RPX;
        y0 = ty * ROWS;
    };

    // pixels: the tile and chunk to fetch next, and this thread's items of that tile's halo as
    // offsets (in 16 bytes) into its image
    int ft = t_beg, fch = 0, fb = 0, fy = 0, fx = 0;
    uint32_t off[NI];
    const uint32_t img_items = (uint32_t)a.g.Hin * (uint32_t)a.g.Win * (uint32_t)(a.g.cs >> 3);
    auto image = [&]() { return a.g.p + (size_t)fb * img_items * 8 + a.g.c0; };
    auto window = [&]() {                                     // the image in elements of 16 bytes
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(image()), 16, img_items, 0x00027000);
    };
    auto img = window();
    const __bf16* big = nullptr;
    auto aim = [&]() {
        tile_at(ft, fb, fy, fx);
        if constexpr (BIG) big = image();
        else img = window();
        const int yb = (MODE == MODE_UP ? fy / 2 : fy) - 1, xb = (MODE == MODE_UP ? fx / 2 : fx) - 1;
        if constexpr (MODE != MODE_POOL)
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                const int first = (k + 1) * 256 > ITEMS && k * 256 + wave * 64 >= ITEMS
                                      ? wave * 64 : k * 256 + wave * 64;
                const int it = min(first + lane, ITEMS - 1);
                const int pix = it >> 2, r = pix / XC, c = pix - r * XC;
                off[k] = ((uint32_t)halo(yb + r, a.g.Hin) * (uint32_t)a.g.Win +
                          (uint32_t)halo(xb + c, a.g.Win)) * (uint32_t)(a.g.cs >> 3) +
                         ((it & 3) ^ ((c >> 1) & 3));
            }
    };
    // fetch it into buffer `to`.  Every wave issues NI loads on every path, past the last
    // item its first one again and past the last tile that tile again (into a buffer that is
    // not read any more), so that the compiler and arrive() know how many are outstanding:
    // behind a branch, the streamed weights' waits would take in these loads too
    auto fetch = [&](int to) {
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            const int first = (k + 1) * 256 > ITEMS && k * 256 + wave * 64 >= ITEMS
                                  ? wave * 64 : k * 256 + wave * 64;
            __bf16* dst = &sA[to * BUF + first * 8];
            if constexpr (MODE == MODE_POOL) {
                const int it = min(first + lane, ITEMS - 1);
                const int pix = it >> 2, r = pix / XC, c = pix - r * XC;
                *reinterpret_cast<bf16x8*>(dst + lane * 8) = gather8<MODE_POOL>(
                    a.g, fb, halo(fy - 1 + r, a.H), halo(fx - 1 + c, a.W),
                    32 * fch + 8 * ((it & 3) ^ ((c >> 1) & 3)));
            } else {
                typedef __attribute__((address_space(3))) void* to_t;
                typedef const __attribute__((address_space(1))) void* from_t;
                if constexpr (BIG) {
                    // the compiler takes these for flat accesses and waits for all of them
                    // where it would wait for some of the streamed weights
                    __builtin_amdgcn_global_load_lds((from_t)(big + 32 * fch + (size_t)off[k] * 8),
                                                     (to_t)dst, 16, 0, 0);
                } else {
#ifdef __HIP_DEVICE_COMPILE__                                  // (unknown to the host's pass)
                    __builtin_amdgcn_struct_ptr_buffer_load_lds(img, (to_t)dst, 16, off[k], 0,
                                                                64 * fch, 0, 0);
#endif
                }
            }
        }
        if (++fch == nchunk) {
            fch = 0;
            if (ft + 1 < t_end) {
                ++ft;
                aim();
            }
        }
    };

    // weights: operand (tap, h) is channels 16h..+15 of the chunk; packed (weights_bf16) they
    // are 1 KB runs in the order lanes take them.  Through a buffer descriptor, so that an
    // address is a lane's offset plus a scalar
    bf16x8 W[NW > 0 ? NW : 1][9][2];
    const auto wsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(a.w), 0, a.Cout * 9 * a.g.C * 2, 0x00027000);
    const int wchunk = a.packed ? a.Cout / 32 * 18 * 1024 : 64;
    const int wtap = a.packed ? 2048 : a.g.C * 2, whalf = a.packed ? 1024 : 32;
    const int wlane = a.packed ? cb / 32 * 18 * 1024 + lane * 16 : (cb + l32) * 9 * a.g.C * 2 + 16 * g;
    auto load_w = [&](int into, int chunk, int dy) {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                W[into][3 * dy + dx][h] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                wsrc, wlane, chunk * wchunk + (3 * dy + dx) * wtap + h * whalf, 0));
    };

    // where the lane reads its operands: position (rg RW + i, l32 + dx) of the halo, halved
    // ((v + 1) >> 1) for an upsampled input (rg RW is even there, or RW is 1); pat[.][dx][h]
    // for the first rows of each kind
    constexpr int RK = MODE == MODE_UP ? 2 : 1;
    int pat[RK][3][2];
#pragma unroll
    for (int i = 0; i < RK; ++i)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int row = MODE == MODE_UP ? (rg * RW + i + 1) >> 1 : rg * RW;
                const int col = MODE == MODE_UP ? (l32 + dx + 1) >> 1 : l32 + dx;
                pat[i][dx][h] = (row * XC + col) * 32 + 8 * ((2 * h + g) ^ ((col >> 1) & 3));
            }

    f32x16 acc[RW][1];
    // The products of one chunk, from buffer `from` with weights W[w]; `next`: the chunk whose
    // weights replace them (streamed weights only).  Input row i of the wave's halo gives 6
    // operands (dx, h), each for the output rows i - dy; operand s = 6 i + 2 dx + h is read
    // two ahead of its products.
    auto products = [&](int from, auto w_, int next) {
        constexpr int w = decltype(w_)::value;
        const __bf16* px = &sA[from * BUF];
        auto pixels = [&](int s) {
            const int i = s / 6;
            const __bf16* q = px + pat[i % RK][s % 6 / 2][s & 1] + i / RK * XC * 32;
            return *reinterpret_cast<const bf16x8*>(q);
        };
        constexpr int NS = 6 * (RW + 2);
        bf16x8 F[3];
        F[0] = pixels(0);
        F[1] = pixels(1);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int i = s / 6, k = s % 6;
            if (s + 2 < NS) F[(s + 2) % 3] = pixels(s + 2);
#pragma unroll
            for (int dy = 2; dy >= 0; --dy) {
                const int r = i - dy;
                if (r < 0 || r >= RW) continue;
                acc[r][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(W[w][3 * dy + k / 2][k & 1],
                                                                    F[s % 3], acc[r][0], 0, 0, 0);
            }
            // the order to keep: the read two ahead, then these products
            if (s + 2 < NS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            const int n = (i < 2 ? i : 2) - (i < RW ? 0 : i - RW + 1) + 1;
            if (n == 1) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (n == 2) __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            if (n == 3) __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
            // tap row dy is done after input row RW - 1 + dy
            if (NW == 0 && k == 5 && i >= RW - 1) load_w(0, next, i - (RW - 1));
        }
    };
    // End of a chunk's products: this wave's part of the next chunk has to be in LDS, then
    // every wave's.  Loads complete in order, and that fetch was followed by the latest one's
    // NI and by the streamed weights of two chunks: so many may be outstanding.
    auto arrive = [&]() {
        constexpr int LATER = (NW == 0 ? 36 : 0) + NI;
        static_assert(LATER < 64, "the counter has six bits");
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LATER) : "memory");
    };

    aim();
    fetch(0);
    fetch(1);
    if constexpr (NW > 0)
        static_for<0, NW>([&](auto c_) {
            constexpr int c = decltype(c_)::value;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) load_w(c, c, dy);
        });
    else
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) load_w(0, 0, dy);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    int buf = 0;
    for (int t = t_beg; t < t_end; ++t) {
        RowTile at;
        int y0, x0;
        tile_at(t, at.b, y0, x0);
        at.y = y0 + rg * RW;
        at.x = x0 + l32;
        at.cb = cb;
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[r][0][j] = 0.0f;
        auto chunk = [&](auto w_, int next) {
            const int two = buf == 0 ? 2 : buf - 1;          // (buf + 2) % 3
            fetch(two);
            __builtin_amdgcn_sched_barrier(0);               // arrive() counts what follows it
            products(buf, w_, next);
            arrive();
            buf = buf == 2 ? 0 : buf + 1;
        };
        if constexpr (NW > 0) {
            static_for<0, NW>([&](auto c_) { chunk(c_, 0); });
        } else {
            for (int ch = 0; ch < nchunk; ++ch)
                chunk(std::integral_constant<int, 0>{}, ch + 1 == nchunk ? 0 : ch + 1);
        }
        if constexpr (EPI == EPI_OUT) rows_out<RW>(a, acc, at, lane, l32, g, sBias + 32 * wcb, sO);
        else if constexpr (EPI == EPI_HEAD) rows_head<RW>(a, acc, at, g, sBias + 32 * wcb, sH);
        else rows_bwd<RW, EPI - EPI_BWD>(a, acc, at, lane, l32, g, sO);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // no load outlives its LDS
}

// ---------------------------------------------------------------------------
// First layer (8 input channels, same resolution): the whole K = 9 taps x 8 channels
// fits one stage.  K is ordered (tap, channel) and padded to 10 taps, so each 16-wide
// MFMA K step covers taps 2k (lanes 0-31) and 2k+1 (lanes 32-63).
// ---------------------------------------------------------------------------
constexpr int BPAD1 = 88;   // 10 taps x 8 channels + pad: conflict-free 16-byte reads

__global__ void __launch_bounds__(256, 2) k_conv_first(ConvP a) {
    __shared__ __align__(16) __bf16 sA[HP * HP * 8];
    __shared__ __align__(16) __bf16 sB[32 * BPAD1];
    __shared__ __align__(16) float sBias[32];
    if (threadIdx.x < 32)
        sBias[threadIdx.x] = a.bias ? a.bias[blockIdx.y * 32 + threadIdx.x] : 0.0f;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    const int tx_n = (a.W + TP - 1) / TP, ty_n = (a.H + TP - 1) / TP;
    int blk = blockIdx.x;
    const int tx = blk % tx_n;
    blk /= tx_n;
    const int ty = blk % ty_n;
    const int b = blk / ty_n;
    const int x0 = tx * TP, y0 = ty * TP;
    const int co0 = blockIdx.y * 32;
    const bf16x8 zero8 = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
    for (int it = threadIdx.x; it < HP * HP; it += 256) {
        const int py = it / HP, px = it - py * HP;
        *reinterpret_cast<bf16x8*>(&sA[it * 8]) =
            gather8<MODE_SAME>(a.g, b, halo(y0 - 1 + py, a.H), halo(x0 - 1 + px, a.W), 0);
    }
    for (int it = threadIdx.x; it < 32 * 10; it += 256) {
        const int col = it / 10, tap = it - col * 10;
        const int co = co0 + col;
        *reinterpret_cast<bf16x8*>(&sB[col * BPAD1 + tap * 8]) =
            (tap < 9 && co < a.Cout)
                ? *reinterpret_cast<const bf16x8*>(a.w + ((size_t)co * 9 + tap) * 8)
                : zero8;
    }
    __syncthreads();
    f32x16 acc[2][1];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[mb][0][j] = 0.0f;
    const int prow = 4 * wave + (l32 >> 4), pcol = l32 & 15;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int tap = 2 * k + g;
        const int dy = tap / 3, dx = tap % 3;
        const bf16x8 Bm = *reinterpret_cast<const bf16x8*>(&sB[l32 * BPAD1 + tap * 8]);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            const bf16x8 A =
                tap < 9 ? *reinterpret_cast<const bf16x8*>(
                              &sA[((prow + 2 * mb + dy) * HP + pcol + dx) * 8])
                        : zero8;
            acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Bm, A, acc[mb][0], 0, 0, 0);
        }
    }
    tile_epilogue_direct<1>(a, acc, b, y0, x0, co0, wave, l32, g, sBias);
}

// ---------------------------------------------------------------------------
// Inference stem: the first layer (8 input channels) computed straight into the second
// layer's staged halo patch.  A workgroup's 16x16 output tile of the second layer needs
// the first layer's activations on its 18x18 halo patch; it computes them from a 20x20
// patch of the input with k_conv_first's MFMA sequence, bias, SiLU and BF16 rounding (so
// they are bitwise the values the first layer would have stored, the periodic wrap
// commuting with the convolution) and writes them to LDS as the second layer's input patch;
// the second layer's products (k_conv_rows' order) and its epilogue follow.  Both layers'
// weight operands stay in registers; workgroups walk runs of tiles with the next tile's
// input loads in flight.  The first layer's activations never reach HBM; training keeps
// the two layers apart (its backward pass needs them).  Needs H, W >= 16 (one period of
// wrap covers the patch).  Measured: 127 us at batch 32; first 151 against 158 us for the two
// kernels (the pair is bound by its per-tile chain of load, two MFMA phases and stores,
// not by the HBM bytes it saves).
// ---------------------------------------------------------------------------
constexpr int HP2 = HP + 2;                       // input patch edge
constexpr int STEM_PIX = HP * HP;                 // first-layer pixels per tile
constexpr int STEM_BLK = (STEM_PIX + 31) / 32;    // their 32-pixel MFMA blocks

__global__ void __launch_bounds__(256, 2) k_conv_stem(ConvP a0, ConvP a, int tiles_per_wg) {
    __shared__ __align__(16) __bf16 sX[HP2 * HP2 * 8];
    __shared__ __align__(16) __bf16 sA[HP * ROWA];
    static_assert(4 * 64 * OROW <= HP * ROWA, "epilogue staging must fit the patch buffer");
    __shared__ __align__(16) float sBias[64];          // of the first layer, then the second
    if (threadIdx.x < 64) {
        const float* b = threadIdx.x < 32 ? a0.bias : a.bias;
        sBias[threadIdx.x] = b ? b[threadIdx.x & 31] : 0.0f;
    }
    constexpr int X_PER_T = (HP2 * HP2 + 255) / 256;   // 16-byte input items per thread
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    const int tx_n = (a.W + TP - 1) / TP, ty_n = (a.H + TP - 1) / TP;
    const int ntile = a.B * tx_n * ty_n;
    // a contiguous run of tiles per XCD, as k_conv_rows
    const int xcd = blockIdx.x % 8, xq = gridDim.x / 8, xr = gridDim.x % 8;
    const int t_beg = (xcd * xq + min(xcd, xr) + (int)blockIdx.x / 8) * tiles_per_wg;
    const int t_end = min(ntile, t_beg + tiles_per_wg);
    const bf16x8 zero8 = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
    auto tile_xy = [&](int t, int& b, int& y0, int& x0) {
        const int tx = t % tx_n;
        t /= tx_n;
        const int ty = t % ty_n;
        b = t / ty_n;
        x0 = tx * TP;
        y0 = ty * TP;
    };
    // a tile's input pixels (y0 - 2 + qy, x0 - 2 + qx), into registers
    bf16x8 rx[X_PER_T];
    auto load_x = [&](int t) {
        int b, y0, x0;
        tile_xy(t, b, y0, x0);
#pragma unroll
        for (int k = 0; k < X_PER_T; ++k) {
            const int it = threadIdx.x + 256 * k;
            if (it < HP2 * HP2) {
                const int qy = it / HP2, qx = it - qy * HP2;
                rx[k] = gather8<MODE_SAME>(a0.g, b, wrap(y0 - 2 + qy, a.H),
                                           wrap(x0 - 2 + qx, a.W), 0);
            }
        }
    };
    // both layers' weight operands, held in registers for the workgroup's life: lane l32 is output channel l32;
    // first layer: taps 2s + g (the tenth zero) of 8 channels; second layer: tap t, input
    // channels 16h + 8g .. + 7
    bf16x8 w0[5], w1[9][2];
#pragma unroll
    for (int s5 = 0; s5 < 5; ++s5) {
        const int tap = 2 * s5 + g;
        w0[s5] = tap < 9 ? *reinterpret_cast<const bf16x8*>(a0.w + ((size_t)l32 * 9 + tap) * 8)
                         : zero8;
    }
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            w1[tap][h] = *reinterpret_cast<const bf16x8*>(a.w + ((2 * tap + h) * 64 + lane) * 8);
    if (t_beg < t_end) load_x(t_beg);
    for (int t = t_beg; t < t_end; ++t) {
        int b, y0, x0;
        tile_xy(t, b, y0, x0);
        __syncthreads();                           // the previous tile is done with sX, sA
#pragma unroll
        for (int k = 0; k < X_PER_T; ++k) {
            const int it = threadIdx.x + 256 * k;
            if (it < HP2 * HP2) *reinterpret_cast<bf16x8*>(&sX[it * 8]) = rx[k];
        }
        __syncthreads();
        if (t + 1 < t_end) load_x(t + 1);          // in flight while this tile computes
        // the first layer on the 18x18 halo patch, 32 pixels (in row-major patch order) per
        // MFMA block; the last block's spare lanes repeat its last pixel and store nothing
        for (int k = wave; k < STEM_BLK; k += 4) {
            const int p = 32 * k + l32;
            const int pc = p < STEM_PIX ? p : STEM_PIX - 1;
            const int py = pc / HP, px = pc - py * HP;
            f32x16 acc;
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = 0.0f;
#pragma unroll
            for (int s = 0; s < 5; ++s) {
                const int tap = 2 * s + g;
                const int dy = tap / 3, dx = tap % 3;
                const bf16x8 Bm = w0[s];
                const bf16x8 A = tap < 9 ? *reinterpret_cast<const bf16x8*>(
                                               &sX[((py + dy) * HP2 + px + dx) * 8])
                                         : zero8;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Bm, A, acc, 0, 0, 0);
            }
            if (p < STEM_PIX) {
                float v[16];
                bf16x4 o[4];
                const f32x16 one[1][1] = {{acc}};
                tile_values(one, 0, 0, g, sBias, v);
                to_bf16(v, a0.act, o);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<bf16x4*>(&sA[py * ROWA + px * APAD + 8 * q + 4 * g]) = o[q];
            }
        }
        __syncthreads();
        // the second layer, over its one input chunk
        f32x16 acc[2][1];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[mb][0][j] = 0.0f;
        const int prow = 4 * wave + (l32 >> 4), pcol = l32 & 15;
        // K steps s = 2 tap + h, the patch operands of step s + 1 read ahead of step s's
        // MFMAs
        auto ld = [&](int s, bf16x8 (&A)[2]) {
            const int tap = s >> 1, h = s & 1;
            const int dy = tap / 3, dx = tap % 3;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                A[mb] = *reinterpret_cast<const bf16x8*>(
                    &sA[(prow + 2 * mb + dy) * ROWA + (pcol + dx) * APAD + 16 * h + 8 * g]);
        };
        bf16x8 Ac[2];
        ld(0, Ac);
#pragma unroll
        for (int s = 0; s < 18; ++s) {
            bf16x8 An[2];
            if (s + 1 < 18) ld(s + 1, An);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
                acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[s >> 1][s & 1], Ac[mb],
                                                                     acc[mb][0], 0, 0, 0);
            if (s + 1 < 18) {
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // the next reads,
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // then these MFMAs
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) Ac[mb] = An[mb];
            }
        }
        __syncthreads();                 // every wave is done reading the patch
        tile_epilogue_staged<1>(a, acc, b, y0, x0, 0, wave, l32, g, sBias + 32, sA);
    }
}

// ---------------------------------------------------------------------------
// Weight gradient staged through LDS: dW[o, tap, c] = sum_p dz[p, o] in[p + off(tap), c], and
// with it the bias gradient sum_p dz[p, o].  A workgroup owns 32 output x 32 input channels
// and all 9 taps, and a contiguous range of 16x16 pixel patches (split K).  A patch's dz and
// input halo are staged as they lie in memory, 32 channels (64 bytes) a pixel; the products
// sum over pixels, so each operand (8 pixels of one channel per lane) is read with gfx950's
// transposing LDS reads, at any pixel offset: no transposed or shifted copies.  Wave w
// reduces over patch rows 4w..4w+3; it reads each input row once for the three dy that use
// it (22 operand reads per 36 MFMAs).  The bias is a tenth product with a matrix of ones, in
// the workgroups of input channels 0..31.  The 4 wave sums are added in a fixed order and
// the workgroup's sums go to part[split].  Bound by the matrix cores together with the L2
// reads (37 KB a patch) and their latency; the form before this one transposed through 176 two-byte LDS
// writes per thread and patch and ran the layer 64 -> 64 on 16x128x128 in 76 us; this one
// takes 32 us (0.6 PFLOP/s; 19 GFLOP), of which the matrix cores are busy 9.  Without its
// products, its loads or its final sums it takes 5 to 8 us less each: they overlap in part
// only.  (Loads straight into LDS in two stages changed nothing; sums of one tap at a time in
// place of three cost 2.5 us.)
// ---------------------------------------------------------------------------
// Operand of a product over 16 consecutive pixels: lane l gets pixels 8(l/32)..+7 of channel
// l%32 from pixel-major LDS of 64 bytes a pixel.  A transposing read takes, in each group of
// 16 lanes, 4 pixels x 16 channels (lane i of the group supplies pixel i/4, channels
// 4(i%4)..+3) and returns to lane i the 4 pixels of channel i.  p: the lane's own address for
// the first 4 pixels; the next 4 are `next` BF16 further.
__device__ __forceinline__ bf16x8 read_pixels(const __bf16* p, int next) {
    typedef __attribute__((address_space(3))) bf16x4* lds4;
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds4)(p));
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds4)(p + next));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

constexpr int RED_STRIDE = 33;                 // floats per output channel of a wave's sums

template <int MODE>
__global__ void __launch_bounds__(256, 2) k_wgrad_tiled(WgradP a, int patches_per_split,
                                                        int npatch, int nsplit) {
    // the halo of an upsampled input is staged at its own resolution
    constexpr int XE = MODE == MODE_UP ? UPH : HP;
    union Shared {
        struct {
            __bf16 d[TP * TP * 32], x[XE * XE * 32];
        } in;
        float red[3][4][32][RED_STRIDE];           // of three taps' sums: wave, output, input channel
    };
    __shared__ __align__(16) Shared sh;
    __bf16 *const sD = sh.in.d, *const sX = sh.in.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    const int C = a.g.C;
    // workgroup -> (split, channel pair): all pairs of a split on one XCD (workgroups go
    // round the 8 XCDs), so that a patch comes from memory once and then from that XCD's L2
    const int no = (a.Cout + 31) / 32, npair = no * ((C + 31) / 32);
    const int split = (blockIdx.x >> 3) / npair * 8 + (blockIdx.x & 7);
    const int pair = (blockIdx.x >> 3) % npair;
    if (split >= nsplit) return;
    const int o0 = pair % no * 32, c0 = pair / no * 32;
    const int tx_n = (a.W + TP - 1) / TP, ty_n = (a.H + TP - 1) / TP;
    const int pbeg = split * patches_per_split;
    const int pend = min(npatch, pbeg + patches_per_split);
    const bf16x8 zero8 = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
    const bool with_bias = c0 == 0;

    f32x16 acc[10];                                // the taps, then the bias
#pragma unroll
    for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[t][j] = 0.0f;

    const HaloCols<XE> hc;
    bf16x8 rd[4], rx[hc.N];
    auto load = [&](int patch) {
        int q = patch;
        const int tx = q % tx_n;
        q /= tx_n;
        const int ty = q % ty_n;
        const int b = q / ty_n;
        const int x0 = tx * TP, y0 = ty * TP;
        // dz: wave w stages rows 4w..4w+3, a lane one (pixel, group) of each
        const int x = x0 + (lane >> 2), o = o0 + 8 * (lane & 3);
        const bool in = x < a.W && o < a.Cout;
        const __bf16* d = a.dz + (((size_t)b * a.H + y0 + 4 * wave) * a.W + x) * a.Cout + o;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            rd[k] = zero8;
            if (in && y0 + 4 * wave + k < a.H) rd[k] = *reinterpret_cast<const bf16x8*>(d);
            d += (size_t)a.W * a.Cout;
        }
        if constexpr (MODE == MODE_UP) {
            hc.load(a.g, b, y0 / 2 - 1, x0 / 2 - 1, c0, rx);
        } else if constexpr (MODE == MODE_SAME) {
            hc.load(a.g, b, y0 - 1, x0 - 1, c0, rx);
        } else {
            const int c = c0 + 8 * (hc.col & 3);
#pragma unroll
            for (int k = 0; k < hc.N; ++k)
                rx[k] = hc.has(k) && c < C
                            ? gather8<MODE>(a.g, b, halo(y0 - 1 + hc.row0 + k, a.H),
                                            halo(x0 - 1 + (hc.col >> 2), a.W), c)
                            : zero8;
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<bf16x8*>(&sD[((4 * wave + k) * TP * 4 + lane) * 8]) = rd[k];
#pragma unroll
        for (int k = 0; k < hc.N; ++k)
            if (hc.has(k))
                *reinterpret_cast<bf16x8*>(&sX[((hc.row0 + k) * hc.COLS + hc.col) * 8]) = rx[k];
    };
    // this lane's pixel (of the first 4) and channel in a transposing read
    const int pk = 8 * g + ((lane & 15) >> 2), ck = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const __bf16* dzp = &sD[(4 * wave * TP + pk) * 32 + ck];
    const __bf16* xp[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
        xp[dx] = MODE == MODE_UP ? &sX[(2 * wave * UPH + ((pk + dx + 1) >> 1)) * 32 + ck]
                                 : &sX[(4 * wave * HP + pk + dx) * 32 + ck];
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;

    if (pbeg < pend) load(pbeg);
    for (int patch = pbeg; patch < pend; ++patch) {
        lds_barrier();
        store();
        lds_barrier();
        if (patch + 1 < pend) load(patch + 1);
        bf16x8 A[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) A[r] = read_pixels(dzp + r * TP * 32, 4 * 32);
        if (with_bias)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[9] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[r], ones, acc[9], 0, 0, 0);
        // halo rows 4w + i: output row r uses row i = r + dy for tap row dy
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            bf16x8 Bv[3];
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
                Bv[dx] = MODE == MODE_UP ? read_pixels(xp[dx] + ((i + 1) >> 1) * UPH * 32, 2 * 32)
                                         : read_pixels(xp[dx] + i * HP * 32, 4 * 32);
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int r = i - dy;
                if (r < 0 || r > 3) continue;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[3 * dy + dx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        A[r], Bv[dx], acc[3 * dy + dx], 0, 0, 0);
            }
        }
    }
    // fixed-order sum of the 4 waves, three taps (then the bias) at a time: part[split] holds
    // [Cout][9][C], then [Cout].  (Barriers that wait for each tap's stores measured
    // 12% slower over the network's layers.)
    float* part = a.part + (size_t)split * ((size_t)a.Cout * 9 * C + a.Cout);
    auto put = [&](auto first, auto count, auto&& store_at) {
        lds_barrier();
#pragma unroll
        for (int t = 0; t < count; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j)
                sh.red[t][wave][8 * (j >> 2) + 4 * g + (j & 3)][l32] = acc[first + t][j];
        lds_barrier();
#pragma unroll
        for (int t = 0; t < count; ++t)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int o = (threadIdx.x >> 5) + 8 * k, c = threadIdx.x & 31;
                store_at(first + t, o, c,
                         ((sh.red[t][0][o][c] + sh.red[t][1][o][c]) + sh.red[t][2][o][c]) +
                             sh.red[t][3][o][c]);
            }
    };
    auto put_tap = [&](int tap, int o, int c, float v) {
        if (o0 + o < a.Cout && c0 + c < C) part[((size_t)(o0 + o) * 9 + tap) * C + c0 + c] = v;
    };
    static_for<0, 3>([&](auto d) {
        put(std::integral_constant<int, 3 * decltype(d)::value>{}, std::integral_constant<int, 3>{},
            put_tap);
    });
    if (with_bias)
        put(std::integral_constant<int, 9>{}, std::integral_constant<int, 1>{},
            [&](int, int o, int c, float v) {
                if (c == 0 && o0 + o < a.Cout) part[(size_t)a.Cout * 9 * C + o0 + o] = v;
            });
}

// Sum over the splits: sum_s part[s][i], i < n, rows of `stride`, into out[i] for i < nhead
// and tail[i - nhead] from there on.  A block takes 64 consecutive i; its 16 rows of lanes
// take every 16th split, each with four independent partial sums (in float64: the adds are
// free beside the loads) so that several loads are in flight; every combination is in a
// fixed order, so the result does not depend on scheduling.  (With 4 rows of lanes a
// level-0 layer's 512 splits were a chain of 32 waits.)
constexpr int RS_ROWS = 16;
__global__ void __launch_bounds__(64 * RS_ROWS)
k_reduce_splits(const float* __restrict__ part, int nsplit, size_t stride, size_t n, size_t nhead,
                float* __restrict__ out, float* __restrict__ tail) {
    __shared__ double sred[RS_ROWS][64];
    const int ci = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const size_t i = (size_t)blockIdx.x * 64 + ci;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < n) {
        int k = sl;
        for (; k + 3 * RS_ROWS < nsplit; k += 4 * RS_ROWS)
#pragma unroll
            for (int u = 0; u < 4; ++u) s[u] += part[(size_t)(k + u * RS_ROWS) * stride + i];
        for (; k < nsplit; k += RS_ROWS) s[0] += part[(size_t)k * stride + i];
    }
    sred[sl][ci] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    if (sl == 0 && i < n) {
        double t = sred[0][ci];
#pragma unroll
        for (int r = 1; r < RS_ROWS; ++r) t += sred[r][ci];
        if (i < nhead) out[i] = (float)t;
        else tail[i - nhead] = (float)t;
    }
}

// The 1x1 head in training, forward and backward in one pass over the last layer's
// activations, for HEAD_PPB pixels per block: out[p, o] = bh[o] + sum_c act[p, c] wh[o, c]
// (the order of head_half, as at inference), the squared error against y, dout =
// 2 (out - y) / n, the last layer's dz[p, c] = silu'(z[p, c]) sum_o dout[p, o] wh[o, c], and
// the partial sums part[block][o * 32 + c] of dout[p, o] act[p, c], part[block][128 + o] of
// dout[p, o] and err[block] of the squared error.  First a thread takes a pixel (out and
// dout, kept in LDS), then a pair of channels of every 16th pixel, so that the 128 sums need
// one reduction over 16 threads at the end (a thread per pixel for all of it spent 790
// shuffles on them; with separate passes for out, dout and the rest: 115 us on 16x256x256).
constexpr int HEAD_PPB = 1024;
__global__ void __launch_bounds__(256) k_head_train(const __bf16* __restrict__ act,
                                                    const float* __restrict__ wh,
                                                    const float* __restrict__ bh,
                                                    const float* __restrict__ y,
                                                    const __bf16* __restrict__ z, size_t P,
                                                    float scale, __bf16* __restrict__ dz,
                                                    float* __restrict__ part,
                                                    double* __restrict__ err) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    __shared__ float4 sd[256];
    __shared__ double sred[16][136];
    __shared__ double serr[256];
    const int c = 2 * (threadIdx.x & 15), r = threadIdx.x >> 4;
    float w[4][2];
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int e = 0; e < 2; ++e) w[o][e] = wh[32 * o + c + e];
    double dw[4][2] = {}, db = 0.0, e2 = 0.0;
    const size_t pb = (size_t)blockIdx.x * HEAD_PPB;
    const size_t pe = pb + HEAD_PPB < P ? pb + HEAD_PPB : P;
    for (size_t p0 = pb; p0 < pe; p0 += 256) {
        const size_t p = p0 + threadIdx.x;
        float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p < pe) {
            float v0[16], v1[16], h0[4], h1[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bf16x8 v = *reinterpret_cast<const bf16x8*>(act + p * 32 + 8 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v0[4 * q + e] = (float)v[e];
                    v1[4 * q + e] = (float)v[4 + e];
                }
            }
            head_half(v0, 0, wh, h0);
            head_half(v1, 1, wh, h1);
            const float4 t = reinterpret_cast<const float4*>(y)[p];
            d = make_float4(((h0[0] + h1[0]) + bh[0]) - t.x, ((h0[1] + h1[1]) + bh[1]) - t.y,
                            ((h0[2] + h1[2]) + bh[2]) - t.z, ((h0[3] + h1[3]) + bh[3]) - t.w);
            e2 += ((double)d.x * d.x + (double)d.y * d.y) + ((double)d.z * d.z + (double)d.w * d.w);
            d = make_float4(2.0f * d.x / scale, 2.0f * d.y / scale, 2.0f * d.z / scale,
                            2.0f * d.w / scale);
        }
        __syncthreads();
        sd[threadIdx.x] = d;
        __syncthreads();
        const int np = (int)(pe - p0 < 256 ? pe - p0 : 256);
#pragma unroll
        for (int k0 = 0; k0 < 16; k0 += 8) {
            float s[4][2] = {}, sb = 0.0f;
#pragma unroll
            for (int k = k0; k < k0 + 8; ++k) {
                const int j = r + 16 * k;
                if (j < np) {
                    const float4 q = sd[j];
                    const float dd[4] = {q.x, q.y, q.z, q.w};
                    const bf16x2 av = *reinterpret_cast<const bf16x2*>(act + (p0 + j) * 32 + c);
                    const bf16x2 zv = *reinterpret_cast<const bf16x2*>(z + (p0 + j) * 32 + c);
                    bf16x2 ov;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float gr =
                            fmaf(dd[3], w[3][e],
                                 fmaf(dd[2], w[2][e], fmaf(dd[0], w[0][e], dd[1] * w[1][e])));
#pragma unroll
                        for (int o = 0; o < 4; ++o) s[o][e] = fmaf(dd[o], (float)av[e], s[o][e]);
                        ov[e] = (__bf16)(gr * silu_grad((float)zv[e]));
                    }
                    *reinterpret_cast<bf16x2*>(dz + (p0 + j) * 32 + c) = ov;
                    if (c < 8) sb += dd[c >> 1];
                }
            }
#pragma unroll
            for (int o = 0; o < 4; ++o)
#pragma unroll
                for (int e = 0; e < 2; ++e) dw[o][e] += (double)s[o][e];
            db += (double)sb;
        }
    }
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int e = 0; e < 2; ++e) sred[r][32 * o + c + e] = dw[o][e];
    if (c < 8) sred[r][128 + (c >> 1)] = db;
    serr[threadIdx.x] = e2;
    __syncthreads();
    if (threadIdx.x < 132) {
        double t = 0.0;
        for (int k = 0; k < 16; ++k) t += sred[k][threadIdx.x];
        part[(size_t)blockIdx.x * 132 + threadIdx.x] = (float)t;
    }
    for (int n = 128; n > 0; n >>= 1) {
        if (threadIdx.x < (unsigned)n) serr[threadIdx.x] += serr[threadIdx.x + n];
        __syncthreads();
    }
    if (threadIdx.x == 0) err[blockIdx.x] = serr[0];
}

__global__ void __launch_bounds__(256) k_sum_f64(const double* __restrict__ part, int n,
                                                 double* __restrict__ out) {
    __shared__ double sred[256];
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) v += part[i];
    sred[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < (unsigned)w) sred[threadIdx.x] += sred[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sred[0];
}

// Adam (Kingma & Ba) on FP32 masters
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, size_t n, float lr, float c1, float c2) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
}

// Position of the weight of output channel o, tap, input channel c (Cout x 9 x C of them) in
// the order the row kernel's lanes take them: [chunk of 32 c][block of 32 o][tap][16 c][8 c]
// [o][8]
__device__ __forceinline__ size_t packed_at(int Cout, int o, int tap, int c) {
    const size_t block = (size_t)(c >> 5) * (Cout >> 5) + (o >> 5);
    return ((block * 18 + 2 * tap + ((c >> 4) & 1)) * 64 + ((c >> 3) & 1) * 32 + (o & 31)) * 8 + (c & 7);
}

// BF16 copies of one layer's weights w [Cout][9][Cin]: wf in packed order (the first layer's
// 8 input channels as they are) and, for the input gradient, wt, the weights of a layer Cout
// -> Cin with the taps mirrored (tap -> 8 - tap), packed
__global__ void k_weights_bf16(const float* __restrict__ w, int Cout, int Cin, __bf16* __restrict__ wf,
                               __bf16* __restrict__ wt) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t n = (size_t)Cout * 9 * Cin;
    if (i >= n) return;
    const int ci = (int)(i % Cin);
    const int tap = (int)((i / Cin) % 9);
    const int co = (int)(i / (9 * (size_t)Cin));
    const bool packed = Cin % 32 == 0;
    wf[packed ? packed_at(Cout, co, tap, ci) : i] = (__bf16)w[i];
    if (wt && packed) wt[packed_at(Cin, ci, 8 - tap, co)] = (__bf16)w[i];
}

// density of sample b at order parameter phi (clamped: phi overshoots [0, 1] slightly and
// rho must stay positive for the velocity conversion)
__device__ __forceinline__ float dens(const DensTab& d, size_t b, float phi) {
    return fmaf(fminf(fmaxf(phi, 0.0f), 1.0f), d.rd[b], d.rl[b]);
}

// network input from solver fields, sample b = blockIdx.y of the batch:
// x[b, y, x, :] = ((phi - s0) k0, (P - s1) k1, (u_x - s2) k2, (u_y - s3) k3,
// lrr_b lrr_scale, 0, 0, 0) with u = J / rho(phi)
__global__ void k_pack(const float* __restrict__ phi, const float* __restrict__ P,
                       const float* __restrict__ J, DensTab d, Norm nm, size_t HW,
                       __bf16* __restrict__ x) {
    const size_t s = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= HW) return;
    const size_t b = blockIdx.y;
    const size_t i = b * HW + s;
    const float rho = dens(d, b, phi[i]);
    const float f[4] = {phi[i], P[i], J[2 * b * HW + s] / rho, J[(2 * b + 1) * HW + s] / rho};
    bf16x8 v;
    for (int c = 0; c < 4; ++c) v[c] = (__bf16)((f[c] - nm.shift[c]) * nm.scale[c]);
    v[4] = (__bf16)(d.lrr[b] * nm.lrr_scale);
    v[5] = v[6] = v[7] = (__bf16)0.0f;
    *reinterpret_cast<bf16x8*>(x + i * 8) = v;
}

// training target of sample b = blockIdx.y: y[s, c] = (f1_c - f0_c) / out_scale[c] for
// (phi, P, u_x, u_y)
__global__ void k_pack_target(const float* __restrict__ phi0, const float* __restrict__ P0,
                              const float* __restrict__ J0, const float* __restrict__ phi1,
                              const float* __restrict__ P1, const float* __restrict__ J1, DensTab d,
                              Norm nm, size_t HW, float* __restrict__ y) {
    const size_t s = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= HW) return;
    const size_t b = blockIdx.y;
    const size_t i = b * HW + s, jx = 2 * b * HW + s, jy = (2 * b + 1) * HW + s;
    const float r0 = dens(d, b, phi0[i]), r1 = dens(d, b, phi1[i]);
    float4 v;
    v.x = (phi1[i] - phi0[i]) / nm.out_scale[0];
    v.y = (P1[i] - P0[i]) / nm.out_scale[1];
    v.z = (J1[jx] / r1 - J0[jx] / r0) / nm.out_scale[2];
    v.w = (J1[jy] / r1 - J0[jy] / r0) / nm.out_scale[3];
    reinterpret_cast<float4*>(y)[i] = v;
}

// a predicted residual applied to sample b = blockIdx.y in place: phi and P advance by
// out * out_scale, the velocity J / rho(phi) likewise, and J = rho(phi_new) u_new
__global__ void k_apply(const float* __restrict__ out, Norm nm, DensTab d, size_t HW,
                        float* __restrict__ phi, float* __restrict__ P, float* __restrict__ J) {
    const size_t s = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= HW) return;
    const size_t b = blockIdx.y;
    const size_t i = b * HW + s, jx = 2 * b * HW + s, jy = (2 * b + 1) * HW + s;
    const float4 o = reinterpret_cast<const float4*>(out)[i];
    const float r0 = dens(d, b, phi[i]);
    const float ux = J[jx] / r0 + o.z * nm.out_scale[2];
    const float uy = J[jy] / r0 + o.w * nm.out_scale[3];
    const float ph = phi[i] + o.x * nm.out_scale[0];
    const float r1 = dens(d, b, ph);
    phi[i] = ph;
    P[i] += o.y * nm.out_scale[1];
    J[jx] = r1 * ux;
    J[jy] = r1 * uy;
}

// max |a - b| per block for sample blockIdx.y of a batch of fields of n values:
// part[sample][block]; a non-finite difference propagates (fmaxf would drop it)
__global__ void __launch_bounds__(256) k_maxdiff(const float* __restrict__ a, const float* __restrict__ b,
                                                 size_t n, float* __restrict__ part) {
    __shared__ float sred[256];
    const size_t off = (size_t)blockIdx.y * n;
    float m = 0.f;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const float d = fabsf(a[off + i] - b[off + i]);
        m = d > m || d != d ? d : m;
    }
    sred[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < (unsigned)w) {
            const float o = sred[threadIdx.x + w];
            if (o > sred[threadIdx.x] || o != o) sred[threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = sred[0];
}

// largest hand-over speed |J| / rho'(phi) per block for sample blockIdx.y (see maxspeed):
// part[sample][block]; a non-finite speed propagates
__global__ void __launch_bounds__(256) k_maxspeed(const float* __restrict__ phi,
                                                  const float* __restrict__ J, DensTab d, int H,
                                                  int W, float* __restrict__ part) {
    __shared__ float sred[256];
    const size_t b = blockIdx.y;
    const size_t n = (size_t)H * W;
    const float* ph = phi + b * n;
    float m = 0.f;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const int y = (int)(i / W), x = (int)(i - (size_t)y * W);
        const int xm = x == 0 ? W - 1 : x - 1, xp = x == W - 1 ? 0 : x + 1;
        const int ym = y == 0 ? H - 1 : y - 1, yp = y == H - 1 ? 0 : y + 1;
        const float c = ph[i];
        // (2/T) sum_i w_i (phi(x + c_i) - phi(x)), D2Q9 weights 1/9 (axes) and 1/36
        const float ax = (ph[(size_t)y * W + xm] - c) + (ph[(size_t)y * W + xp] - c) +
                         (ph[(size_t)ym * W + x] - c) + (ph[(size_t)yp * W + x] - c);
        const float dg = (ph[(size_t)ym * W + xm] - c) + (ph[(size_t)ym * W + xp] - c) +
                         (ph[(size_t)yp * W + xm] - c) + (ph[(size_t)yp * W + xp] - c);
        const float lap = 6.0f * fmaf(1.0f / 36.0f, dg, (1.0f / 9.0f) * ax);
        const float rho = fmaf(c, d.rd[b], d.rl[b]);
        const float rp = fmaf(d.beta[b] * 0.25f * d.rd[b], lap, rho);
        const float jx = J[2 * b * n + i], jy = J[(2 * b + 1) * n + i];
        const float u = rp > 0.0f ? sqrtf(jx * jx + jy * jy) / rp : INFINITY;
        m = u > m || u != u ? u : m;
    }
    sred[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < (unsigned)w) {
            const float o = sred[threadIdx.x + w];
            if (o > sred[threadIdx.x] || o != o) sred[threadIdx.x] = o;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[b * gridDim.x + blockIdx.x] = sred[0];
}

// sum of a float field in float64, per block, for sample blockIdx.y of a batch of
// fields of n values: part[sample][block]
__global__ void __launch_bounds__(256) k_sum_field(const float* __restrict__ a, size_t n,
                                                   double* __restrict__ part) {
    __shared__ double sred[256];
    const size_t off = (size_t)blockIdx.y * n;
    double m = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        m += (double)a[off + i];
    sred[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < (unsigned)w) sred[threadIdx.x] += sred[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = sred[0];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned blocks(size_t n) { return (unsigned)((n + 255) / 256); }

template <int NCB, int RW, int NW, int MODE, int EPI, bool BIG = false>
static hipError_t launch_rows_k(const ConvP& a, hipStream_t st) {
    // as many workgroups as are resident at once (2 per CU); each walks a contiguous run of
    // tiles so that the loads of its next tiles overlap the products of the current one
    constexpr int ROWS = 4 / NCB * RW;
    const int ntile = a.B * ((a.H + ROWS - 1) / ROWS) * ((a.W + RPX - 1) / RPX);
    const int nblk_n = a.Cout / (32 * NCB);
    const int per = std::max(1, (ntile * nblk_n + 511) / 512);
    hipLaunchKernelGGL((k_conv_rows<NCB, RW, NW, MODE, EPI, BIG>), dim3((ntile + per - 1) / per, nblk_n),
                       dim3(256), 0, st, a, per);
    return hipGetLastError();
}

template <int NCB, int RW, int MODE, int EPI>
static hipError_t launch_rows_c(const ConvP& a, hipStream_t st) {
    // weights resident for one chunk, or two where the registers allow it
    if (a.g.C == 32) return launch_rows_k<NCB, RW, 1, MODE, EPI>(a, st);
    if constexpr (RW <= 2 && (RW == 1 || (EPI != EPI_HEAD && EPI != EPI_BWD + BWD_SAME &&
                                       EPI != EPI_BWD + BWD_POOL)))
        if (a.g.C == 64) return launch_rows_k<NCB, RW, 2, MODE, EPI>(a, st);
    return launch_rows_k<NCB, RW, 0, MODE, EPI>(a, st);
}

template <int NCB, int MODE, int EPI>
static hipError_t launch_rows_w(const ConvP& a, hipStream_t st) {
    // rows per wave: 4 (one channel block a workgroup: 2, as LDS holds two workgroups of 8
    // rows a CU; 64 input channels: 2, with both chunks' weights resident) where that gives
    // every CU two workgroups, fewer for small batches, whose latency counts (a pooled output
    // and an upsampled input's gradient need pairs of rows in one wave)
    const auto wgs = [&](int rw) {
        const int rows = 4 / NCB * rw;
        return (long)a.B * ((a.H + rows - 1) / rows) * ((a.W + RPX - 1) / RPX) * (a.Cout / (32 * NCB));
    };
    // (a buffer's address arithmetic has 32 bits: images of 4 GiB and more take plain addresses)
    if constexpr (MODE != MODE_POOL)
        if ((double)a.g.Hin * a.g.Win * a.g.cs * 2 >= 4294967296.0)
            return launch_rows_k<NCB, 2, 0, MODE, EPI, true>(a, st);
    if constexpr (NCB == 2)
        if (wgs(4) >= 512 && a.g.C != 64) return launch_rows_c<NCB, 4, MODE, EPI>(a, st);
    if constexpr (EPI != EPI_BWD + BWD_UP)
        if (wgs(2) < 512 && !a.pout) return launch_rows_c<NCB, 1, MODE, EPI>(a, st);
    return launch_rows_c<NCB, 2, MODE, EPI>(a, st);
}

template <int NCB>
static hipError_t launch_rows(const ConvP& a, hipStream_t st) {
    if (a.pout && (a.H % 2 || a.W % 2 || !a.out)) return hipErrorInvalidValue;
    if (a.bwd >= 0) {
        if (a.g.mode != MODE_SAME || !a.zin || !a.dz || a.bias || a.zout || a.out || a.pout ||
            a.head_out || a.dz_c0 % 32 || (a.bwd != BWD_SAME && a.dz_c0) ||
            (a.bwd == BWD_POOL && !a.fout) || (a.dz_c0 && !a.fout) ||
            (a.bwd == BWD_UP && (a.H % 2 || a.W % 2)))
            return hipErrorInvalidValue;
        if (a.bwd == BWD_SAME) return launch_rows_w<NCB, MODE_SAME, EPI_BWD + BWD_SAME>(a, st);
        if (a.bwd == BWD_UP) return launch_rows_w<NCB, MODE_SAME, EPI_BWD + BWD_UP>(a, st);
        return launch_rows_w<NCB, MODE_SAME, EPI_BWD + BWD_POOL>(a, st);
    }
    if (a.head_out) {
        if (NCB != 1 || a.Cout != 32 || a.g.mode != MODE_SAME || a.out || a.zout || a.fout ||
            a.pout || !a.head_w || !a.head_b)
            return hipErrorInvalidValue;
        return launch_rows_w<1, MODE_SAME, EPI_HEAD>(a, st);
    }
    if (a.g.mode == MODE_POOL) return launch_rows_w<NCB, MODE_POOL, EPI_OUT>(a, st);
    if (a.g.mode == MODE_UP) return launch_rows_w<NCB, MODE_UP, EPI_OUT>(a, st);
    return launch_rows_w<NCB, MODE_SAME, EPI_OUT>(a, st);
}

hipError_t conv_stem(const ConvP& a0, const ConvP& a, hipStream_t st) {
    if (a0.g.C != 8 || a0.g.mode != MODE_SAME || a0.Cout != 32 || a.g.C != 32 ||
        a.g.mode != MODE_SAME || a.Cout != 32 || a0.B != a.B || a0.H != a.H || a0.W != a.W ||
        a.H < TP || a.W < TP || !a.out || a.head_out || a.fout || a.zout || a0.zout ||
        (a.pout && (a.H % 2 || a.W % 2)))
        return hipErrorInvalidValue;
    // as many workgroups as are resident at once (2 per CU), each walking a run of tiles
    // with the next tile's input loads in flight during the current tile's work
    const int ntile = a.B * ((a.H + TP - 1) / TP) * ((a.W + TP - 1) / TP);
    const int per = std::max(1, (ntile + 511) / 512);
    hipLaunchKernelGGL(k_conv_stem, dim3((ntile + per - 1) / per), dim3(256), 0, st, a0, a, per);
    return hipGetLastError();
}

hipError_t conv3x3(const ConvP& a, hipStream_t st) {
    if (a.g.C == 8 && a.g.mode == MODE_SAME && a.Cout % 32 == 0) {
        if (a.pout || a.head_out || a.bwd >= 0) return hipErrorInvalidValue;
        const dim3 grid(a.B * ((a.H + TP - 1) / TP) * ((a.W + TP - 1) / TP), a.Cout / 32);
        hipLaunchKernelGGL(k_conv_first, grid, dim3(256), 0, st, a);
        return hipGetLastError();
    }
    // (an image of 64 GiB and more is past the row kernel's offsets)
    if (a.g.C % 32 == 0 && a.Cout % 32 == 0 &&
        (double)a.g.Hin * a.g.Win * (a.g.cs / 8) < 4294967296.0)
        return a.Cout % 64 == 0 ? launch_rows<2>(a, st) : launch_rows<1>(a, st);
    if (a.pout || a.head_out || a.bwd >= 0) return hipErrorInvalidValue;   // only the row kernel fuses
    const int P = a.B * a.H * a.W;
    hipLaunchKernelGGL(k_conv3x3, dim3((P + 255) / 256, (a.Cout + 31) / 32), dim3(256), 0, st, a);
    return hipGetLastError();
}

int wgrad_patches(int B, int H, int W) { return B * ((H + TP - 1) / TP) * ((W + TP - 1) / TP); }

// splits of the patch range: about 512 workgroups in all (2 per CU)
int wgrad_nsplit(int B, int H, int W, int Cout, int Cin, int* per_split) {
    const int np = wgrad_patches(B, H, W);
    const int blocks = ((Cout + 31) / 32) * ((Cin + 31) / 32);
    int ns = (512 + blocks - 1) / blocks;
    if (ns > np) ns = np;
    if (ns < 1) ns = 1;
    const int per = (np + ns - 1) / ns;
    *per_split = per;
    return (np + per - 1) / per;
}

size_t wgrad_part_floats(int B, int H, int W, int Cout, int Cin) {
    int per;
    return (size_t)wgrad_nsplit(B, H, W, Cout, Cin, &per) * ((size_t)Cout * 9 * Cin + Cout);
}

hipError_t wgrad(const WgradP& a, float* dw, float* db, hipStream_t st) {
    int per;
    const int ns = wgrad_nsplit(a.B, a.H, a.W, a.Cout, a.g.C, &per);
    const int np = wgrad_patches(a.B, a.H, a.W);
    const int npair = ((a.Cout + 31) / 32) * ((a.g.C + 31) / 32);
    const dim3 grid(npair * ((ns + 7) / 8) * 8);
    if (a.g.mode == MODE_POOL)
        hipLaunchKernelGGL((k_wgrad_tiled<MODE_POOL>), grid, dim3(256), 0, st, a, per, np, ns);
    else if (a.g.mode == MODE_UP)
        hipLaunchKernelGGL((k_wgrad_tiled<MODE_UP>), grid, dim3(256), 0, st, a, per, np, ns);
    else
        hipLaunchKernelGGL((k_wgrad_tiled<MODE_SAME>), grid, dim3(256), 0, st, a, per, np, ns);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t nw = (size_t)a.Cout * 9 * a.g.C;
    return reduce_splits(a.part, ns, nw + a.Cout, db ? nw + a.Cout : nw, nw, dw, db, st);
}

hipError_t reduce_splits(const float* part, int nsplit, size_t stride, size_t n, size_t nhead,
                         float* out, float* tail, hipStream_t st) {
    hipLaunchKernelGGL(k_reduce_splits, dim3((unsigned)((n + 63) / 64)), dim3(64 * RS_ROWS), 0, st,
                       part, nsplit, stride, n, nhead, out, tail);
    return hipGetLastError();
}

hipError_t head_train(const __bf16* act, const float* wh, const float* bh, const float* y,
                      const __bf16* z, size_t P, __bf16* dz, float* part, double* err,
                      double* loss, hipStream_t st) {
    const unsigned nb = head_blocks(P);
    hipLaunchKernelGGL(k_head_train, dim3(nb), dim3(256), 0, st, act, wh, bh, y, z, P,
                       (float)(P * 4), dz, part, err);
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(256), 0, st, err, (int)nb, loss);
    return hipGetLastError();
}

unsigned head_blocks(size_t P) { return (unsigned)((P + HEAD_PPB - 1) / HEAD_PPB); }

hipError_t adam(float* w, const float* g, float* m, float* v, size_t n, float lr, int t,
                hipStream_t st) {
    // bias corrections from the exact betas, so that at t = 1 they equal the FP32 (1 - beta)
    // factors of the moment updates and m / c1 = g
    const float c1 = (float)(1.0 - pow(0.9, t)), c2 = (float)(1.0 - pow(0.999, t));
    hipLaunchKernelGGL(k_adam, dim3(blocks(n)), dim3(256), 0, st, w, g, m, v, n, lr, c1, c2);
    return hipGetLastError();
}

hipError_t weights_bf16(const float* w, int Cout, int Cin, __bf16* wf, __bf16* wt, hipStream_t st) {
    hipLaunchKernelGGL(k_weights_bf16, dim3(blocks((size_t)Cout * 9 * Cin)), dim3(256), 0, st, w,
                       Cout, Cin, wf, wt);
    return hipGetLastError();
}

hipError_t pack(const float* phi, const float* P, const float* J, const DensTab& d, int B,
                const Norm& nm, size_t HW, __bf16* x, hipStream_t st) {
    if (B < 1 || B > LRR_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pack, dim3(blocks(HW), B), dim3(256), 0, st, phi, P, J, d, nm, HW, x);
    return hipGetLastError();
}

hipError_t pack_target(const float* phi0, const float* P0, const float* J0, const float* phi1,
                       const float* P1, const float* J1, const DensTab& d, int B, const Norm& nm,
                       size_t HW, float* y, hipStream_t st) {
    if (B < 1 || B > LRR_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_pack_target, dim3(blocks(HW), B), dim3(256), 0, st, phi0, P0, J0, phi1,
                       P1, J1, d, nm, HW, y);
    return hipGetLastError();
}

hipError_t apply(const float* out, const Norm& nm, const DensTab& d, int B, size_t HW, float* phi,
                 float* P, float* J, hipStream_t st) {
    if (B < 1 || B > LRR_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_apply, dim3(blocks(HW), B), dim3(256), 0, st, out, nm, d, HW, phi, P, J);
    return hipGetLastError();
}

// grid y is at most 65535: larger batches take several launches
constexpr int MAX_GRID_Y = 65535;

hipError_t maxdiff(const float* a, const float* b, int B, size_t n, float* part, int nblk,
                   hipStream_t st) {
    for (int b0 = 0; b0 < B; b0 += MAX_GRID_Y) {
        const int nb = B - b0 < MAX_GRID_Y ? B - b0 : MAX_GRID_Y;
        hipLaunchKernelGGL(k_maxdiff, dim3(nblk, nb), dim3(256), 0, st, a + b0 * n, b + b0 * n, n,
                           part + (size_t)b0 * nblk);
    }
    return hipGetLastError();
}

hipError_t maxspeed(const float* phi, const float* J, const DensTab& d, int B, int H, int W,
                    float* part, int nblk, hipStream_t st) {
    if (B < 1 || B > LRR_MAX || H < 1 || W < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_maxspeed, dim3(nblk, B), dim3(256), 0, st, phi, J, d, H, W, part);
    return hipGetLastError();
}

hipError_t sum_field(const float* a, int B, size_t n, double* part, int nblk, hipStream_t st) {
    for (int b0 = 0; b0 < B; b0 += MAX_GRID_Y) {
        const int nb = B - b0 < MAX_GRID_Y ? B - b0 : MAX_GRID_Y;
        hipLaunchKernelGGL(k_sum_field, dim3(nblk, nb), dim3(256), 0, st, a + b0 * n, n,
                           part + (size_t)b0 * nblk);
    }
    return hipGetLastError();
}

}  // namespace pfsur
