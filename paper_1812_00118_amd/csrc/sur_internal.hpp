// Host-side declarations shared by the surrogate's C-ABI layer and its kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pfsur {

// how a convolution reads its input relative to its output resolution
enum { MODE_SAME = 0, MODE_UP = 1, MODE_POOL = 2 };

// channels [c0, c0 + C) of a BF16 NHWC tensor [B][Hin][Win][cs]
struct GatherP {
    const __bf16* p;
    int Hin, Win;
    int cs, c0, C;
    int mode;
};

// out[p, co] for p over B x H x W output pixels, co < Cout; weights [Cout][9][C] BF16, or (packed)
// in the order weights_bf16 lays them out in (C and Cout multiples of 32).
// Epilogue: v = acc + bias; zout (BF16 [P][Cout]) <- v; out (BF16 at channel stride
// out_cs, offset out_c0) <- act ? silu(v) : v; fout (FP32 at f_cs, f_c0) <- v;
// pout (BF16 [B][H/2][W/2][pout_cs], channels from 0; needs out and even H, W) <- the 2x2
// average of what out receives, as the pooling gather computes it.  head_out (FP32
// [P][4]; 32-channel same-resolution layers only) <- the 1x1 head (head_w [4][32],
// head_b [4]) applied to the BF16-rounded activations, as in training.
// bwd >= 0 (input gradients; -1 elsewhere): the output is a gradient of activations, and what
// is stored is dz = (that gradient) silu'(zin) of the layer that produced them, BF16 at
// channel stride dz_cs, of the output channels from dz_c0 on (see tile_epilogue_bwd).
enum { BWD_SAME = 0, BWD_UP = 1, BWD_POOL = 2 };
struct ConvP {
    GatherP g;
    int B, H, W;
    const __bf16* w;
    int packed;
    int Cout;
    const float* bias;
    int act;
    __bf16* zout;
    __bf16* out;
    int out_cs, out_c0;
    float* fout;
    int f_cs, f_c0;
    __bf16* pout;
    int pout_cs;
    const float* head_w;
    const float* head_b;
    float* head_out;
    int bwd;
    const __bf16* zin;
    __bf16* dz;
    int dz_cs, dz_c0;
};

// sums over pixels of dz[p, co] in[p + off(tap), ci] and of dz[p, co]; part: wgrad_part_floats
// floats of partial sums
struct WgradP {
    GatherP g;
    int B, H, W;
    const __bf16* dz;
    int Cout;
    float* part;
};

struct Norm {
    float shift[4], scale[4], out_scale[4], lrr_scale;
};

// per-sample densities of one launch over at most LRR_MAX samples: rho(phi) = rl +
// clamp(phi, 0, 1) rd, and lrr = log10(rho_H / rho_L).  The network sees and predicts
// the velocity J / rho(phi) rather than the momentum J, which spans the density ratio.
constexpr int LRR_MAX = 64;
struct DensTab {
    float rl[LRR_MAX], rd[LRR_MAX], lrr[LRR_MAX];
    float beta[LRR_MAX];   // speed check: 1 if the solver uses Eq. 13's modified density
};

hipError_t conv3x3(const ConvP& a, hipStream_t st);
// the first two layers at inference: a0 the first (8 input channels, its outputs not
// stored), a the second (32 -> 32 channels, same resolution)
hipError_t conv_stem(const ConvP& a0, const ConvP& a, hipStream_t st);
// dw [Cout][9][C] and db [Cout]
hipError_t wgrad(const WgradP& a, float* dw, float* db, hipStream_t st);
size_t wgrad_part_floats(int B, int H, int W, int Cout, int Cin);
// sum over the splits of part[split][i], i < n (rows of `stride`): out[i] for i < nhead, then
// tail[i - nhead]
hipError_t reduce_splits(const float* part, int nsplit, size_t stride, size_t n, size_t nhead,
                         float* out, float* tail, hipStream_t st);
// the head's loss (sum of squared errors), its weight gradient's partial sums (part, 132 per
// block, then 4) and the last layer's dz; err: a double per block of head_blocks
hipError_t head_train(const __bf16* act, const float* wh, const float* bh, const float* y,
                      const __bf16* z, size_t P, __bf16* dz, float* part, double* err,
                      double* loss, hipStream_t st);
unsigned head_blocks(size_t P);
hipError_t adam(float* w, const float* g, float* m, float* v, size_t n, float lr, int t,
                hipStream_t st);
hipError_t weights_bf16(const float* w, int Cout, int Cin, __bf16* wf, __bf16* wt, hipStream_t st);
// B <= LRR_MAX samples each (fields per sample: phi, P [HW], J [2][HW])
hipError_t pack(const float* phi, const float* P, const float* J, const DensTab& d, int B,
                const Norm& nm, size_t HW, __bf16* x, hipStream_t st);
hipError_t pack_target(const float* phi0, const float* P0, const float* J0, const float* phi1,
                       const float* P1, const float* J1, const DensTab& d, int B, const Norm& nm,
                       size_t HW, float* y, hipStream_t st);
hipError_t apply(const float* out, const Norm& nm, const DensTab& d, int B, size_t HW, float* phi,
                 float* P, float* J, hipStream_t st);
hipError_t maxdiff(const float* a, const float* b, int B, size_t n, float* part, int nblk,
                   hipStream_t st);
hipError_t sum_field(const float* a, int B, size_t n, double* part, int nblk, hipStream_t st);
// per block, max over sites of the speed a hand-over to a D2Q9 solver would give,
// |J| / rho'(phi) with rho' = rho_L + phi rho_dif + beta rho_dif lap(phi) / 4 (periodic
// central Laplacian; rho' <= 0 counts as infinite), for sample blockIdx.y of
// B <= LRR_MAX (phi [B][H][W], J [B][2][H][W]): part[sample][block]
hipError_t maxspeed(const float* phi, const float* J, const DensTab& d, int B, int H, int W,
                    float* part, int nblk, hipStream_t st);

}  // namespace pfsur
