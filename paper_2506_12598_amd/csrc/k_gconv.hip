// Grouped convolution (1 < groups < channels) on the matrix cores.
//
// A grouped convolution is a dense one whose weight matrix is block-diagonal.  Groups of a few channels are far
// narrower than the 32-deep, 16-wide operands of the matrix instruction, so S neighbouring groups are taken together
// as one "super-group": its S*cig input channels and S*cog output channels form a small dense problem whose weight
// block holds the S group blocks on its diagonal and zeros elsewhere (S is the smallest divisor of `groups` that makes
// S*cig a multiple of 32 and S*cog a multiple of 16, see gconv_mfma_pick).  The zeros are multiplied like any other
// value -- with S = 8 seven eighths of the multiply-adds are wasted -- which is still far cheaper than the scalar
// multiply-adds of the direct kernel: a ResNeXt 3x3 layer at 56x56 is 29 MFLOP of real work.
//
// The weights lie in the 1 KB blocks the matrix instruction consumes: block (sg, nb, t) at ((sg * NB + nb) * KT + t) KB,
// t = tap * (S*cig / 32) + kb.  Read with nb running over all super-groups this is the layout of a dense layer of Cout channels
// and K = taps x S*cig, so the wave-split-K kernel (k_wsk_lean.hip: gconv_mfma_kernel; windows of more than 31 taps: the general form in
// k_wsk.hip) serves it: a tile column only has to know which channels of x its super-group reads.  3 x 3 windows over super-groups of 32
// channels, nine steps in all, have a form that reads a patch of the image from LDS (k_conv3.hip).  A kernel of its own without one, one
// wavefront per 16 pixels x 32 to 64 channels over all of K, took 4.6 us instead of 2.8 to 3.2 at the ResNeXt shapes at batch
// 1 and 2, 11.3 instead of 2.9 at 49 pixels x 960 channels, and 72.7 instead of 57.2 at batch 8 on 32 CUs.
#include "gemm_common.h"
#include "kernels.h"

namespace eclip {

bool gconv_mfma_pick(int groups, int cig, int cog, int *S_out)
{
    for (int S = 1; S <= groups; ++S) {
        if (groups % S) continue;
        if ((S * cig) % 32 == 0 && (S * cog) % 16 == 0) {
            if (S > 16) return false;            // more than 15/16 of the multiply-adds wasted: the direct kernel
            *S_out = S;
            return true;
        }
    }
    return false;
}

// A tile column stays inside one super-group.
GemmPlan gconv_mfma_plan(const GConvArgs &a, int S, int n_cu)
{
    const long M = (long)a.B * a.Ho * a.Wo, K = (long)a.KH * a.KW * S * (a.Cin / a.groups);
    return conv_wsk_plan_columns(M, a.Cout, K, n_cu, a.groups == S ? 0 : S * (a.Cout / a.groups));
}
const char *gconv_mfma_kernel_name(const GConvArgs &a) { return a.KH * a.KW < 32 ? "gconv_mfma_kernel" : "conv_wsk_kernel"; }

hipError_t launch_gconv_mfma(const GConvArgs &a, int S, int n_cu, hipStream_t s)
{
    if (S < 1 || a.groups % S) return hipErrorInvalidValue;
    const int SI = S * (a.Cin / a.groups), SO = S * (a.Cout / a.groups);
    const long M = (long)a.B * a.Ho * a.Wo, xb = (long)a.B * a.H * a.W * a.Cin * 2, wb = (long)(a.Cout / 16) * a.KH * a.KW * (SI / 32) * 1024;
    if (SI % 32 || SO % 16 || a.Cin % 8 || M >= (1L << 30) || xb >= (1L << 32) - 16 || wb >= (1L << 32) - 16) return hipErrorInvalidValue;
    if (a.dtype != DT_BF16 && a.dtype != DT_F16) return hipErrorInvalidValue;
    if (const int blocks = gconv3_blocks(a, S, n_cu)) return launch_gconv3(a, S, blocks, s);
    const GemmPlan pl = gconv_mfma_plan(a, S, n_cu);
    int bm, bn;
    conv_wsk_tile(pl.variant, &bm, &bn);
    GemmDev d{};
    d.x = (const uint16_t *)a.x; d.w = (const uint16_t *)a.w; d.bias = (const uint16_t *)a.bias; d.res = (const uint16_t *)a.res;
    d.y = (uint16_t *)a.y;
    d.B = a.B; d.H = a.H; d.W = a.W; d.Cin = SI; d.Ho = a.Ho; d.Wo = a.Wo; d.KH = a.KH; d.KW = a.KW;
    d.stride = a.stride; d.pad = a.pad; d.act = a.act;
    d.M = (int)M; d.N = a.Cout; d.K = a.KH * a.KW * SI;
    d.x_bytes = (unsigned)xb; d.w_bytes = (unsigned)wb;
    d.n_groups = a.groups / S;
    d.ldx = a.Cin; d.ldy = a.Cout;
    d.tiles_m = (int)((M + bm - 1) / bm); d.tiles_n = (a.Cout + bn - 1) / bn;
    d.splits = 1;
    d.raster = pl.raster;
    d.howo = magic_of((unsigned)(a.Ho * a.Wo));
    d.wo = magic_of((unsigned)a.Wo);
    return launch_conv_wsk(d, a.dtype, pl.variant, pl.nw, pl.tiles, s);
}

}  // namespace eclip
