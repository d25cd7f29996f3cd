// Host-callable launchers of the gfx950 kernels.  Every launcher validates nothing: the caller
// (the model loader) has already checked shapes, alignment and capacity.  Internal layout of all
// activations is channels-last: [B][H][W][C] for images, [B][S][Hd] for sequences, [B][n] for vectors.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "se_deal.h"

namespace eclip {

enum { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2 };

// ---- implicit-GEMM convolution / linear on the matrix cores (16-bit types) -------------------
// y[m][n] = act(sum_k A[m][k] * w[n][k] + bias[n] + res[m][n]),  m = (b,oh,ow), k = (kh,kw,ci).
struct ConvGemmArgs {
    const void *x;       // [B][H][W][Cin]           Cin % 8 == 0
    const void *w;       // W[n][k], n = cout, k = (kh, kw, ci), in 1 KB blocks of 16 n x 32 k: block (nb, kb) at
                         // (nb * ceil(K/32) + kb) * 1 KB, lane l of a block = W[16 nb + (l & 15)][32 kb + 8 (l >> 4) .. +7];
                         // rows beyond Cout and k beyond K are zero
    const void *bias;    // [Cout] or null
    const void *res;     // [M][Cout] or null
    void *y;             // [M][Cout] in the model dtype, or null when y32 is used
    float *y32;          // [M][Cout] float output, or null
    float *ws;           // split-K partial sums, >= splits*M*Cout floats when splits > 1
    int B, H, W, Cin, Ho, Wo, Cout, KH, KW, stride, pad, act, dtype;
    int nchw_c = 0;      // > 0: x is [B][nchw_c][H][W] with nchw_c <= 4 real channels, Cin == 8 (wave-split-K plans of conv_gemm_plan_stem only)
    int ldx = 0;         // > 0: elements between consecutive pixels of x (x is the first Cin channels of a wider tensor); a multiple of 8
    int ldy = 0;         // > 0: elements between consecutive rows of y (y points at a channel range of a wider tensor); a multiple of 8,
                         // y 16-byte aligned, res and y32 null
    bool pool = false;   // y is [B][Ho / 2][Wo / 2][Cout], the maxima of 2 x 2 outputs at stride 2 (conv_gemm_pools); Ho and Wo are even: a last row or
                         // column that no window takes is not computed
};
struct GemmPlan {
    int kind;      // 0 = LDS-tiled kernel (large problems), 1 = wave-split-K kernel (few tiles, long K), 2 = 3 x 3 windows from a patch in LDS
    int variant;   // tile shape, see conv_gemm_tile() / conv_wsk_tile() / conv3_tile()
    int splits;    // kind 0: K is cut into this many slices, summed by a second kernel
    int tiles;     // output tiles = workgroups (per slice)
    int nw;        // kinds 1, 2: wavefronts per workgroup, each taking 1/nw of K
    int raster;    // how workgroups walk the tiles: 2 (3) = an XCD owns a contiguous range of tiles counted down the tile columns
                   // (along the tile rows); 1 (kind 0) = 8 x 4 blocks of tiles per XCD.  `tiles` counts the padding of the walk
    double cost = 0.0;   // modelled time, us without the launch; 0: chosen by measurement or forced
};
bool conv_gemm_plan_stem(long M, long N, long K, int n_cu, size_t ws_floats, double stage_us, GemmPlan *out, int even_cu = 0);   // ConvGemmArgs::nchw_c
// Tile ids of the LDS-tiled kernels.  0, 1: 128x128x32, 64x64x64 (4 wavefronts); 3: 256x256x32 (8 wavefronts on the ping-pong
// schedule, both operands in LDS); 5, 8, 13, 15, 16: ping-pong with the weights straight from memory: 256x256x32, 192x128x64, 64x128x64,
// 96x64x64, 96x192x64; 17..31: both operands copied straight into LDS (4 wavefronts): 256x256x32, 256x128x64, 128x256x64, 128x128x64,
// 192x128x64, 128x64x64, 64x128x64, 256x192x32, 192x256x32, 64x64x64; 27, 28: 128x64x32, 128x128x32 (small rings: three or four
// workgroups per CU); 29, 30, 31: 128x256x32, 128x192x32, 192x128x32 (two workgroups per CU; layers of GemmTraits::copied only)
void conv_gemm_tile(int variant, int *bm, int *bn, int *bk);
const char *conv_gemm_kernel_name(int variant);
int conv_gemm_threads(int variant);
enum { CONV_WSK_VARIANTS = 6 };          // 16x64, 32x64, 64x64, 16x16, 16x32, 32x32
void conv_wsk_tile(int variant, int *bm, int *bn);
size_t conv_wsk_lds_bytes(int variant, int nw);
hipError_t conv_gemm_init();   // raises the dynamic LDS limit of the LDS-tiled kernels once per process
hipError_t conv_wsk_init();    // raises the dynamic LDS limit of the wave-split-K kernels once per process
// the address form in which the lean wave-split-K kernel takes a layer (k_wsk_lean.hip; it is priced differently), and two layers in one launch from
// the form of each; -1: the general kernel
int conv_wsk_lean_form(int KH, int KW, int stride, int pad, int Cin, int Cout);
int conv_wsk_lean_pair_form(int form0, int form1);
int conv_wsk_lean_depth(int variant, int nw);         // K steps its wavefronts keep in flight
// What the planner has to know beyond the size of a problem and of its share.
struct GemmTraits {
    bool lean = true;    // the lean form of the wave-split-K kernel takes the layer
    int even_cu = 0;     // CuShare::even_cu of the stream; 0: the same as n_cu
    bool copied = false; // the copied tiles take the layer in a fast address form and with their fast epilogue (conv_gemm_is_copied)
    bool conv3 = false;  // the patch kernel takes the layer (conv3_takes); then its geometry:
    int B = 0, Ho = 0, Wo = 0, Cin = 0, stride = 0;
    bool gelu = false;   // the layer's activation is GELU: arithmetic that tiles with a compute unit to themselves pay after their K loop
};
bool conv_gemm_is_copied(int KH, int KW, int Cin, int Cout);
// Chooses tile shape and K split for a stream restricted to n_cu compute units.
GemmPlan conv_gemm_plan(long M, long N, long K, int n_cu, size_t ws_floats, const GemmTraits &traits = GemmTraits());
// every plan worth timing for a problem (measured plan selection)
std::vector<GemmPlan> conv_gemm_candidates(long M, long N, long K, int n_cu, size_t ws_floats, const GemmTraits &traits = GemmTraits());
double conv_wsk_cost_estimate(long M, long N, long K, int n_cu, int variant, int nw);   // the general form's loop by the planner's model, us
// the wave-split-K shape of the lowest estimate whose tile columns divide `columns` channels (0: any); n_cu: CuShare::even_cu
GemmPlan conv_wsk_plan_columns(long M, long N, long K, int n_cu, int columns);
// *n_launched (optional) is increased by the number of kernels launched (2 when K is split).
bool conv_gemm_pools(const ConvGemmArgs &a, const GemmPlan &p);      // a plan's kernel can take the max-pool behind a layer along
hipError_t launch_conv_gemm(const ConvGemmArgs &a, const GemmPlan &p, const SeDeal &deal, hipStream_t s, uint32_t *n_launched);
// Two layers that do not depend on each other in one launch (wave-split-K kernel only).  conv_gemm_plan_pair takes
// the layers' own plans and returns true, with a common plan for each, when sharing a launch is modelled to pay.
// form0, form1: conv_wsk_lean_form of each; n_cu: CuShare::even_cu of the stream.
bool conv_gemm_plan_pair(const GemmPlan &s0, long M0, long N0, long K0, int form0, const GemmPlan &s1, long M1, long N1, long K1, int form1, int n_cu,
                         GemmPlan *p0, GemmPlan *p1);
hipError_t launch_conv_gemm_pair(const ConvGemmArgs &a0, const GemmPlan &p0, const ConvGemmArgs &a1, const GemmPlan &p1, hipStream_t s,
                                 uint32_t *n_launched);

// ---- 3 x 3 convolutions of small requests from an image patch in LDS (k_conv3.hip) ---------------
enum { CONV3_VARIANTS = 6, CONV3_MAX_LDS = 128 * 1024 };         // output pixels 4x4, 8x4, 8x8 (two widths of 16 and 32 channels each)
bool conv3_takes(int KH, int KW, int stride, int pad, int H, int W, int Cin, int Cout, int ldx);
void conv3_tile(int variant, int *th, int *tw, int *bn);         // output pixels down and across, channels
long conv3_tiles(int variant, int B, int Ho, int Wo, int Cout);
size_t conv3_lds_bytes(int variant, int nw, int stride, int Cin);
bool conv3_launchable(int variant, int nw, const GemmTraits &t, int Cout);
double conv3_cost(int variant, int nw, const GemmTraits &t, long N, int n_cu);           // on the scale of the other plans' costs; n_cu: CuShare::even_cu
hipError_t conv3_init();       // raises the dynamic LDS limit once per process
hipError_t launch_conv3(const ConvGemmArgs &a, int variant, int nw, hipStream_t s);

// ---- first layer of an image model, from the caller's planes (k_stem.hip) -----------------------
struct StemArgs {
    const void *x;       // [B][C][H][W], 16-bit
    const void *w;       // stem_weight_elems in the kernel's order: element `at` is logical weight stem_weight_source(at), -1: zero
    const void *bias;    // [N] or null
    void *y;             // [B][Ho][Wo][N], or with `pool` [B][(Ho + 1) / 2][(Wo + 1) / 2][N]
    int B, C, H, W, Ho, Wo, N, KH, KW, stride, pad, act, dtype;
    bool pool;           // followed by a 3 x 3 max-pool of stride 2 and padding 1
};
bool stem_supported(int C, int KH, int KW, int stride, int N);
size_t stem_weight_elems(int KH, int KW, int N);
long stem_weight_source(int KH, int KW, int N, int C, size_t at);       // index into [N][C][KH][KW]
unsigned stem_workgroups(const StemArgs &a, int n_cu, uint32_t *tile_m, uint32_t *tile_n);       // and a workgroup's outputs x channels
hipError_t launch_stem(const StemArgs &a, int n_cu, hipStream_t s);

// ---- float32 direct convolution / linear (plain FMA) -------------------------------------------
struct ConvF32Args {
    const float *x;      // [B][H][W][Cin]
    const float *w;      // [KH][KW][Cin][Cout]
    const float *bias, *res;
    float *y;            // [M][Cout]
    int B, H, W, Cin, Ho, Wo, Cout, KH, KW, stride, pad, act;
    bool nchw = false;   // x is [B][Cin][H][W]
};
struct ConvF32Plan {
    unsigned workgroups, threads;
    int nw, vec;         // wavefronts per sum, channels per load of x
};
ConvF32Plan conv_f32_plan(const ConvF32Args &a, int n_cu);
hipError_t launch_conv_f32(const ConvF32Args &a, int n_cu, hipStream_t s);

// ---- memory-bound kernels ---------------------------------------------------------------------
struct DwConvArgs {
    const void *x, *w, *bias, *res;   // x [B][H][W][C]; w [KH][KW][C]
    void *y;
    int B, H, W, C, Ho, Wo, KH, KW, stride, pad, act, dtype;
};
int dwconv_pixels_per_thread(const DwConvArgs &a, int n_cu);   // 4 (large 3x3 layers, 16-bit types) or 1
int dwconv_strip_rows(const DwConvArgs &a, int n_cu);          // rows per thread of the strip kernel, or 0
unsigned dwconv_workgroups(const DwConvArgs &a, int n_cu);     // of 256 threads
hipError_t launch_dwconv(const DwConvArgs &a, int n_cu, hipStream_t s);

// depthwise 3x3 and the pointwise layer behind it in one launch (k_dwpw.hip): 16-bit types, C % 8 == 0, N % 4 == 0, stride and pad < 256
struct DwPwArgs {
    const void *x, *wd, *bias_d;             // [B][H][W][C]; [3][3][C]; [C] or null
    const void *wp, *bias_p, *res;           // blocked GEMM layout of an N x C matrix; [N] or null; [B][Ho][Wo][N] or null
    void *y;
    int B, H, W, C, Ho, Wo, N, stride, pad, act_d, act_p, dtype;
};
struct DwPwPlan { int tn, wk, wm; };         // 16 tn output channels; wk wavefronts share K, wm the pixels
bool dwpw_plan(long M, int C, int N, int dtype, int n_cu, DwPwPlan *out);      // false: better apart
hipError_t launch_dwpw(const DwPwArgs &a, const DwPwPlan &p, hipStream_t s);

// pointwise expansion, depthwise 3x3 (padding 1, stride 1 or 2) and pointwise layer in one launch (k_expdw.hip): 16-bit types, Cin and C multiples of 8, N of 4
struct ExpDwArgs {
    const void *x, *we, *bias_e;             // [B][H][W][Cin]; blocked GEMM layout of a C x Cin matrix; [C] or null
    const void *wd, *bias_d;                 // [3][3][C]; [C] or null
    const void *wp, *bias_p, *res;           // blocked GEMM layout of an N x C matrix; [N] or null; [B][Ho][Wo][N] or null
    void *y;
    int B, H, W, Cin, C, Ho, Wo, N, stride, act_e, act_d, act_p, dtype;
};
struct ExpDwPlan { int kmax, tn, nw; };      // steps of 32 input channels held; 16 tn output channels; wavefronts
// false: better apart, or (same_sums false) with other sums than apart; n_cu: CuShare::even_cu
bool expdw_plan(int B, int Ho, int Wo, int Cin, int C, int N, int stride, int n_cu, ExpDwPlan *out, bool same_sums = true);
// Whether its sums are those of the launches that the layers have apart: the expansion's plan and dwpw_plan's
bool expdw_sums_as_apart(int Cin, int C, int N, const GemmPlan &expansion, bool lean, const DwPwPlan &dwpw);
hipError_t expdw_init();       // raises the dynamic LDS limit once per process
hipError_t launch_expdw(const ExpDwArgs &a, const ExpDwPlan &p, hipStream_t s);

// grouped convolution, 1 < groups < C: one thread per output element, weights [Cout][KH][KW][Cin/groups]
struct GConvArgs {
    const void *x, *w, *bias, *res;
    void *y;
    int B, H, W, Cin, Ho, Wo, Cout, KH, KW, stride, pad, groups, act, dtype;
};
hipError_t launch_gconv(const GConvArgs &a, int n_cu, hipStream_t s);
// The same on the matrix cores (k_gconv.hip): S neighbouring groups form a dense block-diagonal problem.  gconv_mfma_pick
// returns false when no S <= 16 dividing `groups` makes S*cig a multiple of 32 and S*cog a multiple of 16; the weights
// must then be in the direct kernel's layout, otherwise in the super-group blocks described in k_gconv.hip.
bool gconv_mfma_pick(int groups, int cig, int cog, int *S_out);
hipError_t launch_gconv_mfma(const GConvArgs &a, int S, int n_cu, hipStream_t s);      // n_cu: CuShare::even_cu of the stream
GemmPlan gconv_mfma_plan(const GConvArgs &a, int S, int n_cu);               // tile and grid launch_gconv_mfma uses
const char *gconv_mfma_kernel_name(const GConvArgs &a);
// its form for 3 x 3 windows over super-groups of 32 channels (k_conv3.hip)
int gconv3_blocks(const GConvArgs &a, int S, int n_cu);
unsigned gconv3_workgroups(const GConvArgs &a, int S, int blocks);
hipError_t launch_gconv3(const GConvArgs &a, int S, int blocks, hipStream_t s);
// y[m][0 .. c0) = a[m][:], y[m][c0 .. c0 + c1) = b[m][:]
hipError_t launch_concat(const void *a, const void *b, void *y, long rows, int c0, int c1, int dtype, hipStream_t s);
// y[m][0 .. c) = x[m][:], rows of y ld channels apart (16-bit types, c and ld multiples of 8)
hipError_t launch_chancopy(const void *x, void *y, long rows, int c, int ld, int dtype, hipStream_t s);
// y[m][j] = x[m][(j % groups) * (c / groups) + j / groups]
hipError_t launch_shuffle(const void *x, void *y, long rows, int c, int groups, int dtype, hipStream_t s);

struct PoolArgs {
    const void *x; void *y;
    int B, H, W, C, Ho, Wo, KH, KW, stride, pad, dtype;
};
hipError_t launch_maxpool(const PoolArgs &a, int n_cu, hipStream_t s);
// mean over HW: x [B][HW][C] -> y [B][C] (model dtype) or y32 (float).  Large HW is cut into parts whose float sums
// go through ws (>= B*parts*C floats) and a second kernel; *n_launched grows by the kernels launched.
int gap_parts(int B, int HW, int C, int n_cu);
hipError_t launch_gap(const void *x, void *y, float *y32, float *ws, size_t ws_floats, int B, int HW, int C, int dtype, int n_cu,
                      hipStream_t s, uint32_t *n_launched);

// global average pool and the linear layer that follows it in one launch (see gapfc_supported):
// x [B][HW][C], w in the blocked GEMM layout of an N x C matrix (float32: [C][N]), y [B][N] (model dtype) or y32 (float)
bool gapfc_supported(int B, int HW, int C, int N, int dtype, int n_cu);
hipError_t launch_gapfc(const void *x, const void *w, const void *bias, void *y, float *y32, int B, int HW, int C, int N, int act,
                        int dtype, int n_cu, hipStream_t s);

struct RowArgs {
    const void *x, *res, *gamma, *beta;
    void *y; float *y32;
    long rows; int width; float eps; int dtype;
};
hipError_t launch_layernorm(const RowArgs &a, int n_cu, hipStream_t s);
hipError_t launch_softmax(const RowArgs &a, int n_cu, hipStream_t s);

struct EltArgs {
    const void *x, *bias, *res; void *y; float *y32;
    long rows; int width; int act; int dtype;
};
hipError_t launch_eltwise(const EltArgs &a, int n_cu, hipStream_t s);

struct EmbedArgs {
    const int32_t *ids; const void *tok, *pos, *typ; void *y;
    int B, S, Hd, vocab, dtype;
};
hipError_t launch_embed(const EmbedArgs &a, int n_cu, hipStream_t s);

// ---- fused attention ---------------------------------------------------------------------------
struct AttnArgs {
    const void *qkv;     // [B][S][3*Hd]
    void *y; float *y32; // [B][S][Hd]
    int B, S, Hd, heads, dtype;
};
size_t attention_lds_bytes(int S, int d);
unsigned attention_workgroups(int B, int S, int heads, int n_cu, uint32_t *threads);
hipError_t launch_attention(const AttnArgs &a, const CuShare &cu, hipStream_t s);
hipError_t attention_init();   // raises the dynamic LDS limit once per process

// ---- layout conversion at the model boundary ------------------------------------------------------
// [B][C][H][W] (model dtype) -> [B][H][W][Cp], channels C..Cp-1 zero
hipError_t launch_nchw_to_nhwc(const void *x, void *y, int B, int C, int H, int W, int Cp, int dtype, hipStream_t s);
// internal [B][H][W][C] -> float32 [B][C][H][W]
hipError_t launch_nhwc_to_nchw_f32(const void *x, float *y, int B, int C, int H, int W, int dtype, hipStream_t s);
// n elements of the model dtype -> float32
hipError_t launch_to_f32(const void *x, float *y, long n, int dtype, hipStream_t s);

// ---- diagnostics -------------------------------------------------------------------------------
hipError_t launch_probe(uint32_t *out, int n_blocks, hipStream_t s);
hipError_t launch_tick(uint32_t *p, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, long n, hipStream_t s);

}  // namespace eclip
