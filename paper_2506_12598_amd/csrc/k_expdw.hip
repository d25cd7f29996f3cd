// An inverted bottleneck in one launch: pointwise expansion, depthwise 3 x 3 and the pointwise layer behind it (16-bit types).
//
// In a small request the expansion is a dispatch of 3 to 7 us whose output, six times as wide as its input, is written only to be read back by the
// depthwise + pointwise launch behind it.  Here a workgroup owns 4 x 4 output pixels and 16 TN output channels.  The pixels that their windows reach (6 x 6,
// or 9 x 9 at stride 2) are brought to LDS once; the hidden channels are dealt to the wavefronts in slices of 32.  A wavefront expands a slice
// over those pixels on the matrix cores, rounds it to the storage type into LDS of its own (zero outside the image: it is the depthwise
// layer's padding), and goes on as dwpw_kernel does: a lane computes eight depthwise values, in that kernel's order and rounding, which change lanes and
// enter the matrix instruction.  Border pixels are expanded again by the neighbouring tiles (48 rows of the matrix instruction for 16 pixels, 96 at
// stride 2).  What bounds it: that chain, one to three slices of it per wavefront, and where workgroups queue the expansion's rounding and activation.
#include <cstdio>
#include <cstdlib>

#include "gemm_common.h"
#include "kernels.h"

namespace eclip {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

struct ExpDwDev {
    const uint16_t *x, *we, *bias_e, *wd, *bias_d, *wp, *bias_p, *res;
    uint16_t *y;
    unsigned x_bytes, we_bytes, wd_bytes, wp_bytes, bias_e_bytes, bias_d_bytes, bias_p_bytes, res_bytes, y_bytes;
    int H, W, Cin, C, Ho, Wo, N, kb_e, steps, last_nb, act_e, act_d, act_p;
    unsigned tiles;
    Magic cols, image, row;                  // tile columns; tiles of an image and of a row of it
};

constexpr int exp_side(int sd) { return 3 * sd + 3; }                  // pixels across that a tile's windows reach
constexpr int exp_blocks(int sd) { return (exp_side(sd) * exp_side(sd) + 15) / 16; }
constexpr int HID_PITCH = 80;                                          // bytes of LDS per pixel of a slice: 64 and a shift of the banks
constexpr int exp_pitch(int kmax) { return kmax * 64 + 16; }
constexpr int exp_hidden_bytes(int sd) { return exp_blocks(sd) * 16 * HID_PITCH + 1024; }         // and the nine taps' weights
constexpr int exp_lds_bytes(int kmax, int tn, int nw, int sd)
{
    const int work = exp_blocks(sd) * 16 * exp_pitch(kmax) + nw * exp_hidden_bytes(sd), sum = nw * tn * 1024;
    return work > sum ? work : sum;
}

template <typename T, int KMAX, int TN, int NW, int SD>
__global__ __launch_bounds__(NW * 64) void expdw_kernel(ExpDwDev p)
{
    constexpr int SIDE = exp_side(SD), PIX = SIDE * SIDE, PB = exp_blocks(SD), PITCH = exp_pitch(KMAX);
    constexpr unsigned OOB = 0xffffffffu;
    extern __shared__ __attribute__((aligned(16))) char lds[];         // patch, then per wavefront its slice and taps; the sums come later
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // an XCD owns a contiguous band of pixels and all columns of it
    const unsigned pos = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (pos >= p.tiles) return;              // the grid is a multiple of 8
    const unsigned tile_m = div_by(pos, p.cols), tile_n = pos - tile_m * p.cols.d;
    const unsigned b = div_by(tile_m, p.image), in_image = tile_m - b * p.image.d, ty = div_by(in_image, p.row), tx = in_image - ty * p.row.d;
    const int oy0 = (int)ty * 4, ox0 = (int)tx * 4, iy0 = oy0 * SD - 1, ix0 = ox0 * SD - 1;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc((void *)p.we, 0, (int)p.we_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rbe = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias_e, 0, (int)p.bias_e_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.wd, 0, (int)p.wd_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias_d, 0, (int)p.bias_d_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (int)p.wp_bytes, 0x00020000);

    const int r16 = lane & 15, q = lane >> 4, row = lane >> 2, g = lane & 3;
    // everything a slice reads from memory, in the order of its use.  (With the next slice's on its way while one is worked on, 3 % faster where
    // units are idle, 9 % slower with 64 to 96 channels, and up to 20 % where registers then halve the wavefronts.)
    struct Slice { u32x4 we[KMAX][2], wt, bq, wf[TN]; u32x2 be[2]; };
    auto fetch = [&](Slice &f, int ks) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                f.we[k][j] = __builtin_amdgcn_raw_buffer_load_b128(re, k < p.kb_e ? (unsigned)((2 * ks + j) * p.kb_e + k) * 1024u + (unsigned)lane * 16u : OOB, 0, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) f.be[j] = __builtin_amdgcn_raw_buffer_load_b64(rbe, (unsigned)(32 * ks + 16 * j + 4 * q) * 2u, 0, 0);
        const unsigned c16 = (unsigned)ks * 64u + (unsigned)g * 16u, px = (unsigned)p.C * 2u, none = c16 < px ? 0u : OOB;
        f.wt = __builtin_amdgcn_raw_buffer_load_b128(rw, row < 9 ? (c16 + (unsigned)row * px) | none : OOB, 0, 0);
        f.bq = __builtin_amdgcn_raw_buffer_load_b128(rd, c16 | none, 0, 0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            f.wf[j] = __builtin_amdgcn_raw_buffer_load_b128(rp, (unsigned)lane * 16u, (min((int)tile_n * TN + j, p.last_nb) * p.steps + ks) * 1024, 0);
    };

    // ---- the patch: row `pixel` holds KMAX * 32 channels, zeros beyond Cin and outside the image
    constexpr int CHUNKS = PB * 16 * KMAX * 4;
    u32x4 pv[(CHUNKS + NW * 64 - 1) / (NW * 64)];
#pragma unroll
    for (int c0 = 0; c0 < CHUNKS; c0 += NW * 64) {
        const int c = c0 + tid, pix = c / (KMAX * 4), k = c - pix * (KMAX * 4);
        const int py = pix / SIDE, iy = iy0 + py, ix = ix0 + pix - py * SIDE;
        const bool ok = pix < PIX && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W && k * 8 < p.Cin;
        pv[c0 / (NW * 64)] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? (unsigned)((((int)b * p.H + iy) * p.W + ix) * p.Cin + k * 8) * 2u : OOB, 0, 0);
    }
#pragma unroll
    for (int c0 = 0; c0 < CHUNKS; c0 += NW * 64) {
        const int c = c0 + tid, pix = c / (KMAX * 4), k = c - pix * (KMAX * 4);
        if (CHUNKS % (NW * 64) == 0 || c < CHUNKS) *reinterpret_cast<u32x4 *>(lds + pix * PITCH + k * 16) = pv[c0 / (NW * 64)];
    }

    char *const hid = lds + PB * 16 * PITCH + wave * exp_hidden_bytes(SD), *const taps = hid + PB * 16 * HID_PITCH;
    const int perm_src = (((lane & 15) << 2) | (lane >> 4)) << 2;
    unsigned inside = 0;                     // bit i: pixel 16 i + r16 of the patch lies in the image
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        const int pix = 16 * i + r16, py = pix / SIDE, iy = iy0 + py, ix = ix0 + pix - py * SIDE;
        inside |= (pix < PIX && (unsigned)iy < (unsigned)p.H && (unsigned)ix < (unsigned)p.W ? 1u : 0u) << i;
    }
    auto lo = [](unsigned v) { return Cvt<T>::from_bits(v & 0xffffu); };
    auto hi = [](unsigned v) { return Cvt<T>::from_bits(v >> 16); };
    f32x4 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();

    for (int ks = wave; ks < p.steps; ks += NW) {
        Slice cur;
        fetch(cur, ks);
        // ---- expansion of 32 channels over the patch; the steps are summed one by one, as the wavefronts of conv_wsk_kernel that have one each
        f32x4 e[PB][2];
#pragma unroll
        for (int i = 0; i < PB; ++i) e[i][0] = e[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
#pragma unroll
            for (int i = 0; i < PB; ++i) {
                const uint4 a = *reinterpret_cast<const uint4 *>(lds + (16 * i + r16) * PITCH + k * 64 + q * 16);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint4 we = make_uint4(cur.we[k][j].x, cur.we[k][j].y, cur.we[k][j].z, cur.we[k][j].w);
                    if constexpr (KMAX == 1) e[i][j] = Mma<T>::run(we, a, e[i][j]);
                    else {
                        const f32x4 v = Mma<T>::run(we, a, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                        for (int c = 0; c < 4; ++c) e[i][j][c] += v[c];
                    }
                }
            }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float b0 = lo(cur.be[j].x), b1 = hi(cur.be[j].x), b2 = lo(cur.be[j].y), b3 = hi(cur.be[j].y);
#pragma unroll
            for (int i = 0; i < PB; ++i) { e[i][j][0] += b0; e[i][j][1] += b1; e[i][j][2] += b2; e[i][j][3] += b3; }
        }
        activate(p.act_e, [&](auto f) {
#pragma unroll
            for (int i = 0; i < PB; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c) e[i][j][c] = f(e[i][j][c]);
        });
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const bool in = inside >> i & 1u;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const unsigned v0 = Cvt<T>::pack2(e[i][j][0], e[i][j][1]), v1 = Cvt<T>::pack2(e[i][j][2], e[i][j][3]);
                *reinterpret_cast<uint2 *>(hid + (16 * i + r16) * HID_PITCH + j * 32 + q * 8) = make_uint2(in ? v0 : 0u, in ? v1 : 0u);
            }
        }
        *reinterpret_cast<u32x4 *>(taps + row * 64 + g * 16) = cur.wt;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- depthwise: pixel `row` of the tile, channels 8 g .. + 7 of the slice
        float o[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[2 * i] = lo(cur.bq[i]); o[2 * i + 1] = hi(cur.bq[i]); }
        const char *const at = hid + ((row >> 2) * SD * SIDE + (row & 3) * SD) * HID_PITCH + g * 16;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const u32x4 xv = *reinterpret_cast<const u32x4 *>(at + (t / 3 * SIDE + t % 3) * HID_PITCH), wv = *reinterpret_cast<const u32x4 *>(taps + t * 64 + g * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                o[2 * i] = fmaf(lo(xv[i]), lo(wv[i]), o[2 * i]);
                o[2 * i + 1] = fmaf(hi(xv[i]), hi(wv[i]), o[2 * i + 1]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();     // read before the next slice overwrites it
        activate(p.act_d, [&](auto f) {
#pragma unroll
            for (int c = 0; c < 8; ++c) o[c] = f(o[c]);
        });
        // channels beyond C, whose weights are zeros, are zeros here: expanded from an infinite pixel they would be NaN
        const bool some = 32 * ks + 8 * g < p.C;
        uint4 a;
        a.x = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, some ? (int)Cvt<T>::pack2(o[0], o[1]) : 0);
        a.y = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, some ? (int)Cvt<T>::pack2(o[2], o[3]) : 0);
        a.z = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, some ? (int)Cvt<T>::pack2(o[4], o[5]) : 0);
        a.w = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, some ? (int)Cvt<T>::pack2(o[6], o[7]) : 0);
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j] = Mma<T>::run(make_uint4(cur.wf[j].x, cur.wf[j].y, cur.wf[j].z, cur.wf[j].w), a, acc[j]);
    }

    // ---- sum over the wavefronts, as in dwpw_kernel: 4 channels of one pixel per thread
    constexpr int SLOTS = (TN + NW - 1) / NW, C4 = TN * 4;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias_p, 0, (int)p.bias_p_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)p.res, 0, (int)p.res_bytes, 0x00020000);
    u32x2 bias[SLOTS], res[SLOTS];
    unsigned off[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, m = s / C4, oy = oy0 + (m >> 2), ox = ox0 + (m & 3), n = (int)tile_n * TN * 16 + c4 * 4;
        const bool in = m < 16 && oy < p.Ho && ox < p.Wo && n < p.N;
        off[u] = in ? (unsigned)((((int)b * p.Ho + oy) * p.Wo + ox) * p.N + n) * 2u : OOB;
        bias[u] = __builtin_amdgcn_raw_buffer_load_b64(rb, in ? n * 2 : OOB, 0, 0);
        res[u] = __builtin_amdgcn_raw_buffer_load_b64(rr, off[u], 0, 0);
    }
    __syncthreads();                         // the sums lie where others read
    float4 *red4 = reinterpret_cast<float4 *>(lds);
#pragma unroll
    for (int j = 0; j < TN; ++j) red4[(wave * TN + j) * 64 + q * 16 + (r16 ^ ((j * 4 + q) & 15))] = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    __syncthreads();
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, m = s / C4;
        if (m >= 16) return;
        const int from = (c4 >> 2) * 64 + (c4 & 3) * 16 + (m ^ (c4 & 15));
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 v = red4[w * TN * 64 + from];
            o[0] += v.x; o[1] += v.y; o[2] += v.z; o[3] += v.w;
        }
        o[0] += lo(bias[u].x) + lo(res[u].x); o[1] += hi(bias[u].x) + hi(res[u].x);
        o[2] += lo(bias[u].y) + lo(res[u].y); o[3] += hi(bias[u].y) + hi(res[u].y);
        activate(p.act_p, [&](auto f) {
#pragma unroll
            for (int c = 0; c < 4; ++c) o[c] = f(o[c]);
        });
        const u32x2 v = {Cvt<T>::pack2(o[0], o[1]), Cvt<T>::pack2(o[2], o[3])};
        __builtin_amdgcn_raw_buffer_store_b64(v, ry, off[u], 0, 0);
    }
}

// steps of 32 input channels that a workgroup holds, tile columns of 16 channels, wavefronts
#define ECLIP_EXPDW(X) X(1, 2, 4) X(1, 4, 4) X(3, 4, 8) X(3, 10, 8)
struct Form { int kmax, tn, nw; };
constexpr Form form_of(int Cin, int N)
{
    return Cin <= 32 ? Form{1, N <= 32 ? 2 : 4, 4} : Form{3, N <= 64 ? 4 : 10, 8};
}
template <typename T> const void *kernel_of(int kmax, int tn, int nw, int sd)
{
#define X(K, N, W)                                                                                                          \
    if (kmax == K && tn == N && nw == W) return sd == 1 ? (const void *)expdw_kernel<T, K, N, W, 1> : (const void *)expdw_kernel<T, K, N, W, 2>;
    ECLIP_EXPDW(X)
#undef X
    return nullptr;
}

}  // namespace

hipError_t expdw_init()
{
#define X(K, N, W)                                                                                                          \
    for (int sd = 1; sd <= 2; ++sd)                                                                                         \
        for (const void *k : {kernel_of<bf16_t>(K, N, W, sd), kernel_of<f16_t>(K, N, W, sd)}) {                              \
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, exp_lds_bytes(K, N, W, sd)); \
            if (e != hipSuccess) return e;                                                                                  \
        }
    ECLIP_EXPDW(X)
#undef X
    return hipSuccess;
}

// One launch against two, device time of six in a row as served from graphs: 71 bottlenecks (nine of MobileNetV2 at images of 224 and 112, and 53 of other
// widths: 8 to 96 input, 32 to 576 hidden, 16 to 512 output channels, both strides) x batch 1, 3 and 8 x 32 to 256 CUs, both types.  Every tile column repeats
// the expansion and the depthwise layer, every tile the border; against that stands a hidden tensor written and read back and a launch.  So the kernel pays
// within bounds on its workgroups (columns counted) per compute unit, which stand where the timings cross.  What the rule takes is 1.16 times faster than
// apart on the geometric mean, 0.97 at worst.  Times faster in one launch, and beyond the line:
// - up to 32 input channels, one column, stride 1: 56 x 56 x 24 1.2 and more up to the 49 that were timed; with 64 hidden channels, which occupy half of the
//   wavefronts, 1.0 to 1.2 up to 6.1 (0.98 at 12, 0.65 at 196).  Stride 2: 1.02 to 1.2 up to 6.1 (0.95 at 9.2); with two slices per wavefront and 64 output channels from 0.19 on
//   (0.95 to 0.99 below).
// - two columns: stride 1 1.05 at 6.1 (0.97 at 9.2), stride 2 1.02 at 3.1 (0.99 at 4.6, 0.5 at 98).  Three to eight: 1.02 to 1.2 at 3.0 (0.93 at 3.06, 0.83 at 4, 0.45
//   at 196), stride 2 1.01 to 1.1 at 1.5 (0.82 at 2.25).  More were not timed.
// - up to 96 input and 64 output channels: stride 1 1.1 at the 4 that were timed (64 to 256 hidden channels: 0.99 to 1.1 from 2.3 on), stride 2 1.03 to 1.2 at 2.0 (0.85 to 0.98
//   at 4), with two slices from 0.19 on (0.93 to 0.99 below).
// - more than 64 output channels: up to 1.0, where they gain 1.05 to 1.3 (0.75 to 0.95 at 1.5); with one slice from 0.25 on (0.98 to 0.99 below), with two from
//   0.375 (0.99 to 1.1; 0.9 to 1.04 at 0.25), with three from 0.5 (1.09; 14 x 14 x 96 at 0.375 0.96) and in one column only (0.88 to 0.98 in two).
// - three slices elsewhere from 0.375 on, 1.02 to 1.3 up to 12 at stride 1 and 4 at stride 2.  Four, in kernels for up to 160 input channels, did not pay: 7 x 7 x 160
//   10.5 us apart, 14.3.
// The timings set the lines alone; besides, the sums have to be those of the launches apart (expdw_sums_as_apart).  Of ten bottlenecks of MobileNetV2 at images of 224, 160
// and 96 x batch 1, 3 and 8 x nine shares x both types that the lines take, 727 of 974 have them; MobileNetV2 at batch 3 on 192 CUs: 187 us apart, 174 with them.
bool expdw_plan(int B, int Ho, int Wo, int Cin, int C, int N, int stride, int n_cu, ExpDwPlan *out, bool same_sums)
{
    if (Cin > 96 || (stride != 1 && stride != 2)) return false;
    const auto [kmax, tn, nw] = form_of(Cin, N);
    *out = ExpDwPlan{kmax, tn, nw};
    if (const char *f = getenv("ECLIP_EXPDW")) {             // 0: apart, 1: one launch; anything else: the choice below
        int take = -1;
        if (sscanf(f, "%d", &take) == 1 && (take == 0 || take == 1)) return take == 1;
    }
    if (!same_sums) return false;
    const int slices = ((C + 31) / 32 + nw - 1) / nw, cols = (N + 16 * tn - 1) / (16 * tn);
    const double per_cu = (double)B * ((Ho + 3) / 4) * ((Wo + 3) / 4) * cols / n_cu;
    if (slices > 3 || cols > (tn == 10 ? 2 : 8) || (slices == 3 && cols > 1)) return false;
    double least, most;
    if (tn == 10) {
        least = slices == 1 ? 0.25 : slices == 2 ? 0.37 : 0.45;
        most = 1.0;
    } else if (slices == 3) {
        least = kmax == 3 ? 0.45 : 0.37;
        most = kmax == 3 ? 1.0 : stride == 1 ? 12.5 : 4.0;
    } else {
        least = stride == 2 && slices == 2 && tn == 4 ? 0.18 : 0.0;
        if (kmax == 3) most = stride == 1 ? 4.0 : 2.0;
        else if (cols == 1) most = stride == 1 && C > 64 ? 50.0 : 6.5;
        else if (cols == 2) most = stride == 1 ? 6.5 : 3.1;
        else most = stride == 1 ? 3.0 : 1.5;
    }
    return per_cu >= least && per_cu <= most;
}

// Outputs are the same bits in one launch and apart where both sum in one order.  The pointwise layer: here and in dwpw_kernel wavefront w of W sums slices w,
// w + W, ... and the wavefronts are added in their order, so W has to be the same, or large enough in both that none has two.  The expansion: one step of 32 input
// channels has no order; up to three are added one by one as conv_wsk_kernel does with a step per wavefront, where the LDS tiles keep one running sum.
// (Without this rule one launch took MobileNetV2's layers of 64 and 96 input channels too, and its outputs differed by 0.04 to 0.1 % of their range.)
bool expdw_sums_as_apart(int Cin, int C, int N, const GemmPlan &expansion, bool lean, const DwPwPlan &dwpw)
{
    const Form f = form_of(Cin, N);
    const int slices = (C + 31) / 32;
    if (dwpw.wk != f.nw && (slices > dwpw.wk || slices > f.nw)) return false;
    if (f.kmax == 1) return expansion.kind == 1 || (expansion.kind == 0 && expansion.splits == 1);
    return expansion.kind == 1 && lean;
}

hipError_t launch_expdw(const ExpDwArgs &a, const ExpDwPlan &pl, hipStream_t s)
{
    const void *k = a.dtype == DT_BF16 ? kernel_of<bf16_t>(pl.kmax, pl.tn, pl.nw, a.stride) : a.dtype == DT_F16 ? kernel_of<f16_t>(pl.kmax, pl.tn, pl.nw, a.stride) : nullptr;
    if (!k || a.Cin > 32 * pl.kmax || a.Cin % 8 || a.C % 8 || a.N % 4) return hipErrorInvalidValue;
    ExpDwDev p{};
    p.x = (const uint16_t *)a.x; p.we = (const uint16_t *)a.we; p.bias_e = (const uint16_t *)a.bias_e; p.wd = (const uint16_t *)a.wd;
    p.bias_d = (const uint16_t *)a.bias_d; p.wp = (const uint16_t *)a.wp; p.bias_p = (const uint16_t *)a.bias_p; p.res = (const uint16_t *)a.res;
    p.y = (uint16_t *)a.y;
    p.H = a.H; p.W = a.W; p.Cin = a.Cin; p.C = a.C; p.Ho = a.Ho; p.Wo = a.Wo; p.N = a.N;
    p.kb_e = (a.Cin + 31) / 32; p.steps = (a.C + 31) / 32; p.last_nb = (a.N + 15) / 16 - 1;
    p.act_e = a.act_e; p.act_d = a.act_d; p.act_p = a.act_p;
    p.x_bytes = (unsigned)((size_t)a.B * a.H * a.W * a.Cin * 2);
    p.we_bytes = (unsigned)((a.C + 15) / 16 * p.kb_e) * 1024u;
    p.wd_bytes = 18u * (unsigned)a.C;
    p.wp_bytes = (unsigned)((p.last_nb + 1) * p.steps) * 1024u;
    p.bias_e_bytes = a.bias_e ? (unsigned)a.C * 2u : 0u;
    p.bias_d_bytes = a.bias_d ? (unsigned)a.C * 2u : 0u;
    p.bias_p_bytes = a.bias_p ? (unsigned)a.N * 2u : 0u;
    p.y_bytes = (unsigned)((size_t)a.B * a.Ho * a.Wo * a.N * 2);
    p.res_bytes = a.res ? p.y_bytes : 0u;
    const unsigned across = (unsigned)(a.Wo + 3) / 4, image = across * ((unsigned)(a.Ho + 3) / 4), cols = (unsigned)(a.N + 16 * pl.tn - 1) / (16u * (unsigned)pl.tn);
    p.cols = magic_of(cols); p.image = magic_of(image); p.row = magic_of(across);
    p.tiles = (unsigned)a.B * image * cols;
    void *args[] = {&p};
    return hipLaunchKernel(k, dim3((p.tiles + 7u) & ~7u), dim3((unsigned)pl.nw * 64), args, (size_t)exp_lds_bytes(pl.kmax, pl.tn, pl.nw, a.stride), s);
}

}  // namespace eclip
