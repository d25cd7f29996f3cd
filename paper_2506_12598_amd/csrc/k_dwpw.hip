// Depthwise 3 x 3 convolution and the pointwise (1 x 1) layer that reads it, in one launch (16-bit types).
//
// In a small request each of the two is a dispatch, a trip to memory and a few hundred instructions (MobileNetV2 at batch 3: 3.1 and 3.2 us).  Here a
// workgroup owns 16 WM pixels x 16 TN output channels; the K steps of 32 channels are dealt to WK wavefronts, and a lane computes the
// eight depthwise results (one pixel, 8 channels) that it would otherwise have loaded, in the order and with the rounding of
// dwconv_kernel, before they change lanes and enter the matrix instruction as in the wave-split-K kernel.  Every tile column
// computes the depthwise values of its pixels again: the planner takes columns as wide as the compute units allow.
// What bounds it: the chain of one step (9 + 9 loads, 72 multiply-adds and their conversions per lane), one or two of them per
// wavefront, between the dispatch and the sum over wavefronts; with many pixels per compute unit, those instructions.
#include <cstdio>
#include <cstdlib>

#include "gemm_common.h"
#include "kernels.h"

namespace eclip {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

struct DwPwRest {
    const uint16_t *bias_d, *wp, *bias_p, *res;
    uint16_t *y;
    unsigned bias_d_bytes, bias_p_bytes, res_bytes, y_bytes;
    int N, last_nb, act_d, act_p;
    Magic cols;                              // tile columns
};

template <typename T, int TN, int WK, int WM>
__global__ __launch_bounds__(WK * WM * 64) void dwpw_kernel(const uint16_t *x, const uint16_t *wd, int M, int C, int steps, int H, int W, unsigned howo_d, unsigned howo_mul,
                                                            unsigned wo_d, unsigned wo_mul, unsigned packed, DwPwRest p)
{
    constexpr int NW = WK * WM, BM = WM * 16, BN = TN * 16;
    constexpr unsigned OOB = 0xffffffffu;
    extern __shared__ __attribute__((aligned(16))) float red[];    // [WK][WM * TN][64][4]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / WM, wm = wave % WM;
    // an XCD owns a contiguous band of pixels and all columns of it
    const unsigned pos = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const unsigned tile_m = div_by(pos, p.cols), tile_n = pos - tile_m * p.cols.d;
    const int m_base = (int)tile_m * BM, n_base = (int)tile_n * BN;
    if (m_base >= M) return;                 // the grid is a multiple of 8

    const int stride = (int)(packed >> 10 & 255u), pad = (int)(packed >> 18 & 255u);
    const int row = lane >> 2, g = lane & 3, m = m_base + wm * 16 + row;
    const int perm_src = (((lane & 15) << 2) | (lane >> 4)) << 2;
    const unsigned b = div_by((unsigned)m, Magic{howo_d, howo_mul, packed & 31u}), r = (unsigned)m - b * howo_d;
    const unsigned oh = div_by(r, Magic{wo_d, wo_mul, packed >> 5 & 31u}), ow = r - oh * wo_d;
    const int ih0 = (int)oh * stride - pad, iw0 = (int)ow * stride - pad;
    const unsigned px = (unsigned)C * 2u;
    unsigned base = (unsigned)(((int)b * H + ih0) * W + iw0) * px;
    asm volatile("" : "+v"(base));           // one sum per tap from here, not the products again
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, (int)0xfffffffeu, 0x00020000);       // the border tests are exact
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)wd, 0, (int)(9u * px), 0x00020000);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias_d, 0, (int)p.bias_d_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void *)p.wp, 0, (p.last_nb + 1) * steps * 1024, 0x00020000);
    const bool in_m = m < M;
    const bool row_ok[3] = {in_m && (unsigned)ih0 < (unsigned)H, in_m && (unsigned)(ih0 + 1) < (unsigned)H, in_m && (unsigned)(ih0 + 2) < (unsigned)H};
    const bool col_ok[3] = {(unsigned)iw0 < (unsigned)W, (unsigned)(iw0 + 1) < (unsigned)W, (unsigned)(iw0 + 2) < (unsigned)W};
    unsigned at[9], bad[9];                  // byte offset of every tap's pixel; all ones where that lies in the padding
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        at[t] = base + (unsigned)((t / 3) * W + t % 3) * px;
        bad[t] = row_ok[t / 3] && col_ok[t % 3] ? 0u : OOB;
    }
    char *taps = reinterpret_cast<char *>(red) + wave * 1024;          // this wavefront's part; the sums come later

    f32x4 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto lo = [](unsigned q) { return Cvt<T>::from_bits(q & 0xffffu); };
    auto hi = [](unsigned q) { return Cvt<T>::from_bits(q >> 16); };
    for (int ks = wk; ks < steps; ks += WK) {
        const unsigned c16 = (unsigned)ks * 64u + (unsigned)g * 16u;
        const unsigned none = c16 < px ? 0u : OOB;                     // channels beyond C: zeros throughout
        u32x4 xq[9], wf[TN];
        // the nine taps' weights of the step's channels: lane (row, g) fetches tap `row`, everybody reads them back from LDS
        const u32x4 wt = __builtin_amdgcn_raw_buffer_load_b128(rw, row < 9 ? (c16 + (unsigned)row * px) | none : OOB, 0, 0);
#pragma unroll
        for (int t = 0; t < 9; ++t) xq[t] = __builtin_amdgcn_raw_buffer_load_b128(rx, ((at[t] + c16) | bad[t]) | none, 0, 0);
        const u32x4 bq = __builtin_amdgcn_raw_buffer_load_b128(rd, c16 | none, 0, 0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            wf[j] = __builtin_amdgcn_raw_buffer_load_b128(rp, (unsigned)lane * 16u, (min((n_base >> 4) + j, p.last_nb) * steps + ks) * 1024, 0);
        *reinterpret_cast<u32x4 *>(taps + row * 64 + g * 16) = wt;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        u32x4 wq[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) wq[t] = *reinterpret_cast<const u32x4 *>(taps + t * 64 + g * 16);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float o[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[2 * i] = lo(bq[i]); o[2 * i + 1] = hi(bq[i]); }
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                o[2 * i] = fmaf(lo(xq[t][i]), lo(wq[t][i]), o[2 * i]);
                o[2 * i + 1] = fmaf(hi(xq[t][i]), hi(wq[t][i]), o[2 * i + 1]);
            }
        activate(p.act_d, [&](auto f) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = f(o[e]);
        });
        uint4 a;
        a.x = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)Cvt<T>::pack2(o[0], o[1]));
        a.y = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)Cvt<T>::pack2(o[2], o[3]));
        a.z = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)Cvt<T>::pack2(o[4], o[5]));
        a.w = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)Cvt<T>::pack2(o[6], o[7]));
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j] = Mma<T>::run(make_uint4(wf[j].x, wf[j].y, wf[j].z, wf[j].w), a, acc[j]);
    }

    // ---- sum over the WK wavefronts, as in the wave-split-K kernel: 4 channels of one row per thread
    constexpr int SLOTS = (TN + WK - 1) / WK, C4 = TN * 4;
    const bool sums = TN >= WK || wave < WM * TN;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias_p, 0, (int)p.bias_p_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)p.res, 0, (int)p.res_bytes, 0x00020000);
    u32x2 bias[SLOTS], res[SLOTS];
    unsigned off[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, rr_ = s / C4, mm = m_base + rr_, n = n_base + c4 * 4;
        const bool in = sums && rr_ < BM && mm < M && n < p.N;
        off[u] = in ? (unsigned)(mm * p.N + n) * 2u : OOB;
        bias[u] = __builtin_amdgcn_raw_buffer_load_b64(rb, in ? n * 2 : OOB, 0, 0);
        res[u] = __builtin_amdgcn_raw_buffer_load_b64(rr, off[u], 0, 0);
    }
    float4 *red4 = reinterpret_cast<float4 *>(red);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    if constexpr (TN > 1) __syncthreads();   // a wavefront's sums lie where others read their taps
    {
        const int q = lane >> 4, r16 = lane & 15;
#pragma unroll
        for (int j = 0; j < TN; ++j)
            red4[((wk * WM + wm) * TN + j) * 64 + q * 16 + (r16 ^ (j * 4 + q))] = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    }
    __syncthreads();
    if (!sums) return;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, rr_ = s / C4;
        const int from = ((rr_ >> 4) * TN + (c4 >> 2)) * 64 + (c4 & 3) * 16 + ((rr_ & 15) ^ c4);
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WK; ++w) {
            const float4 v = red4[w * WM * TN * 64 + from];
            o[0] += v.x; o[1] += v.y; o[2] += v.z; o[3] += v.w;
        }
        o[0] += lo(bias[u].x) + lo(res[u].x); o[1] += hi(bias[u].x) + hi(res[u].x);
        o[2] += lo(bias[u].y) + lo(res[u].y); o[3] += hi(bias[u].y) + hi(res[u].y);
        activate(p.act_p, [&](auto f) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f(o[e]);
        });
        const u32x2 v = {Cvt<T>::pack2(o[0], o[1]), Cvt<T>::pack2(o[2], o[3])};
        __builtin_amdgcn_raw_buffer_store_b64(v, ry, off[u], 0, 0);
    }
}

template <typename T, int TN> const void *kernel_of(int wk, int wm)
{
    switch (wk * 16 + wm) {
    case 1 * 16 + 4: return (const void *)dwpw_kernel<T, TN, 1, 4>;
    case 2 * 16 + 2: return (const void *)dwpw_kernel<T, TN, 2, 2>;
    case 4 * 16 + 1: return (const void *)dwpw_kernel<T, TN, 4, 1>;
    case 8 * 16 + 1: return (const void *)dwpw_kernel<T, TN, 8, 1>;
    default: return nullptr;
    }
}
template <typename T> const void *kernel_of(int tn, int wk, int wm)
{
    return tn == 1 ? kernel_of<T, 1>(wk, wm) : tn == 2 ? kernel_of<T, 2>(wk, wm) : tn == 4 ? kernel_of<T, 4>(wk, wm) : nullptr;
}

}  // namespace

// Fitted to 142 problems (MobileNetV2's and ShuffleNet's pairs, M 49 to 100352, 32 to 256 CUs, both types) x 7 to 15 shapes in chains of pairs, us
// a pair: a dispatch and the ends of the kernel, a trip to memory per step of a wavefront, and per CU the steps' instructions (bf16 converts more) and
// the sums.  10 % rms.  Two launches are priced by the bytes and products of both.  Picks cost 2.7 % more than the better of fused and apart on
// average, and 16 % less than always apart (f16, 128 CUs: M 37632, C 32, N 16: 13.5 apart, 7.7 fused; 6272, 192, 32: 9.8, 7.5; 392, 960, 160: 8.7, 7.9;
// left apart, since every column repeats the depthwise values: 6272, 96, 384: 12.3, 15.9).  16 wavefronts sharing K won nowhere.
bool dwpw_plan(long M, int C, int N, int dtype, int n_cu, DwPwPlan *out)
{
    const int steps = (C + 31) / 32;
    double best = 1e30;
    for (int wk : {1, 2, 4, 8}) {
        if (steps < 3 ? wk > steps : wk < 4 || (wk == 8 && steps < 6)) continue;
        const int wm = wk >= 4 ? 1 : 4 / wk;
        for (int tn : {4, 2, 1}) {
            const double tiles = (double)((M + 16 * wm - 1) / (16 * wm)) * ((N + 16 * tn - 1) / (16 * tn)), r = tiles / n_cu;
            const double per_cu = 0.5 * ((r > 1.0 ? r : 1.0) + (double)(long)(r + 1.0 - 1e-9)), slow = dtype == DT_BF16 ? 1.15 : 1.0;
            const double cost = 4.44 + 0.27 * slow * ((steps + wk - 1) / wk) + per_cu * (wm * steps * (0.0618 * slow + 0.0035 * tn) + wk * wm * (0.0324 + 0.0267 * tn));
            if (cost < best) {
                best = cost;
                *out = DwPwPlan{tn, wk, wm};
            }
        }
    }
    if (const char *f = getenv("ECLIP_DWPW")) {              // "channels / 16, wavefronts sharing K"; "0,0": apart; no such shape: the choice above
        int tn = 0, wk = 0;
        if (sscanf(f, "%d,%d", &tn, &wk) == 2) {
            if (tn == 0) return false;
            if ((tn == 1 || tn == 2 || tn == 4) && (wk == 1 || wk == 2 || wk == 4 || wk == 8)) {
                *out = DwPwPlan{tn, wk, wk >= 4 ? 1 : 4 / wk};
                return true;
            }
        }
    }
    const double apart = 7.06 + ((double)M * C * 4.47e-4 + (double)M * N * 1.37e-4 + (double)N * C * 1.26e-4) / n_cu + C * 5.1e-4;
    // The two prices meet 0.25 us apart: timed as served, 500 problems whose prices differ by less than 0.75 us, one launch against two, mean us: where
    // it is priced 0 to 0.125 us higher -0.35, 0.125 to 0.25 -0.08, 0.25 to 0.375 +0.73, beyond +0.4.
    return best < apart + 0.25;
}

hipError_t launch_dwpw(const DwPwArgs &a, const DwPwPlan &pl, hipStream_t s)
{
    const void *k = a.dtype == DT_BF16 ? kernel_of<bf16_t>(pl.tn, pl.wk, pl.wm) : a.dtype == DT_F16 ? kernel_of<f16_t>(pl.tn, pl.wk, pl.wm) : nullptr;
    if (!k) return hipErrorInvalidValue;
    const uint16_t *x = (const uint16_t *)a.x, *wd = (const uint16_t *)a.wd;
    int M = a.B * a.Ho * a.Wo, C = a.C, steps = (a.C + 31) / 32, H = a.H, W = a.W;
    Magic howo = magic_of((unsigned)(a.Ho * a.Wo)), wo = magic_of((unsigned)a.Wo);
    unsigned packed = howo.shift | wo.shift << 5 | (unsigned)a.stride << 10 | (unsigned)a.pad << 18;
    DwPwRest p{};
    p.bias_d = (const uint16_t *)a.bias_d; p.wp = (const uint16_t *)a.wp; p.bias_p = (const uint16_t *)a.bias_p; p.res = (const uint16_t *)a.res;
    p.y = (uint16_t *)a.y;
    p.bias_d_bytes = a.bias_d ? (unsigned)C * 2u : 0u;
    p.bias_p_bytes = a.bias_p ? (unsigned)a.N * 2u : 0u;
    p.y_bytes = (unsigned)M * (unsigned)a.N * 2u;
    p.res_bytes = a.res ? p.y_bytes : 0u;
    p.N = a.N; p.last_nb = (a.N + 15) / 16 - 1; p.act_d = a.act_d; p.act_p = a.act_p;
    const unsigned tiles_m = (unsigned)((M + 16 * pl.wm - 1) / (16 * pl.wm)), cols = (unsigned)((a.N + 16 * pl.tn - 1) / (16 * pl.tn));
    p.cols = magic_of(cols);
    void *args[] = {&x, &wd, &M, &C, &steps, &H, &W, &howo.d, &howo.mul, &wo.d, &wo.mul, &packed, &p};
    return hipLaunchKernel(k, dim3((tiles_m * cols + 7u) & ~7u), dim3((unsigned)(pl.wk * pl.wm) * 64), args, (size_t)pl.wk * pl.wm * pl.tn * 1024, s);
}

}  // namespace eclip
