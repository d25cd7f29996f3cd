// Wave-split-K implicit GEMM, the form that nearly every batch-1 layer takes (see k_wsk.hip for the method and for the form that
// takes everything else).
//
// A launch of a batch-1 layer lasts four to six microseconds, of which 1.6 are the dispatch and about 0.7 the weights' way from
// memory.  Cycle stamps in the general form put the rest into instructions: a wavefront issues one vector instruction
// in four to five cycles, the code is cold at every launch and arrives at about a byte per cycle, and the general form spends
// 1400 bytes on the prologue (four integer divisions), 250 to 400 on every K step it loads (each lane walks its own window
// position) and 1600 cycles after the last barrier, where bias, residual and the epilogue's code are fetched one after the
// other.  Here the host prepares what is uniform (steps per wavefront, magic numbers for the divisions, sizes in bytes), and the
// three address forms need one or three vector instructions per load:
//   ROWS       1 x 1 window, stride 1, no padding: pixel m of the operand is row m; the position along K is the load's scalar offset
//   ROWS_TAIL  the same with K not a multiple of 32: the last step's lanes beyond K load zeros
//   WINDOW     Cin a multiple of 32, at most 32 taps: a K step lies inside one tap, so the tap's offset is a scalar
//              and one bit per row and tap says whether the tap lies inside the image
// Bias and residual are fetched while the K loop waits for its operands, through descriptors of zero bytes when there are
// none; the partial tiles lie in LDS so that the summing threads store whole rows.
// Chains of layers with weights of their own, M x N x K, 256 CUs, us per launch in the general form and in this one: 196 x 128 x 512 4.24,
// 2.61; 3136 x 64 x 256 3.96, 2.78; 128 x 768 x 768 4.17, 3.30; 128 x 3072 x 768 6.06, 4.72; 3 x 3 windows 3136 x 64 x 576 5.15, 3.64 and
// 49 x 512 x 4608 8.05, 7.29.  What is left of the short ones is the dispatch and one trip to memory.
#include "gemm_common.h"
#include "kernels.h"

namespace eclip {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

enum { WSK_ROWS, WSK_ROWS_TAIL, WSK_WINDOW, WSK_FORMS };

__device__ __forceinline__ unsigned div_by(unsigned n, const Magic &m) { return __umulhi(n + n, m.mul) >> m.shift; }

// One layer as the kernel wants it.
struct WskDev {
    const uint16_t *x, *w, *bias, *res;
    void *y;
    unsigned x_bytes, w_bytes, bias_bytes, res_bytes, y_bytes;      // 0 for an absent bias / residual: loads return zeros
    int M, N, steps, per_wave;               // K steps of 32, and how many of them a wavefront takes
    int px, ldy;                             // bytes between pixels of x, elements between rows of y
    int act, f32;                            // f32: y holds floats
    int dealt, per, limit;                   // GemmPlan::raster 2 or 3: tile columns (rows) per XCD and in all
    Magic inner;                             // tiles along the other dimension
    int k_tail;                              // ROWS_TAIL: k's of the last step
    // WINDOW
    Magic howo, wo, cb;                      // output pixels per image and per row; K steps per tap
    int W, H, KW, KH, stride, pad, img;      // img: bytes of an image of x
    int next_col, next_row;                  // added to the byte offset from a tap's last step to the next tap's first, and at a row's end
};

// All arguments in scalar registers here, fetched together: left to itself the compiler fetches each where it is needed, four
// trips to a cold cache one after the other.
__device__ __forceinline__ void fetch_now(WskDev &p, int &n0)
{
    asm volatile("" : "+s"(p.x), "+s"(p.w), "+s"(p.bias), "+s"(p.res), "+s"(p.y), "+s"(p.x_bytes), "+s"(p.w_bytes), "+s"(p.bias_bytes), "+s"(p.res_bytes),
                 "+s"(p.y_bytes), "+s"(p.M), "+s"(p.N), "+s"(p.steps), "+s"(p.per_wave), "+s"(p.px), "+s"(p.ldy), "+s"(p.dealt),
                 "+s"(p.per), "+s"(p.limit), "+s"(p.inner.d), "+s"(p.inner.mul), "+s"(p.inner.shift), "+s"(n0));
}

template <typename T, int TM, int TN, int NW, int D, int FORM>
__global__ __launch_bounds__(NW * 64) void conv_wsk_kernel(WskDev p0, WskDev p1, int n0)
{
    extern __shared__ __attribute__((aligned(16))) float red[];    // [NW][TM*TN][64][4]
    constexpr int BM = TM * 16, BN = TN * 16, BLK = TM * TN;
    constexpr unsigned OOB = 0xffffffffu;
    // one launch can carry two independent layers: workgroups 0 .. n0-1 work on p0, the rest on p1
    WskDev p = p0;
    fetch_now(p, n0);
    int bid = (int)blockIdx.x;
    if (__builtin_expect(bid >= n0, 0)) {
        p = p1;
        bid -= n0;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile_m, tile_n;
    {
        const unsigned xcd = p.dealt ? bid & 7 : 0, q = p.dealt ? bid >> 3 : bid;
        const unsigned r = div_by(q, p.inner), rem = q - r * p.inner.d;
        const unsigned a = xcd * (unsigned)p.per + r;
        if (p.dealt && (r >= (unsigned)p.per || a >= (unsigned)p.limit)) return;
        tile_m = p.dealt == 3 ? a : rem;
        tile_n = p.dealt == 3 ? rem : a;
    }
    const int m_base = tile_m * BM, n_base = tile_n * BN;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.w, 0, (int)p.w_bytes, 0x00020000);

    // this wavefront's K steps
    const int ks0 = wave * p.per_wave, n_steps = min(p.per_wave, p.steps - ks0);

    // im2col operand in tile order: lane l takes row l >> 2, 16-byte chunk l & 3 of the step's 64 bytes; it changes lanes before use
    const int row = lane >> 2, g = lane & 3;
    const int perm_src = (((lane & 15) << 2) | (lane >> 4)) << 2;
    unsigned a_off[TM];                      // byte offset of the lane's chunk at K step 0 (of tap 0, modulo 2^32 in the padding)
    unsigned bad[TM];                        // WINDOW: one bit per tap, set where the tap lies outside the image
    int so, tap = 0, kw = 0, left = 0;       // WINDOW: byte offset, tap, its column and its remaining steps; ROWS: byte offset
    if constexpr (FORM == WSK_WINDOW) {
        tap = (int)div_by((unsigned)ks0, p.cb);
        const int cs = ks0 - tap * (int)p.cb.d;
        left = (int)p.cb.d - cs;
        int kh = 0;
        for (kw = tap; kw >= p.KW; kw -= p.KW) ++kh;
        so = (kh * p.W + kw) * p.px + cs * 64;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m_base + i * 16 + row;
            const unsigned b = div_by((unsigned)m, p.howo), r = m - b * p.howo.d;
            const unsigned oh = div_by(r, p.wo), ow = r - oh * p.wo.d;
            const int ih = (int)oh * p.stride - p.pad, iw = (int)ow * p.stride - p.pad;
            a_off[i] = b * (unsigned)p.img + (unsigned)((ih * p.W + iw) * p.px + g * 16);
            // columns lo .. hi of the window lie inside the image's row
            const int lo = max(-iw, 0), hi = min(p.W - iw, p.KW);
            const unsigned cols = hi > lo ? ((2u << (hi - 1)) - 1u) & ~((1u << lo) - 1u) : 0u;
            unsigned ok = 0;
            for (int k = 0; k < p.KH; ++k) ok |= ((unsigned)(ih + k) < (unsigned)p.H ? cols : 0u) << (k * p.KW);
            bad[i] = m < p.M ? ~ok : ~0u;
        }
    } else {
        so = ks0 * 64;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m_base + i * 16 + row;
            a_off[i] = m < p.M ? (unsigned)(m * p.px + g * 16) : OOB;
        }
    }
    // weights: 1 KB blocks of 16 rows x 32 k in lane order; tile columns beyond the last block read that one again (their results
    // are not stored)
    int b_so[TN];
    const int last_nb = ((p.N + 15) >> 4) - 1;
#pragma unroll
    for (int j = 0; j < TN; ++j) b_so[j] = (min((n_base >> 4) + j, last_nb) * p.steps + ks0) * 1024;
    int tail_in = FORM == WSK_ROWS_TAIL ? p.steps - 1 - ks0 : 0;     // steps until the ragged one

    struct Frag { uint4 a[TM]; uint4 b[TN]; };
    // Loads the next K step.  RUNS_ON: the load may lie beyond the slice (its values are then not used); the scalar offsets stay
    // inside the tensors, as the descriptor's bounds are only relied on for the lanes' own offsets.
    const int so_max = (p.steps - 1) * 64, b_max = (int)(p.w_bytes - 1024u);
    auto load = [&](Frag &f, auto runs_on) {
        if constexpr (decltype(runs_on)::value && FORM != WSK_WINDOW) so = min(so, so_max);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            u32x4 v;
            if constexpr (FORM == WSK_WINDOW) {
                const unsigned out = (unsigned)__builtin_amdgcn_sbfe((int)bad[i], tap, 1);
                v = __builtin_amdgcn_raw_buffer_load_b128(rx, (a_off[i] + (unsigned)so) | out, 0, 0);
            } else if constexpr (FORM == WSK_ROWS_TAIL) {
                v = __builtin_amdgcn_raw_buffer_load_b128(rx, tail_in == 0 && g * 8 >= p.k_tail ? OOB : a_off[i], so, 0);
            } else {
                v = __builtin_amdgcn_raw_buffer_load_b128(rx, a_off[i], so, 0);
            }
            f.a[i] = make_uint4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if constexpr (decltype(runs_on)::value) b_so[j] = (int)min((unsigned)b_so[j], (unsigned)b_max);
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16, b_so[j], 0);
            f.b[j] = make_uint4(v.x, v.y, v.z, v.w);
            b_so[j] += 1024;
        }
        so += 64;
        if constexpr (FORM == WSK_ROWS_TAIL) --tail_in;
        if constexpr (FORM == WSK_WINDOW) {
            const bool wrap = --left == 0;
            left = wrap ? (int)p.cb.d : left;
            tap += wrap;
            kw += wrap;
            const bool wrap2 = kw == p.KW;
            kw = wrap2 ? 0 : kw;
            so += (wrap ? p.next_col : 0) + (wrap2 ? p.next_row : 0);
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](const Frag &f) {
        uint4 a[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            a[i].x = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)f.a[i].x);
            a[i].y = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)f.a[i].y);
            a[i].z = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)f.a[i].z);
            a[i].w = (unsigned)__builtin_amdgcn_ds_bpermute(perm_src, (int)f.a[i].w);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::run(f.b[j], a[i], acc[i][j]);
    };

    // A slice of at most D steps is loaded whole; a longer one keeps D steps in flight.
    Frag f[D];
    int rest = n_steps;
    if (__builtin_expect(rest > D, 0)) {
        static_for<D>([&](auto dc) { load(f[decltype(dc)::value], std::false_type()); });
        do {
            static_for<D>([&](auto dc) {
                consume(f[decltype(dc)::value]);
                load(f[decltype(dc)::value], std::true_type());
            });
            rest -= D;
        } while (rest > D);
    } else {
        static_for<D>([&](auto dc) {
            if (decltype(dc)::value < rest) load(f[decltype(dc)::value], std::false_type());
        });
    }

    // the summing thread's outputs: 4 channels of one row, neighbouring threads along the row
    constexpr int SLOTS = (BLK + NW - 1) / NW, C4 = TN * 4;
    const bool sums = BLK >= NW || wave < BLK;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias, 0, (int)p.bias_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)p.res, 0, (int)p.res_bytes, 0x00020000);
    u32x2 bias[SLOTS], res[SLOTS];
    unsigned off[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, r = s / C4;
        const int m = m_base + r, n = n_base + c4 * 4;
        const bool in = sums && m < p.M && n < p.N;
        off[u] = in ? (unsigned)(m * p.ldy + n) * 2u : OOB;
        bias[u] = __builtin_amdgcn_raw_buffer_load_b64(rb, in ? n * 2 : OOB, 0, 0);
        res[u] = __builtin_amdgcn_raw_buffer_load_b64(rr, off[u], 0, 0);
    }

    static_for<D>([&](auto dc) {
        if (decltype(dc)::value < rest) consume(f[decltype(dc)::value]);
    });

    // ---- cross-wavefront sum through LDS.  Lane (q, r) of block (i, j) holds row 16 i + r, channels 16 j + 4 q .. +3; its place in
    // the block is rotated by the column so that a row's columns lie in different banks when the summing threads read along it.
    float4 *red4 = reinterpret_cast<float4 *>(red);
    {
        const int q = lane >> 4, r16 = lane & 15;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
                red4[(wave * BLK + i * TN + j) * 64 + q * 16 + (r16 ^ (j * 4 + q))] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    }
    __syncthreads();
    if (!sums) return;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, r = s / C4;
        const int at = ((r >> 4) * TN + (c4 >> 2)) * 64 + (c4 & 3) * 16 + ((r & 15) ^ c4);
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 v = red4[w * BLK * 64 + at];
            o[0] += v.x; o[1] += v.y; o[2] += v.z; o[3] += v.w;
        }
        o[0] += Cvt<T>::from_bits(bias[u].x & 0xffffu); o[1] += Cvt<T>::from_bits(bias[u].x >> 16);
        o[2] += Cvt<T>::from_bits(bias[u].y & 0xffffu); o[3] += Cvt<T>::from_bits(bias[u].y >> 16);
        o[0] += Cvt<T>::from_bits(res[u].x & 0xffffu); o[1] += Cvt<T>::from_bits(res[u].x >> 16);
        o[2] += Cvt<T>::from_bits(res[u].y & 0xffffu); o[3] += Cvt<T>::from_bits(res[u].y >> 16);
        if (p.act == ACT_GELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = gelu_erf(o[e]);
        } else if (p.act != ACT_NONE) {
            const float top = p.act == ACT_RELU6 ? 6.0f : __builtin_inff();
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fminf(fmaxf(o[e], 0.0f), top);
        }
        if (p.f32) {
            const u32x4 v = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
            __builtin_amdgcn_raw_buffer_store_b128(v, ry, off[u] == OOB ? OOB : off[u] * 2u, 0, 0);
        } else {
            const u32x2 v = {Cvt<T>::pack2(o[0], o[1]), Cvt<T>::pack2(o[2], o[3])};
            __builtin_amdgcn_raw_buffer_store_b64(v, ry, off[u], 0, 0);
        }
    }
}

// K steps in flight per wavefront: as many as fit about 100 registers (16 wavefronts leave 128 per lane)
template <int TM, int TN, int NW> struct LeanDepth {
    static constexpr int value = (TM + TN) <= 2 ? (NW == 16 ? 8 : 12) : (TM + TN) <= 3 ? (NW == 16 ? 6 : 8) : (TM + TN) <= 4 ? (NW == 16 ? 4 : 6)
                                 : (TM + TN) <= 5 ? (NW == 16 ? 4 : 6) : (TM + TN) <= 6 ? (NW == 16 ? 2 : 4) : 3;
};

WskDev wsk_dev(const GemmDev &d, int nw, int bm, int bn)
{
    WskDev v{};
    v.x = d.x; v.w = d.w; v.bias = d.bias; v.res = d.res;
    v.f32 = d.y32 != nullptr;
    v.y = v.f32 ? (void *)d.y32 : (void *)d.y;
    v.x_bytes = d.x_bytes; v.w_bytes = d.w_bytes;
    v.bias_bytes = d.bias ? (unsigned)d.N * 2u : 0u;
    v.res_bytes = d.res ? (unsigned)d.M * (unsigned)d.N * 2u : 0u;
    v.y_bytes = ((unsigned)(d.M - 1) * (unsigned)d.ldy + (unsigned)d.N) * (v.f32 ? 4u : 2u);
    v.M = d.M; v.N = d.N;
    v.steps = (d.K + 31) / 32;
    v.per_wave = (v.steps + nw - 1) / nw;
    v.px = d.ldx * 2; v.ldy = d.ldy; v.act = d.act;
    v.dealt = d.raster;
    const int tm = (d.M + bm - 1) / bm, tn = (d.N + bn - 1) / bn;
    v.limit = d.raster == 3 ? tm : tn;
    v.per = d.raster ? (v.limit + 7) / 8 : 0;
    v.inner = magic_of((unsigned)(d.raster == 3 ? tn : tm));
    v.k_tail = d.K - 32 * (v.steps - 1);
    v.howo = magic_of((unsigned)(d.Ho * d.Wo)); v.wo = magic_of((unsigned)d.Wo); v.cb = magic_of((unsigned)(d.Cin >= 32 ? d.Cin / 32 : 1));
    v.W = d.W; v.H = d.H; v.KW = d.KW; v.KH = d.KH; v.stride = d.stride; v.pad = d.pad;
    v.img = d.H * d.W * v.px;
    v.next_col = v.px - d.Cin * 2;
    v.next_row = (d.W - d.KW) * v.px;
    return v;
}

template <typename T, int TM, int TN, int NW>
const void *kernel_of(int form)
{
    constexpr int D = LeanDepth<TM, TN, NW>::value;
    switch (form) {
    case WSK_ROWS: return (const void *)conv_wsk_kernel<T, TM, TN, NW, D, WSK_ROWS>;
    case WSK_ROWS_TAIL: return (const void *)conv_wsk_kernel<T, TM, TN, NW, D, WSK_ROWS_TAIL>;
    default: return (const void *)conv_wsk_kernel<T, TM, TN, NW, D, WSK_WINDOW>;
    }
}
template <typename T, int TM, int TN>
const void *kernel_of(int nw, int form)
{
    switch (nw) {
    case 4: return kernel_of<T, TM, TN, 4>(form);
    case 8: return kernel_of<T, TM, TN, 8>(form);
    case 16:
        if constexpr (TM * TN <= 8) return kernel_of<T, TM, TN, 16>(form);
        return nullptr;                          // 16 partial 64x64 tiles would not fit in LDS
    default: return nullptr;
    }
}
template <typename T>
const void *kernel_of(int variant, int nw, int form)
{
    switch (variant) {
    case 0: return kernel_of<T, 1, 4>(nw, form);
    case 1: return kernel_of<T, 2, 4>(nw, form);
    case 2: return kernel_of<T, 4, 4>(nw, form);
    case 3: return kernel_of<T, 1, 1>(nw, form);
    case 4: return kernel_of<T, 1, 2>(nw, form);
    case 5: return kernel_of<T, 2, 2>(nw, form);
    default: return nullptr;
    }
}

}  // namespace

// The address form of a layer, or -1 when only the general kernel takes it.  Four output channels per summing thread need N and the
// row pitch of y to be multiples of 4.
int wsk_lean_form(const GemmDev &d)
{
    if (d.nchw_c || d.N % 4 || d.ldy % 4) return -1;
    if (d.KH == 1 && d.KW == 1 && d.stride == 1 && d.pad == 0) return d.K % 32 ? WSK_ROWS_TAIL : WSK_ROWS;
    return d.Cin % 32 == 0 && d.KH * d.KW <= 32 ? WSK_WINDOW : -1;
}

// The form that serves two layers of one launch: their common one, or WINDOW, of which ROWS is a case.
int wsk_lean_pair_form(const GemmDev &d0, const GemmDev &d1)
{
    const int f0 = wsk_lean_form(d0), f1 = wsk_lean_form(d1);
    if (f0 == f1) return f0;
    return (f0 == WSK_ROWS || f0 == WSK_WINDOW) && (f1 == WSK_ROWS || f1 == WSK_WINDOW) ? WSK_WINDOW : -1;
}

hipError_t wsk_lean_init()
{
    for (int v = 0; v < CONV_WSK_VARIANTS; ++v)
        for (int nw = 4; nw <= 16; nw *= 2)
            for (int form = 0; form < WSK_FORMS; ++form)
                for (const void *k : {kernel_of<bf16_t>(v, nw, form), kernel_of<f16_t>(v, nw, form)}) {
                    if (!k) continue;
                    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
                    if (e != hipSuccess) return e;
                }
    return hipSuccess;
}

hipError_t launch_wsk_lean(const GemmDev &d0, const GemmDev &d1, int n0, int dtype, int form, int variant, int nw, int tiles, hipStream_t s)
{
    const void *k = dtype == DT_BF16 ? kernel_of<bf16_t>(variant, nw, form) : kernel_of<f16_t>(variant, nw, form);
    if (!k) return hipErrorInvalidValue;
    int bm, bn;
    conv_wsk_tile(variant, &bm, &bn);
    WskDev p0 = wsk_dev(d0, nw, bm, bn), p1 = &d1 == &d0 ? p0 : wsk_dev(d1, nw, bm, bn);
    void *args[] = {&p0, &p1, &n0};
    return hipLaunchKernel(k, dim3((unsigned)tiles), dim3((unsigned)nw * 64), args, conv_wsk_lds_bytes(variant, nw), s);
}

}  // namespace eclip
