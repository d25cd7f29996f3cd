// Wave-split-K implicit GEMM, the form that nearly every batch-1 layer takes (see k_wsk.hip for the method and for the form that
// takes everything else).
//
// A launch of a batch-1 layer lasts four to six microseconds, of which 1.6 are the dispatch and about 0.7 the weights' way from
// memory.  Cycle stamps in the general form put the rest into the number of instructions that a wavefront issues one after the
// other, four to five cycles each, scalar or vector (two kilobytes of straight code run at that rate the first time too: in a
// chain of layers the code does not arrive late).  The general form spends 1400 bytes of code on the prologue (four integer
// divisions), 250 to 400 on every K step it loads (each lane walks its own window position) and 1600 cycles after the last
// barrier, where bias and residual are fetched one after the other.  Here the host prepares what is uniform (steps per wavefront, magic numbers for the divisions, sizes in bytes), and the
// three address forms need one or three vector instructions per load:
//   ROWS       1 x 1 window, stride 1, no padding: pixel m of the operand is row m; the position along K is the load's scalar offset
//   ROWS_TAIL  the same with K not a multiple of 32: the last step's lanes beyond K load zeros
//   WINDOW     Cin a multiple of 32, at most 31 taps: a K step lies inside one tap, so the tap's offset is a scalar
//              and one bit per row and tap says whether the tap lies inside the image
// Bias and residual are fetched while the K loop waits for its operands, through descriptors of zero bytes when there are
// none; the partial tiles lie in LDS so that the summing threads store whole rows.
// Chains of layers with weights of their own, M x N x K, 256 CUs, us per launch in the general form and in this one: 196 x 128 x 512 4.24,
// 2.37; 3136 x 64 x 256 4.02, 2.58; 128 x 768 x 768 4.16, 3.19; 128 x 3072 x 768 6.03, 4.34; 3 x 3 windows 3136 x 64 x 576 5.07, 3.14 and
// 49 x 512 x 4608 8.02, 6.79.  What is left of the short ones is the dispatch and one trip to memory.  (Without the arguments in
// registers 2.75, 2.91, 3.54, 4.81, 3.60, 7.03.)
#include "gemm_common.h"
#include "kernels.h"

namespace eclip {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

enum { WSK_ROWS, WSK_ROWS_TAIL, WSK_WINDOW, WSK_FORMS };


// n bits from bit `at` on; n < 32
__device__ __forceinline__ unsigned bits_from(int at, int n) { return ((1u << n) - 1u) << (at & 31); }

// One layer as the kernel wants it, in two parts.  The head is what the loads of the K loop need: 14 words of it (with the first
// layer's workgroups) are separate arguments, which the hardware puts into scalar registers before the wavefront starts, where a
// trip to the cold argument block costs 150 to 630 cycles.
struct WskHead {
    const uint16_t *x, *w;
    unsigned x_bytes;
    int M, last_nb, steps;                   // rows; last 16-row block of the weights; K steps of 32
    int px;                                  // bytes between pixels of x
    unsigned walk;                           // bits 0-1: GemmPlan::raster 2 or 3 (0: plain); bits 8-15: shift of the division by inner_d;
                                             // bits 16-23: log2 of the tile columns of a group of channels, 255: not a power of two (group)
    int per;                                 // tiles, of which an XCD owns an eighth in a row
    unsigned inner_d, inner_mul;             // tiles along the other dimension, and the multiplier of the division by them
};
struct WskRest {
    const uint16_t *bias, *res;
    void *y;
    unsigned bias_bytes, res_bytes, y_bytes; // 0 for an absent bias / residual: loads return zeros
    int N, ldy;                              // elements between rows of y
    int act, f32;                            // f32: y holds floats
    int k_tail;                              // ROWS_TAIL: k's of the last step
    Magic group;                             // gconv_mfma_kernel: tile columns of a group
    // WINDOW
    Magic howo, wo, cb;                      // output pixels per image and per row; K steps per tap
    int W, H, KW, KH, stride, pad;
    unsigned taps_col;                       // one bit at the first tap of every window row
    int next_col, next_row;                  // added to the byte offset from a tap's last step to the next tap's first, and at a row's end
};

// GROUPED: the channels fall into groups and a tile column's K runs over its own group's input channels, which are consecutive
// and as many as a window tap has K steps of.
template <typename T, int TM, int TN, int NW, int D, int FORM, bool GROUPED>
__device__ __forceinline__ void wsk_body(float *red, const uint16_t *x, const uint16_t *w, unsigned x_bytes, int M, int last_nb, int steps,
                                         int px, unsigned walk, int per, unsigned inner_d, unsigned inner_mul, int n0,
                                         const WskRest &r0, const WskHead &h1, const WskRest &r1)
{
    constexpr int BM = TM * 16, BN = TN * 16, BLK = TM * TN;
    constexpr unsigned OOB = 0xffffffffu;
    // one launch can carry two independent layers: workgroups 0 .. n0-1 work on the first, the rest on the second
    int bid = (int)blockIdx.x;
    WskRest p = r0;
    if (__builtin_expect(bid >= n0, 0)) {
        bid -= n0;
        x = h1.x; w = h1.w; x_bytes = h1.x_bytes; M = h1.M; last_nb = h1.last_nb; steps = h1.steps; px = h1.px; walk = h1.walk;
        per = h1.per; inner_d = h1.inner_d; inner_mul = h1.inner_mul;
        p = r1;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile_m, tile_n;
    {
        const unsigned dealt = walk & 3u, xcd = dealt ? bid & 7 : 0;
        const unsigned t = dealt ? ((unsigned)per * xcd >> 3) + ((unsigned)bid >> 3) : (unsigned)bid;
        if (dealt && t >= ((unsigned)per * (xcd + 1u) >> 3)) return;
        const unsigned r = div_by(t, Magic{inner_d, inner_mul, walk >> 8 & 255u}), rem = t - r * inner_d;
        tile_m = dealt == 3 ? r : rem;
        tile_n = dealt == 3 ? rem : r;
    }
    const int m_base = tile_m * BM, n_base = tile_n * BN;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, (int)x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)w, 0, (last_nb + 1) * steps * 1024, 0x00020000);

    // this wavefront's K steps
    const int per_wave = (steps + NW - 1) / NW, ks0 = wave * per_wave, n_steps = min(per_wave, steps - ks0);

    // byte offset of the tile's group in a pixel
    unsigned group = 0;
    if constexpr (GROUPED) {
        const unsigned shift = walk >> 16, idx = shift == 255u ? div_by((unsigned)tile_n, p.group) : (unsigned)tile_n >> shift;
        group = idx * (unsigned)(FORM == WSK_WINDOW ? (int)p.cb.d : steps) * 64u;
    }

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
        so = (kh * p.W + kw) * px + cs * 64;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m_base + i * 16 + row;
            const unsigned b = div_by((unsigned)m, p.howo), r = m - b * p.howo.d;
            const unsigned oh = div_by(r, p.wo), ow = r - oh * p.wo.d;
            const int ih = (int)oh * p.stride - p.pad, iw = (int)ow * p.stride - p.pad;
            a_off[i] = (unsigned)(((int)b * p.H + ih) * p.W + iw) * (unsigned)px + (unsigned)g * 16u + group;
            // taps of columns lo_w .. hi_w - 1 and rows lo_h .. hi_h - 1 lie inside the image
            const int lo_w = max(-iw, 0), n_w = max(min(p.W - iw, p.KW) - lo_w, 0);
            const int lo_h = max(-ih, 0), n_h = max(min(p.H - ih, p.KH) - lo_h, 0);
            const unsigned cols = bits_from(lo_w, n_w), rows = p.taps_col & bits_from(lo_h * p.KW, n_h * p.KW);
            bad[i] = m < M ? ~(cols * rows) : ~0u;
        }
    } else {
        so = ks0 * 64;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m_base + i * 16 + row;
            a_off[i] = m < M ? (unsigned)m * (unsigned)px + (unsigned)g * 16u + group : OOB;
        }
    }
    // weights: 1 KB blocks of 16 rows x 32 k in lane order; tile columns beyond the last block read that one again (their results
    // are not stored)
    int b_so[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) b_so[j] = (min((n_base >> 4) + j, last_nb) * steps + ks0) * 1024;
    int tail_in = FORM == WSK_ROWS_TAIL ? steps - 1 - ks0 : 0;       // steps until the ragged one

    struct Frag { uint4 a[TM]; uint4 b[TN]; };
    // Loads the next K step.  runs_on: it may lie beyond the slice; then every lane's offset is beyond the tensor and the scalar
    // offsets are 0, so that nothing is fetched.
    auto load = [&](Frag &f, auto runs_on, int more) {
        unsigned none = 0;
        int so_a = so, so_b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) so_b[j] = b_so[j];
        if constexpr (decltype(runs_on)::value) {
            none = more > 0 ? 0u : OOB;
            so_a = more > 0 ? so : 0;
#pragma unroll
            for (int j = 0; j < TN; ++j) so_b[j] = more > 0 ? b_so[j] : 0;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            u32x4 v;
            if constexpr (FORM == WSK_WINDOW) {
                const unsigned out = (unsigned)__builtin_amdgcn_sbfe((int)bad[i], tap, 1);
                v = __builtin_amdgcn_raw_buffer_load_b128(rx, (a_off[i] + (unsigned)so) | out | none, 0, 0);
            } else if constexpr (FORM == WSK_ROWS_TAIL) {
                v = __builtin_amdgcn_raw_buffer_load_b128(rx, tail_in == 0 && g * 8 >= p.k_tail ? OOB : a_off[i] | none, so_a, 0);
            } else {
                v = __builtin_amdgcn_raw_buffer_load_b128(rx, a_off[i] | none, so_a, 0);
            }
            f.a[i] = make_uint4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, (unsigned)lane * 16u | none, so_b[j], 0);
            f.b[j] = make_uint4(v.x, v.y, v.z, v.w);
            b_so[j] += 1024;
        }
        so += 64;
        if constexpr (FORM == WSK_ROWS_TAIL) --tail_in;
        if constexpr (FORM == WSK_WINDOW) {
            if (--left == 0) {
                asm volatile("");                // stays a branch: as selects it would cost every step 14 scalar instructions
                left = (int)p.cb.d;
                ++tap;
                so += p.next_col;
                if (++kw == p.KW) {
                    asm volatile("");
                    kw = 0;
                    so += p.next_row;
                }
            }
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
        static_for<D>([&](auto dc) { load(f[decltype(dc)::value], std::false_type(), 0); });
        do {
            static_for<D>([&](auto dc) {
                consume(f[decltype(dc)::value]);
                load(f[decltype(dc)::value], std::true_type(), rest - D - decltype(dc)::value);
            });
            rest -= D;
        } while (rest > D);
    } else {
        static_for<D>([&](auto dc) {
            if (decltype(dc)::value < rest) load(f[decltype(dc)::value], std::false_type(), 0);
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
        const bool in = sums && m < M && n < p.N;
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
        activate(p.act, [&](auto f) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f(o[e]);
        });
        if (p.f32) {
            const u32x4 v = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
            __builtin_amdgcn_raw_buffer_store_b128(v, ry, off[u] == OOB ? OOB : off[u] * 2u, 0, 0);
        } else {
            const u32x2 v = {Cvt<T>::pack2(o[0], o[1]), Cvt<T>::pack2(o[2], o[3])};
            __builtin_amdgcn_raw_buffer_store_b64(v, ry, off[u], 0, 0);
        }
    }
}

#define WSK_ARGS                                                                                                                          \
    const uint16_t *x, const uint16_t *w, unsigned x_bytes, int M, int last_nb, int steps, int px, unsigned walk, int per, unsigned inner_d, \
        unsigned inner_mul, int n0, WskRest r0, WskHead h1, WskRest r1
template <typename T, int TM, int TN, int NW, int D, int FORM>
__global__ __launch_bounds__(NW * 64) void conv_wsk_kernel(WSK_ARGS)
{
    extern __shared__ __attribute__((aligned(16))) float red[];    // [NW][TM*TN][64][4]
    wsk_body<T, TM, TN, NW, D, FORM, false>(red, x, w, x_bytes, M, last_nb, steps, px, walk, per, inner_d, inner_mul, n0, r0, h1, r1);
}
// Grouped convolutions whose super-groups (k_gconv.hip) are multiples of a tile's channels, or one: the same, each tile column on
// its own channels of x.
template <typename T, int TM, int TN, int NW, int D, int FORM>
__global__ __launch_bounds__(NW * 64) void gconv_mfma_kernel(WSK_ARGS)
{
    extern __shared__ __attribute__((aligned(16))) float red[];
    wsk_body<T, TM, TN, NW, D, FORM, true>(red, x, w, x_bytes, M, last_nb, steps, px, walk, per, inner_d, inner_mul, n0, r0, h1, r1);
}
#undef WSK_ARGS

// K steps in flight per wavefront: as many as fit about 100 registers (16 wavefronts leave 128 per lane)
template <int TM, int TN, int NW> struct LeanDepth {
    static constexpr int value = (TM + TN) <= 2 ? (NW == 16 ? 8 : 12) : (TM + TN) <= 3 ? (NW == 16 ? 6 : 8) : (TM + TN) <= 4 ? (NW == 16 ? 4 : 6)
                                 : (TM + TN) <= 5 ? (NW == 16 ? 4 : 6) : (TM + TN) <= 6 ? (NW == 16 ? 2 : 4) : 3;
};

WskHead wsk_head(const GemmDev &d, int bm, int bn)
{
    WskHead v{};
    v.x = d.x; v.w = d.w; v.x_bytes = d.x_bytes;
    v.M = d.M; v.last_nb = (d.N + 15) / 16 - 1; v.steps = (d.K + 31) / 32; v.px = d.ldx * 2;
    const int tm = (d.M + bm - 1) / bm, tn = (d.N + bn - 1) / bn;
    v.per = tm * tn;
    const Magic inner = magic_of((unsigned)(d.raster == 3 ? tn : tm));
    v.inner_d = inner.d; v.inner_mul = inner.mul;
    v.walk = (unsigned)d.raster | inner.shift << 8;
    if (d.n_groups > 1) {
        const unsigned columns = (unsigned)(d.N / d.n_groups / bn);
        v.walk |= (columns & (columns - 1) ? 255u : (unsigned)__builtin_ctz(columns)) << 16;
    } else if (d.n_groups == 1) {
        v.walk |= 31u << 16;                 // every tile column is in it
    }
    return v;
}
WskRest wsk_rest(const GemmDev &d, int bn)
{
    WskRest v{};
    v.bias = d.bias; v.res = d.res;
    v.f32 = d.y32 != nullptr;
    v.y = v.f32 ? (void *)d.y32 : (void *)d.y;
    v.bias_bytes = d.bias ? (unsigned)d.N * 2u : 0u;
    v.res_bytes = d.res ? (unsigned)d.M * (unsigned)d.N * 2u : 0u;
    v.y_bytes = ((unsigned)(d.M - 1) * (unsigned)d.ldy + (unsigned)d.N) * (v.f32 ? 4u : 2u);
    v.N = d.N; v.ldy = d.ldy; v.act = d.act;
    v.k_tail = d.K - 32 * ((d.K + 31) / 32 - 1);
    v.group = magic_of((unsigned)(d.n_groups > 1 ? d.N / d.n_groups / bn : 1));
    v.howo = magic_of((unsigned)(d.Ho * d.Wo)); v.wo = magic_of((unsigned)d.Wo); v.cb = magic_of((unsigned)(d.Cin >= 32 ? d.Cin / 32 : 1));
    v.W = d.W; v.H = d.H; v.KW = d.KW; v.KH = d.KH; v.stride = d.stride; v.pad = d.pad;
    for (int k = 0; k < d.KH && k * d.KW < 32; ++k) v.taps_col |= 1u << (k * d.KW);
    v.next_col = d.ldx * 2 - d.Cin * 2;
    v.next_row = (d.W - d.KW) * d.ldx * 2;
    return v;
}

template <typename T, int TM, int TN, int NW>
const void *kernel_of(int form, bool grouped)
{
    constexpr int D = LeanDepth<TM, TN, NW>::value;
    if (grouped) {                               // see conv_wsk_plan_columns
        if constexpr (TM * TN > 8 || NW > 8) return nullptr;
        else if (form == WSK_ROWS) return (const void *)gconv_mfma_kernel<T, TM, TN, NW, D, WSK_ROWS>;
        else if (form == WSK_WINDOW) return (const void *)gconv_mfma_kernel<T, TM, TN, NW, D, WSK_WINDOW>;
        else return nullptr;
    }
    switch (form) {
    case WSK_ROWS: return (const void *)conv_wsk_kernel<T, TM, TN, NW, D, WSK_ROWS>;
    case WSK_ROWS_TAIL: return (const void *)conv_wsk_kernel<T, TM, TN, NW, D, WSK_ROWS_TAIL>;
    default: return (const void *)conv_wsk_kernel<T, TM, TN, NW, D, WSK_WINDOW>;
    }
}
template <typename T, int TM, int TN>
const void *kernel_of(int nw, int form, bool grouped)
{
    switch (nw) {
    case 4: return kernel_of<T, TM, TN, 4>(form, grouped);
    case 8: return kernel_of<T, TM, TN, 8>(form, grouped);
    case 16:
        if constexpr (TM * TN <= 8) return kernel_of<T, TM, TN, 16>(form, grouped);
        return nullptr;                          // 16 partial 64x64 tiles would not fit in LDS
    default: return nullptr;
    }
}
template <typename T>
const void *kernel_of(int variant, int nw, int form, bool grouped)
{
    switch (variant) {
    case 0: return kernel_of<T, 1, 4>(nw, form, grouped);
    case 1: return kernel_of<T, 2, 4>(nw, form, grouped);
    case 2: return kernel_of<T, 4, 4>(nw, form, grouped);
    case 3: return kernel_of<T, 1, 1>(nw, form, grouped);
    case 4: return kernel_of<T, 1, 2>(nw, form, grouped);
    case 5: return kernel_of<T, 2, 2>(nw, form, grouped);
    default: return nullptr;
    }
}

}  // namespace

int conv_wsk_lean_form(int KH, int KW, int stride, int pad, int Cin, int Cout)
{
    GemmDev d{};
    d.KH = KH; d.KW = KW; d.stride = stride; d.pad = pad; d.Cin = Cin; d.N = d.ldy = Cout; d.K = KH * KW * Cin;
    return wsk_lean_form(d);
}
int conv_wsk_lean_depth(int variant, int nw)
{
    static const int depth[CONV_WSK_VARIANTS][2] = {{LeanDepth<1, 4, 8>::value, LeanDepth<1, 4, 16>::value}, {LeanDepth<2, 4, 8>::value, LeanDepth<2, 4, 16>::value},
                                                    {LeanDepth<4, 4, 8>::value, LeanDepth<4, 4, 16>::value}, {LeanDepth<1, 1, 8>::value, LeanDepth<1, 1, 16>::value},
                                                    {LeanDepth<1, 2, 8>::value, LeanDepth<1, 2, 16>::value}, {LeanDepth<2, 2, 8>::value, LeanDepth<2, 2, 16>::value}};
    return depth[variant][nw == 16];
}

// The address form of a layer, or -1 when only the general kernel takes it.  Four output channels per summing thread need N and the
// row pitch of y to be multiples of 4.
int wsk_lean_form(const GemmDev &d)
{
    if (d.nchw_c || d.N % 4 || d.ldy % 4) return -1;
    if (d.KH == 1 && d.KW == 1 && d.stride == 1 && d.pad == 0) return d.K % 32 ? WSK_ROWS_TAIL : WSK_ROWS;
    return d.Cin % 32 == 0 && d.KH * d.KW < 32 ? WSK_WINDOW : -1;
}

// The form that serves two layers of one launch: their common one, or WINDOW, of which ROWS is a case.
int conv_wsk_lean_pair_form(int f0, int f1)
{
    if (f0 == f1) return f0;
    return (f0 == WSK_ROWS || f0 == WSK_WINDOW) && (f1 == WSK_ROWS || f1 == WSK_WINDOW) ? WSK_WINDOW : -1;
}
int wsk_lean_pair_form(const GemmDev &d0, const GemmDev &d1) { return conv_wsk_lean_pair_form(wsk_lean_form(d0), wsk_lean_form(d1)); }

hipError_t wsk_lean_init()
{
    for (int v = 0; v < CONV_WSK_VARIANTS; ++v)
        for (int nw = 4; nw <= 16; nw *= 2)
            for (int form = 0; form < WSK_FORMS; ++form)
                for (const void *k : {kernel_of<bf16_t>(v, nw, form, false), kernel_of<f16_t>(v, nw, form, false), kernel_of<bf16_t>(v, nw, form, true),
                                      kernel_of<f16_t>(v, nw, form, true)}) {
                    if (!k) continue;
                    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
                    if (e != hipSuccess) return e;
                }
    return hipSuccess;
}

hipError_t launch_wsk_lean(GemmDev d0, GemmDev d1, int n0, int dtype, int form, int variant, int nw, int tiles, hipStream_t s)
{
    const void *k = dtype == DT_BF16 ? kernel_of<bf16_t>(variant, nw, form, d0.n_groups > 0) : kernel_of<f16_t>(variant, nw, form, d0.n_groups > 0);
    if (!k) return hipErrorInvalidValue;
    int bm, bn;
    conv_wsk_tile(variant, &bm, &bn);
    // Each XCD takes an eighth of the tiles in a row, counted down the tile columns where the weights are the larger operand and along the tile
    // rows where the activations are: its L2 then fetches an eighth of that operand from the last-level cache, not all of it (a load that hits the
    // XCD's own L2 takes 234 cycles, one that another XCD's fetched 550).  With whole columns (rows) per XCD only where their number divides
    // by 8, 22 kinds of request replayed as graphs took 1.4 % longer on the geometric mean, BERT-base 2 x 100 on 224 CUs 424 us instead of 398, ALBERT
    // 200 on 256 427 instead of 402; always along the rows 2.7 %.  The second layer of a launch starts on XCD 0 too, or keeps the plain order.
    const bool single = n0 == tiles;
    auto deal = [&](GemmDev &d, int first) {
        const int t = d.tiles_m * d.tiles_n;
        if (first % 8) d.raster = 0;
        else if (!d.raster && t >= 16) d.raster = d.N >= d.M ? 2 : 3;
        return d.raster ? (t + 7) & ~7 : t;
    };
    n0 = deal(d0, 0);
    tiles = n0 + (single ? 0 : deal(d1, n0));
    WskHead h0 = wsk_head(d0, bm, bn), h1 = wsk_head(d1, bm, bn);
    WskRest r0 = wsk_rest(d0, bn), r1 = wsk_rest(d1, bn);
    if (d0.n_groups > 1 && d0.N / d0.n_groups % bn) return hipErrorInvalidValue;
    void *args[] = {&h0.x, &h0.w, &h0.x_bytes, &h0.M, &h0.last_nb, &h0.steps, &h0.px, &h0.walk, &h0.per, &h0.inner_d, &h0.inner_mul, &n0, &r0, &h1, &r1};
    return hipLaunchKernel(k, dim3((unsigned)tiles), dim3((unsigned)nw * 64), args, conv_wsk_lds_bytes(variant, nw), s);
}

}  // namespace eclip
