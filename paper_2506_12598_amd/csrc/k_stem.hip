// First layer of an image model: a convolution of at most 4 channels read from the caller's [B][C][H][W] planes, 16-bit types, and
// optionally the 3 x 3 stride-2 max-pool behind it, in one launch.
//
// As an implicit GEMM over channels-last pixels this layer takes a re-layout launch, pads 3 channels to 8 (7 x 7 x 3 = 147 products become 416) and
// walks window positions per lane.  Here a workgroup brings the patch of the image that its outputs need into LDS once, four channels
// side by side (8 bytes a pixel), and the matrix instruction's operand is read from there as it lies: 32 consecutive k are
// KWP pixels of 32 / (4 KWP) window rows, so a lane's 8 k's are two neighbouring pixels, one LDS read (two where the stride is odd
// and pairs are not 16-byte aligned).  7 x 7: KWP = 8, one K step per window row (224 products); 3 x 3: KWP = 4, two rows per step (64).  What lies
// beyond a smaller window is another window's pixel, not a zero, and an infinite one times its zero weight would be NaN: it is cleared in the
// operand (ResNet's first layer and pool on 128 CUs at batch 1 6.05 -> 6.17 us, at batch 8 14.8 -> 15.4; VGG-16's first layer at batch 8 on 256 15.2 ->
// 15.5; looking whether a workgroup's patch holds such a value at all cost as much as clearing).  The weights lie in registers for the workgroup's life.
// Results go through LDS in the storage type, so that the stores are 16 bytes along the rows and the
// pool, a selection, takes exactly the values that would have been stored between the layers.
// What bounds it: at batch 1 the dispatch and one trip to memory, on larger problems the writes.
#include "device_common.h"
#include "kernels.h"

namespace eclip {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <typename T> __device__ __forceinline__ f32x4 stem_mma(u32x4 a, u32x4 b, f32x4 c)
{
    if constexpr (std::is_same<T, bf16_t>::value)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

struct StemDev {
    const uint16_t *x, *w, *bias;
    uint16_t *y;
    unsigned x_bytes, bias_bytes;
    int C, H, W, KH, KW, Ho, Wo, N, pad, act;
    int Po, Qo;                              // rows and columns of the output (POOL: of the pool)
    Magic tiles, cols, chunks;               // tiles per image, per row of tiles; 16-byte chunks of a pixel's channels
};

// NBLK: K steps of 32; NB: blocks of 16 output channels; S: stride; TH x TW: outputs per workgroup, of the pool with POOL.
// SMALL (KWP == 8): a window of fewer than 7 rows or columns, else only its last column may be missing.  KWP == 4: windows of 3 or 4 rows and columns.
template <typename T, int NBLK, int KWP, int NB, int S, bool POOL, int TH, int TW, bool SMALL>
__global__ __launch_bounds__(256) void stem_kernel(StemDev p)
{
    constexpr unsigned OOB = 0xffffffffu;
    constexpr int CH = POOL ? 2 * TH + 1 : TH, CW = POOL ? 2 * TW + 1 : TW, PIX = CH * CW;      // outputs of the convolution
    constexpr int ROWS = KWP == 8 ? NBLK : 2 * NBLK;                                            // window rows, with the padding
    constexpr int PR = (CH - 1) * S + ROWS, PC = ((CW - 1) * S + KWP + 1) & ~1;                 // the patch, in pixels
    constexpr int LOADS = (PR * PC + 255) / 256, FRAGS = (PIX + 15) / 16, PITCH = NB * 32 + 16; // PITCH: bytes between pixels of the results
    __shared__ __attribute__((aligned(16))) char patch[LOADS * 256 * 8];
    __shared__ __attribute__((aligned(16))) char outs[PIX * PITCH];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned b = div_by(blockIdx.x, p.tiles), t = blockIdx.x - b * p.tiles.d, tr = div_by(t, p.cols), tc = t - tr * p.cols.d;
    const int o_row = (int)tr * TH, o_col = (int)tc * TW;                    // first output
    const int c_row = POOL ? 2 * o_row - 1 : o_row, c_col = POOL ? 2 * o_col - 1 : o_col;
    const int i_row = c_row * S - p.pad, i_col = c_col * S - p.pad;

    // ---- weights of this wavefront's channels, 1 KB per (step, block of 16) in lane order, and the bias as the sums' start
    constexpr int NBW = NB / 2;                                              // two wavefronts share a half of the channels
    const int jb = (wave & 1) * NBW, q4 = lane >> 4, r16 = lane & 15;
    u32x4 wf[NBLK][NBW];
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
#pragma unroll
        for (int j = 0; j < NBW; ++j) wf[k][j] = *reinterpret_cast<const u32x4 *>(p.w + ((k * NB + jb + j) * 64 + lane) * 8);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias, 0, (int)p.bias_bytes, 0x00020000);
    u32x2 bq[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j) bq[j] = __builtin_amdgcn_raw_buffer_load_b64(rb, (unsigned)((jb + j) * 16 + q4 * 4) * 2u, 0, 0);

    // ---- the patch: one pixel per thread and turn, one load per plane
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const unsigned plane = (unsigned)(p.H * p.W) * 2u, image = b * (unsigned)p.C * plane;
    unsigned short px[LOADS][4];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int at = i * 256 + tid, r = at / PC, c = at - r * PC, ih = i_row + r, iw = i_col + c;
        const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W && at < PR * PC;
        const unsigned off = in ? image + (unsigned)(ih * p.W + iw) * 2u : OOB;
#pragma unroll
        for (int q = 0; q < 4; ++q) px[i][q] = __builtin_amdgcn_raw_buffer_load_b16(rx, q < p.C ? off : OOB, (int)((unsigned)q * plane), 0);
    }
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const u32x2 v = {(unsigned)px[i][0] | (unsigned)px[i][1] << 16, (unsigned)px[i][2] | (unsigned)px[i][3] << 16};
        *reinterpret_cast<u32x2 *>(patch + (i * 256 + tid) * 8) = v;
    }
    f32x4 bias[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
        bias[j] = f32x4{Cvt<T>::from_bits(bq[j].x & 0xffffu), Cvt<T>::from_bits(bq[j].x >> 16), Cvt<T>::from_bits(bq[j].y & 0xffffu), Cvt<T>::from_bits(bq[j].y >> 16)};
    __syncthreads();

    // ---- 16 outputs of the convolution per turn of a wavefront; lane (q4, r16) feeds k's 8 q4 .. +7 of output r16
    const int g_row = KWP == 8 ? 0 : q4 >> 1, g_col = KWP == 8 ? 2 * q4 : 2 * (q4 & 1);
    const bool lo_in = g_col < p.KW, hi_in = g_col + 1 < p.KW;               // the lane's two pixels of a window row
    u32x4 a[NBLK];
    auto fetch = [&](int f) {
        const int i = f * 16 + r16, ic = i < PIX ? i : PIX - 1;
        const int r = ic / CW, c = ic - r * CW;
        const char *at = patch + ((r * S + g_row) * PC + c * S + g_col) * 8;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            const char *s = at + k * (ROWS / NBLK) * PC * 8;
            if constexpr (S % 2 == 0) a[k] = *reinterpret_cast<const u32x4 *>(s);
            else {
                const u32x2 lo = *reinterpret_cast<const u32x2 *>(s), hi = *reinterpret_cast<const u32x2 *>(s + 8);
                a[k] = u32x4{lo.x, lo.y, hi.x, hi.y};
            }
        }
    };
    fetch(wave >> 1);
#pragma unroll 1
    for (int f = wave >> 1; f < FRAGS; f += 2) {
        const int i = f * 16 + r16;
        f32x4 acc[NBW];
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            const bool rows = KWP == 8 ? !SMALL || k < p.KH : k == 0 || 2 + g_row < p.KH, lo = rows && (!SMALL || lo_in), hi = rows && hi_in;
            a[k] = u32x4{lo ? a[k].x : 0u, lo ? a[k].y : 0u, hi ? a[k].z : 0u, hi ? a[k].w : 0u};
        }
#pragma unroll
        for (int k = 0; k < NBLK; ++k)
#pragma unroll
            for (int j = 0; j < NBW; ++j) acc[j] = stem_mma<T>(wf[k][j], a[k], k ? acc[j] : bias[j]);
        fetch(f + 2 < FRAGS ? f + 2 : f);                                    // of the next turn, under this one's epilogue
        activate(p.act, [&](auto f) {
#pragma unroll
            for (int j = 0; j < NBW; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[j][e] = f(acc[j][e]);
        });
        if (i < PIX) {
#pragma unroll
            for (int j = 0; j < NBW; ++j) {
                const u32x2 v = {Cvt<T>::pack2(acc[j][0], acc[j][1]), Cvt<T>::pack2(acc[j][2], acc[j][3])};
                *reinterpret_cast<u32x2 *>(outs + i * PITCH + (jb + j) * 32 + q4 * 8) = v;
            }
        }
    }
    __syncthreads();

    // ---- rows of the output, 16 bytes per thread
    auto store = [&](int i, int ch) {
        const int r = i / TW, c = i - r * TW;
        if (o_row + r >= p.Po || o_col + c >= p.Qo) return;
        u32x4 v;
        if constexpr (POOL) {
            // Windows end at the convolution's edge: there they repeat its first or last row and column, as in the pool kernels, so that a window of
            // NaN stays NaN (ResNet on 128 CUs, against outputs of -infinity beyond the edge: batch 1 6.17 -> 6.28 us, batch 8 15.4 -> 14.6).
            float best[8];
            const int rows[3] = {max(2 * r, -c_row), 2 * r + 1, min(2 * r + 2, p.Ho - 1 - c_row)};
            const int cols[3] = {max(2 * c, -c_col), 2 * c + 1, min(2 * c + 2, p.Wo - 1 - c_col)};
#pragma unroll
            for (int u = 0; u < 9; ++u) {
                const u32x4 d = *reinterpret_cast<const u32x4 *>(outs + (rows[u / 3] * CW + cols[u % 3]) * PITCH + ch * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = Cvt<T>::from_bits(d[e] & 0xffffu), hi = Cvt<T>::from_bits(d[e] >> 16);
                    best[2 * e] = u ? fmaxf(best[2 * e], lo) : lo;
                    best[2 * e + 1] = u ? fmaxf(best[2 * e + 1], hi) : hi;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = Cvt<T>::pack2(best[2 * e], best[2 * e + 1]);
        } else {
            v = *reinterpret_cast<const u32x4 *>(outs + i * PITCH + ch * 16);
        }
        const size_t to = (((size_t)b * p.Po + o_row + r) * p.Qo + o_col + c) * (size_t)p.N + (size_t)ch * 8;
        *reinterpret_cast<u32x4 *>(p.y + to) = v;
    };
    if (p.N == NB * 16) {
#pragma unroll
        for (int idx = tid; idx < TH * TW * NB * 2; idx += 256) store(idx / (NB * 2), idx % (NB * 2));
    } else {
        for (int idx = tid; idx < TH * TW * (int)p.chunks.d; idx += 256) {
            const int i = (int)div_by((unsigned)idx, p.chunks);
            store(i, idx - i * (int)p.chunks.d);
        }
    }
}

// window columns with their padding: 4 or 8; 0: too large
int stem_window(int KH, int KW) { return KH <= 4 && KW <= 4 ? 4 : KH <= 7 && KW <= 8 ? 8 : 0; }

struct Tile { int h, w; };
// Outputs per workgroup: the small tiles where the large ones would leave compute units without a workgroup.
constexpr Tile PLAIN[2] = {{8, 16}, {4, 16}}, POOLED[2] = {{4, 8}, {4, 4}};

struct Cut { int Po, Qo; unsigned rows, cols, grid; bool small; Tile tile; };          // outputs, and the tiles they are cut into
Cut cut_of(const StemArgs &a, int n_cu)
{
    Cut c;
    c.Po = a.pool ? (a.Ho - 1) / 2 + 1 : a.Ho;
    c.Qo = a.pool ? (a.Wo - 1) / 2 + 1 : a.Wo;
    for (int k = 0; k < 2; ++k) {
        c.small = k == 1;
        c.tile = (a.pool ? POOLED : PLAIN)[k];
        c.rows = (unsigned)((c.Po + c.tile.h - 1) / c.tile.h);
        c.cols = (unsigned)((c.Qo + c.tile.w - 1) / c.tile.w);
        c.grid = c.rows * c.cols * (unsigned)a.B;
        if (c.grid >= (unsigned)n_cu) break;
    }
    return c;
}

template <typename T, int NBLK, int KWP, int NB, int S, bool SMALL = false>
hipError_t launch(const StemDev &d, bool pool, bool small, unsigned grid, hipStream_t s)
{
    const void *k = pool ? small ? (const void *)stem_kernel<T, NBLK, KWP, NB, S, true, POOLED[1].h, POOLED[1].w, SMALL>
                                 : (const void *)stem_kernel<T, NBLK, KWP, NB, S, true, POOLED[0].h, POOLED[0].w, SMALL>
                         : small ? (const void *)stem_kernel<T, NBLK, KWP, NB, S, false, PLAIN[1].h, PLAIN[1].w, SMALL>
                                 : (const void *)stem_kernel<T, NBLK, KWP, NB, S, false, PLAIN[0].h, PLAIN[0].w, SMALL>;
    StemDev arg = d;
    void *args[] = {&arg};
    return hipLaunchKernel(k, dim3(grid), dim3(256), args, 0, s);
}
template <typename T>
hipError_t launch(const StemArgs &a, const StemDev &d, bool small, unsigned grid, hipStream_t s)
{
    const bool wide = stem_window(a.KH, a.KW) == 8, many = a.N > 32;
    if (wide && (a.KH < 7 || a.KW < 7)) return many ? launch<T, 7, 8, 4, 2, true>(d, a.pool, small, grid, s) : launch<T, 7, 8, 2, 2, true>(d, a.pool, small, grid, s);
    if (wide) return many ? launch<T, 7, 8, 4, 2>(d, a.pool, small, grid, s) : launch<T, 7, 8, 2, 2>(d, a.pool, small, grid, s);
    if (a.stride == 2) return many ? launch<T, 2, 4, 4, 2>(d, a.pool, small, grid, s) : launch<T, 2, 4, 2, 2>(d, a.pool, small, grid, s);
    return many ? launch<T, 2, 4, 4, 1>(d, a.pool, small, grid, s) : launch<T, 2, 4, 2, 1>(d, a.pool, small, grid, s);
}

}  // namespace

bool stem_supported(int C, int KH, int KW, int stride, int N)
{
    const int w = stem_window(KH, KW);
    return C >= 1 && C <= 4 && w && KH * KW >= 9 && (stride == 2 || (stride == 1 && w == 4)) && N % 8 == 0 && N <= 64;
}
size_t stem_weight_elems(int KH, int KW, int N) { return (size_t)(stem_window(KH, KW) == 8 ? 7 : 2) * (N > 32 ? 4 : 2) * 512; }
long stem_weight_source(int KH, int KW, int N, int C, size_t at)
{
    const int kwp = stem_window(KH, KW), nb = N > 32 ? 4 : 2;
    const int e = (int)(at % 8), lane = (int)(at / 8 % 64), j = (int)(at / 512 % nb), k = (int)(at / 512 / nb), g = lane >> 4;
    const int n = 16 * j + (lane & 15), c = e & 3, kh = kwp == 8 ? k : 2 * k + (g >> 1), kw = (kwp == 8 ? 2 * g : 2 * (g & 1)) + (e >> 2);
    if (n >= N || c >= C || kh >= KH || kw >= KW) return -1;
    return (((long)n * C + c) * KH + kh) * KW + kw;
}

unsigned stem_workgroups(const StemArgs &a, int n_cu, uint32_t *tile_m, uint32_t *tile_n)
{
    const Cut c = cut_of(a, n_cu);
    *tile_m = (uint32_t)(c.tile.h * c.tile.w);
    *tile_n = a.N > 32 ? 64u : 32u;
    return c.grid;
}

hipError_t launch_stem(const StemArgs &a, int n_cu, hipStream_t s)
{
    StemDev d{};
    d.x = (const uint16_t *)a.x; d.w = (const uint16_t *)a.w; d.bias = (const uint16_t *)a.bias; d.y = (uint16_t *)a.y;
    d.x_bytes = (unsigned)((size_t)a.B * a.C * a.H * a.W * 2);
    d.bias_bytes = a.bias ? (unsigned)a.N * 2u : 0u;
    d.C = a.C; d.H = a.H; d.W = a.W; d.KH = a.KH; d.KW = a.KW; d.Ho = a.Ho; d.Wo = a.Wo; d.N = a.N; d.pad = a.pad; d.act = a.act;
    const Cut c = cut_of(a, n_cu);
    d.Po = c.Po; d.Qo = c.Qo;
    d.tiles = magic_of(c.rows * c.cols); d.cols = magic_of(c.cols); d.chunks = magic_of((unsigned)a.N / 8);
    if (a.dtype == DT_BF16) return launch<bf16_t>(a, d, c.small, c.grid, s);
    if (a.dtype == DT_F16) return launch<f16_t>(a, d, c.small, c.grid, s);
    return hipErrorInvalidValue;
}

}  // namespace eclip
