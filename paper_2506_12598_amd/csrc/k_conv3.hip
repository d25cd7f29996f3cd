// 3 x 3 convolutions of small requests from an image patch in LDS (16-bit types, stride 1 or 2, padding 1, Cin a multiple of 32).
//
// What bounds a batch-1 3 x 3 layer is the vector-memory path of a compute unit, some 110 B/ns: ResNet-18's four stages on 128 CUs brought
// 110, 147, 221 and 295 KB through it in the wave-split-K kernel and took 4.4, 4.7, 5.2 and 6.2 us, of which about 3.4 do not depend on the
// bytes.  Half of these are the same pixels again: every one is fetched for each of the nine taps that it lies under.  Here a workgroup owns
// a patch of 4 TH x 4 TW output pixels (TH x TW blocks of the matrix instruction, each 4 x 4 pixels) and 16 TN channels; the input channels are
// dealt to its wavefronts in slices of 32.  A wavefront copies its slice of the patch with its border into LDS (no register, no barrier: nobody
// else reads it), then reads one block of pixels per tap from there.  With the pixels cheap a tile is tall and narrow, which
// leaves the weights, once each, as the traffic.  There is no border test and no change of lanes in the loop: copies from outside the image write
// zeros, and the addresses of the taps are constants.  The sum over wavefronts is that of the wave-split-K kernel.
#include <cstdio>
#include <cstdlib>

#include "gemm_common.h"
#include "kernels.h"

// The compiler calls m0 reserved and warns of every statement that names it; it does take the name as a definition of m0.
#pragma clang diagnostic ignored "-Winline-asm"

namespace eclip {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// 16 bytes per lane from `rsrc` (byte offset voff; zeros beyond its end) to LDS byte lds + 16 * lane; written out because the compiler would wait
// for it before any later LDS read
__device__ __forceinline__ void copy_to_lds(u32x4 rsrc, unsigned voff, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds), "v"(voff), "s"(rsrc) : "memory", "m0");
}

struct Conv3Rest {
    const uint16_t *bias, *res;
    void *y;
    unsigned bias_bytes, res_bytes, y_bytes;
    int ldy, act, Ho, Wo, f32;               // f32: y holds floats
};

// packed: bits 0-1 GemmPlan::raster, 2-6, 7-11 and 12-16 the shifts of the divisions by inner_d, by the patches of an image and by those of a row of
// it; hw: H | W << 16; px_slices: bytes between pixels | slices of 32 channels << 16
// POOL: y holds the maxima of 2 x 2 outputs (ConvGemmArgs::pool).  A form of its own, compiled apart (ECLIP_CONV3_POOL): with the pool as an argument all
// kernels were some 75 instructions longer, about a dozen of them on the way of launches without one.  (ResNet-18 next to itself, 13 of whose 18 launches
// these are, timed in turn: 754 us with the argument and 771 without; 739 before there was a pool and 725 now.  Two runs of one side differ by 2 %.)
template <typename T, int TH, int TW, int TN, int NW, int SD, bool MULTI, bool POOL>
__global__ __launch_bounds__(NW * 64) void conv3_kernel(const uint16_t *x, const uint16_t *w, unsigned packed, int tiles, unsigned inner_d, unsigned inner_mul,
                                                        unsigned hw, unsigned px_slices, unsigned image_d, unsigned image_mul, unsigned row_d, unsigned row_mul,
                                                        Conv3Rest p)
{
    constexpr int TM = TH * TW, BLK = TM * TN, PH = (4 * TH - 1) * SD + 3, PW = (4 * TW - 1) * SD + 3;       // patch with its border
    constexpr int COPIES = (PH * PW * 4 + 63) / 64;                    // of 1 KB, per slice
    constexpr unsigned OOB = 0xffffffffu;
    extern __shared__ __attribute__((aligned(16))) float smem[];       // per wavefront its slices' patches, later [BLK][64][4] sums
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned tile_m, tile_n;
    {
        // an XCD takes an eighth of the tiles in a row, as in the wave-split-K kernel
        const unsigned xcd = blockIdx.x & 7u, t = ((unsigned)tiles * xcd >> 3) + (blockIdx.x >> 3);
        if (t >= ((unsigned)tiles * (xcd + 1u) >> 3)) return;
        const unsigned r = div_by(t, Magic{inner_d, inner_mul, packed >> 2 & 31u}), rem = t - r * inner_d;
        const bool rows = (packed & 3u) == 3u;
        tile_m = rows ? r : rem;
        tile_n = rows ? rem : r;
    }
    const unsigned b = div_by(tile_m, Magic{image_d, image_mul, packed >> 7 & 31u}), in_image = tile_m - b * image_d;
    const unsigned ty = div_by(in_image, Magic{row_d, row_mul, packed >> 12 & 31u}), tx = in_image - ty * row_d;
    const int H = (int)(hw & 0xffffu), W = (int)(hw >> 16), slices = (int)(px_slices >> 16);
    const unsigned px = px_slices & 0xffffu;
    const int oy0 = (int)ty * 4 * TH, ox0 = (int)tx * 4 * TW;
    const int per_wave = MULTI ? (slices + NW - 1) / NW : 1, s0 = wave * per_wave, n_slices = min(per_wave, slices - s0);      // may be 0 or less

    // ---- weights: 1 KB blocks of 16 channels x 32 k in lane order, tap by tap
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)w, 0, (int)0xfffffffeu, 0x00020000);          // never beyond the last block
    u32x4 wf[9][TN];
    const int w_block = (int)tile_n * TN * 9 * slices + s0;
    auto load_w = [&](auto tc, int slice, bool any) {                  // without any, nothing is fetched
        constexpr int t = decltype(tc)::value;
#pragma unroll
        for (int j = 0; j < TN; ++j)
            wf[t][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, any ? (unsigned)lane * 16u : OOB, any ? (w_block + slice + (j * 9 + t) * slices) * 1024 : 0, 0);
    };
    constexpr int EARLY = 3;                 // taps fetched before the patch: their offsets need no vector instruction
    static_for<EARLY>([&](auto tc) { load_w(tc, 0, n_slices > 0); });

    // ---- the patch.  16-byte chunk c of pixel i lies at position c ^ (i / 4 % 4) of its 64 bytes: the 16 pixels of a block then spread over the banks
    const unsigned patch0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float *)smem;
    const int region = max(per_wave * COPIES, BLK) * 1024;             // bytes per wavefront
    const unsigned mine = patch0 + (unsigned)(wave * region);
    u32x4 rx;
    {
        const uint64_t base = (uint64_t)(uintptr_t)x + (uint64_t)b * ((unsigned)(H * W) * px);
        rx.x = (unsigned)base; rx.y = (unsigned)(base >> 32) & 0xffffu; rx.z = (unsigned)(H * W) * px; rx.w = 0x00020000u;
    }
    const unsigned chunk = (unsigned)((lane & 3) ^ (lane >> 4)) * 16u;
    const int iy0 = oy0 * SD - 1, ix0 = ox0 * SD - 1;
    static_for<COPIES>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        const unsigned i = c * 16u + (unsigned)(lane >> 2), py = i / PW, qx = i - py * PW;
        const int iy = iy0 + (int)py, ix = ix0 + (int)qx;
        const bool ok = (unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W && i < PH * PW;
        const unsigned bad = ok && n_slices > 0 ? 0u : OOB;
        const unsigned off = __umul24(__umul24((unsigned)iy, (unsigned)W) + (unsigned)ix, px) + (unsigned)s0 * 64u + chunk;
        if constexpr (MULTI) {
            for (int s = 0; s < n_slices; ++s) copy_to_lds(rx, (off + (unsigned)s * 64u) | bad, mine + (unsigned)((s * COPIES + c) * 1024));
        } else {
            copy_to_lds(rx, off | bad, mine + c * 1024u);
        }
    });
    static_for<9 - EARLY>([&](auto tc) { load_w(std::integral_constant<int, decltype(tc)::value + EARLY>(), 0, n_slices > 0); });

    // ---- the summing thread's outputs: 4 channels of one pixel
    constexpr int SLOTS = (BLK + NW - 1) / NW, C4 = TN * 4;
    const bool sums = BLK >= NW || wave < BLK;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias, 0, (int)p.bias_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)p.res, 0, (int)p.res_bytes, 0x00020000);
    u32x2 bias[SLOTS], res[SLOTS];
    unsigned off[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, r = s / C4, blk = r >> 4;
        const int oy = oy0 + 4 * (blk / TW) + (r >> 2 & 3), ox = ox0 + 4 * (blk % TW) + (r & 3), n = (int)tile_n * TN * 16 + c4 * 4;
        const bool in = sums && blk < TM && oy < p.Ho && ox < p.Wo;
        if constexpr (POOL) off[u] = in && !(r & 5) ? (unsigned)((((int)b * (p.Ho >> 1) + (oy >> 1)) * (p.Wo >> 1) + (ox >> 1)) * p.ldy + n) * 2u : OOB;     // a window's upper left
        else off[u] = in ? (unsigned)((((int)b * p.Ho + oy) * p.Wo + ox) * p.ldy + n) * 2u : OOB;
        bias[u] = __builtin_amdgcn_raw_buffer_load_b64(rb, in ? n * 2 : OOB, 0, 0);
        res[u] = __builtin_amdgcn_raw_buffer_load_b64(rr, off[u], 0, 0);
    }

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // pixel of this lane under tap (0, 0) of block 0, and the byte of its chunk q there and `k` pixels on, k = 4 a + r: 64 k is a constant
    const int r16 = lane & 15, q = lane >> 4, pix0 = (r16 >> 2) * SD * PW + (r16 & 3) * SD;
    const char *const base = reinterpret_cast<const char *>(smem) + wave * region;
    auto at = [&](int k) { return pix0 * 64 + ((q ^ ((((pix0 + (k & 3)) >> 2) + (k >> 2)) & 3)) << 4); };
    // The patch has arrived when no more than what was fetched behind it is on its way (accesses return in order): six taps' weights, bias and
    // residual.  That count has to be what the compiler issues: a fetch that it merged with another or dropped would let this wait end early.
    // None can be: the addresses differ, or their conditions do.  (tests/test_counted_waits.py counts them in the compiled kernels.)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((9 - EARLY) * TN + 2 * SLOTS) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    auto taps = [&](int s, bool more) {
        static_for<9>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int k = (4 * (i / TW) * SD + t / 3) * PW + 4 * (i % TW) * SD + t % 3;
                const uint4 a = *reinterpret_cast<const uint4 *>(base + s * (COPIES * 1024) + at(k) + k * 64);
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::run(make_uint4(wf[t][j].x, wf[t][j].y, wf[t][j].z, wf[t][j].w), a, acc[i][j]);
            }
            if constexpr (MULTI) load_w(tc, s + 1, more);
        });
    };
    if constexpr (MULTI) {
        for (int s = 0; s < n_slices; ++s) taps(s, s + 1 < n_slices);
    } else if (n_slices > 0) {
        taps(0, false);
    }

    // ---- sum over the wavefronts
    float4 *red4 = reinterpret_cast<float4 *>(smem);
    const int region4 = region / 16;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
            red4[wave * region4 + (i * TN + j) * 64 + q * 16 + (r16 ^ (j * 4 + q))] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (!sums) return;
    auto lo = [](unsigned v) { return Cvt<T>::from_bits(v & 0xffffu); };
    auto hi = [](unsigned v) { return Cvt<T>::from_bits(v >> 16); };
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int s = u * NW * 64 + tid, c4 = s % C4, r = s / C4;
        const int from = ((r >> 4) * TN + (c4 >> 2)) * 64 + (c4 & 3) * 16 + ((r & 15) ^ c4);
        if (BLK % NW && (r >> 4) >= TM) return;
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            const float4 part = red4[v * region4 + from];
            o[0] += part.x; o[1] += part.y; o[2] += part.z; o[3] += part.w;
        }
        o[0] += lo(bias[u].x); o[1] += hi(bias[u].x); o[2] += lo(bias[u].y); o[3] += hi(bias[u].y);
        o[0] += lo(res[u].x); o[1] += hi(res[u].x); o[2] += lo(res[u].y); o[3] += hi(res[u].y);
        activate(p.act, [&](auto f) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f(o[e]);
        });
        if (p.f32) {
            const u32x4 v = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
            __builtin_amdgcn_raw_buffer_store_b128(v, ry, off[u] == OOB ? OOB : off[u] * 2u, 0, 0);
        } else {
            if constexpr (POOL)                  // pixels one to the right and one down lie C4 and 4 C4 lanes on; all lanes of the wavefront are here
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = __float_as_int(o[e]);
                    o[e] = fmaxf(o[e], __int_as_float(TN == 2 ? __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true)             // row_ror:8
                                                              : __builtin_amdgcn_ds_swizzle(v, 4 << 10 | 0x1f)));              // lane ^ 4
                    const unsigned m = __float_as_uint(o[e]);
                    const u32x2 both = TN == 2 ? __builtin_amdgcn_permlane32_swap(m, m, false, false) : __builtin_amdgcn_permlane16_swap(m, m, false, false);
                    o[e] = fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));
                }
            const u32x2 v = {Cvt<T>::pack2(o[0], o[1]), Cvt<T>::pack2(o[2], o[3])};
            __builtin_amdgcn_raw_buffer_store_b64(v, ry, off[u], 0, 0);
        }
    }
}

#ifndef ECLIP_CONV3_POOL
// Grouped convolutions whose super-groups (k_gconv.hip) read 32 channels: nine steps of the matrix instruction are all there is to sum, so a wavefront
// does a tile of 16 TN channels by itself and stores from its registers, without a barrier; the four of a workgroup take neighbouring channels of the
// same pixels, whose cache lines they share.
namespace patch {
template <typename T, int TH, int TW, int TN, int SD>
__global__ __launch_bounds__(256) void gconv_mfma_kernel(const uint16_t *x, const uint16_t *w, unsigned packed, int tiles, unsigned cols_d, unsigned cols_mul, unsigned hw,
                                                         unsigned px, unsigned image_d, unsigned image_mul, unsigned row_d, unsigned row_mul, Conv3Rest p)
{
    constexpr int TM = TH * TW, PH = (4 * TH - 1) * SD + 3, PW = (4 * TW - 1) * SD + 3, COPIES = (PH * PW * 4 + 63) / 64;
    constexpr unsigned OOB = 0xffffffffu;
    __shared__ __attribute__((aligned(16))) char smem[4 * COPIES * 1024];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const unsigned groups = (unsigned)(tiles + 3) >> 2, xcd = blockIdx.x & 7u, g = (groups * xcd >> 3) + (blockIdx.x >> 3);
    const unsigned t = g * 4u + (unsigned)wave;
    if (g >= (groups * (xcd + 1u) >> 3) || t >= (unsigned)tiles) return;
    const unsigned tile_m = div_by(t, Magic{cols_d, cols_mul, packed >> 2 & 31u}), col = t - tile_m * cols_d;
    const unsigned b = div_by(tile_m, Magic{image_d, image_mul, packed >> 7 & 31u}), in_image = tile_m - b * image_d;
    const unsigned ty = div_by(in_image, Magic{row_d, row_mul, packed >> 12 & 31u}), tx = in_image - ty * row_d;
    const int H = (int)(hw & 0xffffu), W = (int)(hw >> 16), oy0 = (int)ty * 4 * TH, ox0 = (int)tx * 4 * TW;

    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)w, 0, (int)0xfffffffeu, 0x00020000);          // never beyond the last block
    u32x4 wf[9][TN];
    auto load_w = [&](auto tc) {
        constexpr int k = decltype(tc)::value;
#pragma unroll
        for (int j = 0; j < TN; ++j) wf[k][j] = __builtin_amdgcn_raw_buffer_load_b128(rw, (unsigned)lane * 16u, (((int)col * TN + j) * 9 + k) * 1024, 0);
    };
    constexpr int EARLY = 3;
    static_for<EARLY>([&](auto tc) { load_w(tc); });
    const unsigned mine = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem + (unsigned)wave * (COPIES * 1024u);
    // the group's 32 channels of the image; bits 17-21 of packed: log2 of the tile columns of a super-group
    const unsigned first = (col >> (packed >> 17 & 31u)) * 64u;
    const uint64_t at_x = (uint64_t)(uintptr_t)x + (uint64_t)b * ((unsigned)(H * W) * px) + first;
    const u32x4 rx = {(unsigned)at_x, (unsigned)(at_x >> 32) & 0xffffu, (unsigned)(H * W) * px - first, 0x00020000u};
    const unsigned chunk = (unsigned)((lane & 3) ^ (lane >> 4)) * 16u;
    const int iy0 = oy0 * SD - 1, ix0 = ox0 * SD - 1;
    static_for<COPIES>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        const unsigned i = c * 16u + (unsigned)(lane >> 2), py = i / PW, qx = i - py * PW;
        const int iy = iy0 + (int)py, ix = ix0 + (int)qx;
        const bool ok = (unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)W && i < PH * PW;
        copy_to_lds(rx, ok ? __umul24(__umul24((unsigned)iy, (unsigned)W) + (unsigned)ix, px) + chunk : OOB, mine + c * 1024u);
    });
    static_for<9 - EARLY>([&](auto tc) { load_w(std::integral_constant<int, decltype(tc)::value + EARLY>()); });

    const int r16 = lane & 15, q = lane >> 4, n0 = (int)col * TN * 16 + 4 * q;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias, 0, (int)p.bias_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)p.res, 0, (int)p.res_bytes, 0x00020000);
    u32x2 bias[TN], res[TM][TN];
    unsigned off[TM];
#pragma unroll
    for (int j = 0; j < TN; ++j) bias[j] = __builtin_amdgcn_raw_buffer_load_b64(rb, (unsigned)(n0 + 16 * j) * 2u, 0, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int oy = oy0 + 4 * (i / TW) + (r16 >> 2), ox = ox0 + 4 * (i % TW) + (r16 & 3);
        off[i] = oy < p.Ho && ox < p.Wo ? (unsigned)((((int)b * p.Ho + oy) * p.Wo + ox) * p.ldy + n0) * 2u : OOB;
#pragma unroll
        for (int j = 0; j < TN; ++j) res[i][j] = __builtin_amdgcn_raw_buffer_load_b64(rr, off[i] == OOB ? OOB : off[i] + 32u * j, 0, 0);
    }
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int pix0 = (r16 >> 2) * SD * PW + (r16 & 3) * SD;
    const char *const base = smem + wave * (COPIES * 1024);
    auto at = [&](int k) { return pix0 * 64 + ((q ^ ((((pix0 + (k & 3)) >> 2) + (k >> 2)) & 3)) << 4); };
    // as in conv3_kernel: the patch has arrived when no more than what was fetched behind it is on its way, which has to be what the compiler issues
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((9 - EARLY) * TN + TN + TM * TN) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<9>([&](auto tc) {
        constexpr int k9 = decltype(tc)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int k = (4 * (i / TW) * SD + k9 / 3) * PW + 4 * (i % TW) * SD + k9 % 3;
            const uint4 a = *reinterpret_cast<const uint4 *>(base + at(k) + k * 64);
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::run(make_uint4(wf[k9][j].x, wf[k9][j].y, wf[k9][j].z, wf[k9][j].w), a, acc[i][j]);
        }
    });
    auto lo = [](unsigned v) { return Cvt<T>::from_bits(v & 0xffffu); };
    auto hi = [](unsigned v) { return Cvt<T>::from_bits(v >> 16); };
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float o[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            o[0] += lo(bias[j].x); o[1] += hi(bias[j].x); o[2] += lo(bias[j].y); o[3] += hi(bias[j].y);
            o[0] += lo(res[i][j].x); o[1] += hi(res[i][j].x); o[2] += lo(res[i][j].y); o[3] += hi(res[i][j].y);
            activate(p.act, [&](auto f) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = f(o[e]);
            });
            const u32x2 v = {Cvt<T>::pack2(o[0], o[1]), Cvt<T>::pack2(o[2], o[3])};
            __builtin_amdgcn_raw_buffer_store_b64(v, ry, off[i] == OOB ? OOB : off[i] + 32u * j, 0, 0);
        }
}

template <typename T, int TN, int SD> const void *kernel_of(int blocks)
{
    return blocks == 1 ? (const void *)gconv_mfma_kernel<T, 1, 1, TN, SD> : blocks == 2 ? (const void *)gconv_mfma_kernel<T, 2, 1, TN, SD>
                                                                                        : (const void *)gconv_mfma_kernel<T, 2, 2, TN, SD>;
}
template <typename T> const void *kernel_of(int tn, int sd, int blocks)
{
    if (tn == 2) return sd == 1 ? kernel_of<T, 2, 1>(blocks) : kernel_of<T, 2, 2>(blocks);
    return sd == 1 ? kernel_of<T, 1, 1>(blocks) : kernel_of<T, 1, 2>(blocks);
}
}  // namespace patch
constexpr bool kPool = false;
#else
constexpr bool kPool = true;
#endif

struct Shape { int th, tw, tn; };
constexpr Shape kShapes[CONV3_VARIANTS] = {{1, 1, 1}, {1, 1, 2}, {2, 1, 1}, {2, 1, 2}, {2, 2, 1}, {2, 2, 2}};

template <typename T, int V, int NW, int SD> const void *kernel_of(bool multi)
{
    constexpr Shape s = kShapes[V];
    if (!multi) return (const void *)conv3_kernel<T, s.th, s.tw, s.tn, NW, SD, false, kPool>;
    if constexpr (NW < 8 || (NW == 16 && V == 5)) return nullptr;
    else return (const void *)conv3_kernel<T, s.th, s.tw, s.tn, NW, SD, true, kPool>;
}
template <typename T, int V, int SD> const void *kernel_of(int nw, bool multi)
{
    switch (nw) {
    case 2: return kernel_of<T, V, 2, SD>(multi);
    case 4: return kernel_of<T, V, 4, SD>(multi);
    case 8: return kernel_of<T, V, 8, SD>(multi);
    case 16: return kernel_of<T, V, 16, SD>(multi);
    default: return nullptr;
    }
}
template <typename T, int SD> const void *kernel_of(int v, int nw, bool multi)
{
    switch (v) {
    case 0: return kernel_of<T, 0, SD>(nw, multi);
    case 1: return kernel_of<T, 1, SD>(nw, multi);
    case 2: return kernel_of<T, 2, SD>(nw, multi);
    case 3: return kernel_of<T, 3, SD>(nw, multi);
    case 4: return kernel_of<T, 4, SD>(nw, multi);
    case 5: return kernel_of<T, 5, SD>(nw, multi);
    default: return nullptr;
    }
}
template <typename T> const void *kernel_of(int v, int nw, int sd, bool multi) { return sd == 1 ? kernel_of<T, 1>(v, nw, multi) : kernel_of<T, 2>(v, nw, multi); }
const void *kernel_of(int dtype, int v, int nw, int sd, bool multi)
{
    return dtype == DT_BF16 ? kernel_of<bf16_t>(v, nw, sd, multi) : dtype == DT_F16 ? kernel_of<f16_t>(v, nw, sd, multi) : nullptr;
}

}  // namespace

const void *conv3_pool_kernel(int dtype, int v, int nw, int sd, bool multi)
#ifdef ECLIP_CONV3_POOL
{
    return kernel_of(dtype, v, nw, sd, multi);
}
#else
    ;                                        // the pooling forms, compiled from this file a second time

void conv3_tile(int variant, int *th, int *tw, int *bn)
{
    *th = 4 * kShapes[variant].th;
    *tw = 4 * kShapes[variant].tw;
    *bn = 16 * kShapes[variant].tn;
}

size_t conv3_lds_bytes(int variant, int nw, int stride, int Cin)
{
    const Shape s = kShapes[variant];
    const int ph = (4 * s.th - 1) * stride + 3, pw = (4 * s.tw - 1) * stride + 3, copies = (ph * pw * 4 + 63) / 64;
    const int per_wave = (Cin / 32 + nw - 1) / nw * copies, sums = s.th * s.tw * s.tn;
    return (size_t)nw * (per_wave > sums ? per_wave : sums) * 1024;
}

long conv3_tiles(int variant, int B, int Ho, int Wo, int Cout)
{
    int th, tw, bn;
    conv3_tile(variant, &th, &tw, &bn);
    return (long)B * ((Ho + th - 1) / th) * ((Wo + tw - 1) / tw) * (Cout / bn);
}

hipError_t conv3_init()
{
    for (int v = 0; v < CONV3_VARIANTS; ++v)
        for (int nw = 2; nw <= 16; nw *= 2)
            for (int sd = 1; sd <= 2; ++sd)
                for (bool multi : {false, true})
                    for (int dtype : {DT_BF16, DT_F16})
                        for (const void *k : {kernel_of(dtype, v, nw, sd, multi), conv3_pool_kernel(dtype, v, nw, sd, multi)}) {
                            if (!k) continue;
                            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, CONV3_MAX_LDS);
                            if (e != hipSuccess) return e;
                        }
    return hipSuccess;
}

// A slice per wavefront and fewer than half of the wavefronts without one, or several slices for each of 8 or 16 wavefronts.
bool conv3_launchable(int variant, int nw, const GemmTraits &t, int Cout)
{
    const int slices = t.Cin / 32;
    if (variant < 0 || variant >= CONV3_VARIANTS || (nw != 2 && nw != 4 && nw != 8 && nw != 16)) return false;
    if (slices > nw ? nw < 8 || slices > 4 * nw || (nw == 16 && variant == 5) : slices <= nw / 2) return false;      // (16 wavefronts leave 8 x 8 x 32 too few registers)
    return Cout % (16 * kShapes[variant].tn) == 0 && conv3_lds_bytes(variant, nw, t.stride, t.Cin) <= CONV3_MAX_LDS;
}

// Fitted to 132 layers (images of 5 x 5 to 56 x 56, 64 to 512 channels, both strides, batch 1 to 8, on 64, 128 and 256 CUs) x up to 12 shapes, in chains of 40
// layers with weights of their own; near the best shapes to 9 % rms.  A dispatch with its trip to memory, per compute unit the bytes of
// weights and patches and the matrix instructions, and what a further round of workgroups waits for.  Put on the scale of the wave-split-K costs (their
// cost is 1.25 times the measured time less 3.2 us).  Picks are 2.8 % over the best of all kernels' plans; against the plans
// without this kernel these layers take 15 % less: 7 x 7 x 512 at batch 1 on 128 CUs 5.95 -> 4.34 us, at batch 4 on 256 7.5 -> 5.2; 28 x 28 x 128 4.85 -> 3.74;
// 56 x 56 x 64 at batch 4 on 256 6.3 -> 4.8.  Many rounds of workgroups stay with the LDS tiles (14 x 14 x 512, stride 2, batch 8 on 64 CUs: 14.1 and 33.7 here).
double conv3_cost(int variant, int nw, const GemmTraits &t, long N, int n_cu)
{
    const Shape s = kShapes[variant];
    const int slices = t.Cin / 32, per_wave = (slices + nw - 1) / nw, blocks = s.th * s.tw * s.tn;
    const int ph = (4 * s.th - 1) * t.stride + 3, pw = (4 * s.tw - 1) * t.stride + 3, copies = (ph * pw * 4 + 63) / 64;
    const double tiles = (double)conv3_tiles(variant, t.B, t.Ho, t.Wo, (int)N), r = tiles / n_cu;
    const double per_cu = 0.5 * ((r > 1.0 ? r : 1.0) + (double)(long)(r + 1.0 - 1e-9));
    const int lds_kb = (int)(conv3_lds_bytes(variant, nw, t.stride, t.Cin) / 1024);
    int at_once = (s.tn == 1 || s.th * s.tw < 4 ? 32 : 16) / nw;
    if (at_once > 160 / lds_kb) at_once = 160 / lds_kb;
    if (at_once < 1) at_once = 1;
    const double rounds = (double)(long)(r / at_once + 1.0 - 1e-9);
    const double us = 2.774 + 0.342 * (per_wave - 1) + per_cu * slices * (9 * s.tn * 0.00509 + copies * 0.00828 + 9 * blocks * 0.00152) + 0.829 * (rounds - 1.0) +
                      per_wave * 9 * blocks * 0.00154 + 0.444 * (r < 1.0 ? r : 1.0) + (variant == 4 ? 0.673 : variant == 5 ? 0.577 : 0.0);
    return 1.25 * us - 3.2;
}

// 16-bit types, whole slices and blocks of channels; sizes that the kernel packs into 16 bits or multiplies in 24
bool conv3_takes(int KH, int KW, int stride, int pad, int H, int W, int Cin, int Cout, int ldx)
{
    return KH == 3 && KW == 3 && (stride == 1 || stride == 2) && pad == 1 && Cin % 32 == 0 && Cout % 16 == 0 && H < 4096 && W < 4096 && ldx % 8 == 0 && ldx < 32768 &&
           (long)H * W * ldx * 2 < (1l << 31);
}

hipError_t launch_conv3(const ConvGemmArgs &a, int variant, int nw, hipStream_t s)
{
    const int ldx = a.ldx ? a.ldx : a.Cin, ldy = a.ldy ? a.ldy : a.Cout;
    int th, tw, bn;
    if (variant < 0 || variant >= CONV3_VARIANTS || a.nchw_c || !conv3_takes(a.KH, a.KW, a.stride, a.pad, a.H, a.W, a.Cin, a.Cout, ldx)) return hipErrorInvalidValue;
    conv3_tile(variant, &th, &tw, &bn);
    const size_t lds = conv3_lds_bytes(variant, nw, a.stride, a.Cin);
    const bool multi = a.Cin / 32 > nw;
    const void *k = a.pool ? conv3_pool_kernel(a.dtype, variant, nw, a.stride, multi) : kernel_of(a.dtype, variant, nw, a.stride, multi);
    if (!k || a.Cout % bn || lds > CONV3_MAX_LDS) return hipErrorInvalidValue;
    const uint16_t *x = (const uint16_t *)a.x, *w = (const uint16_t *)a.w;
    const int tiles_x = (a.Wo + tw - 1) / tw, tiles_y = (a.Ho + th - 1) / th, tiles_n = a.Cout / bn, tiles_m = a.B * tiles_x * tiles_y;
    int tiles = tiles_m * tiles_n;
    // down the tile columns where the weights are the larger operand, along the rows where the activations are
    const bool rows = (long)a.Cout * 9 < (long)a.B * a.H * a.W;
    Magic inner = magic_of((unsigned)(rows ? tiles_n : tiles_m)), image = magic_of((unsigned)(tiles_x * tiles_y)), row = magic_of((unsigned)tiles_x);
    unsigned packed = (rows ? 3u : 2u) | inner.shift << 2 | image.shift << 7 | row.shift << 12;
    unsigned hw = (unsigned)a.H | (unsigned)a.W << 16, px_slices = (unsigned)(ldx * 2) | (unsigned)(a.Cin / 32) << 16;
    Conv3Rest p{};
    p.bias = (const uint16_t *)a.bias; p.res = (const uint16_t *)a.res; p.f32 = a.y32 != nullptr;
    p.y = p.f32 ? (void *)a.y32 : a.y;
    p.bias_bytes = a.bias ? (unsigned)a.Cout * 2u : 0u;
    const unsigned elems = (unsigned)((a.B * a.Ho * a.Wo >> (a.pool ? 2 : 0)) - 1) * (unsigned)ldy + (unsigned)a.Cout;
    p.y_bytes = elems * (p.f32 ? 4u : 2u);
    p.res_bytes = a.res ? elems * 2u : 0u;
    p.ldy = ldy; p.act = a.act; p.Ho = a.Ho; p.Wo = a.Wo;
    void *args[] = {&x, &w, &packed, &tiles, &inner.d, &inner.mul, &hw, &px_slices, &image.d, &image.mul, &row.d, &row.mul, &p};
    return hipLaunchKernel(k, dim3((unsigned)(tiles + 7) & ~7u), dim3((unsigned)nw * 64), args, lds, s);
}

// Tile of the grouped form: blocks of 4 x 4 pixels per wavefront (1, 2 or 4), 0: left to the wave-split-K kernel.  n_cu: CuShare::even_cu.  One block while
// few workgroups share a compute unit, then two to halve the fetches of the weights, four beyond five workgroups (a lone wavefront takes a
// microsecond longer over four).  Against the wave-split-K kernel, us in chains of 40 layers: 56 x 56 x 128 at batch 1 on 128 CUs 6.1, with two blocks 4.4 (one
// 4.9, four 5.6); at batch 4 on 64 18.5, 11.8 (15.5, 12.1); 14 x 14 x 512 at batch 2 on 256 4.75, 3.7; 7 x 7 x 1024 at batch 8 on 128 5.95, 4.3; of
// 132 layers none with a workgroup per CU was slower, those with fewer within what the host's pace blurs.
int gconv3_blocks(const GConvArgs &a, int S, int n_cu)
{
    const int SI = S * (a.Cin / a.groups), SO = S * (a.Cout / a.groups), tn = SO % 32 ? 1 : 2, cols = SO / (16 * tn);
    if (SI != 32 || SO % 16 || (cols & (cols - 1)) || !conv3_takes(a.KH, a.KW, a.stride, a.pad, a.H, a.W, a.Cin, a.Cout, a.Cin)) return 0;
    if (const char *f = getenv("ECLIP_GCONV3")) {                    // blocks; 0: the wave-split-K kernel; no such number: the choice below
        int blocks = -1;
        if (sscanf(f, "%d", &blocks) == 1 && (blocks == 0 || blocks == 1 || blocks == 2 || blocks == 4)) return blocks;
    }
    const double per_cu = (double)gconv3_workgroups(a, S, 1) / n_cu;
    return per_cu <= 1.75 ? 1 : per_cu <= 5.0 ? 2 : 4;
}
unsigned gconv3_workgroups(const GConvArgs &a, int S, int blocks)
{
    const int th = blocks > 1 ? 8 : 4, tw = blocks > 2 ? 8 : 4, tn = S * (a.Cout / a.groups) % 32 ? 1 : 2;
    const long tiles = (long)a.B * ((a.Ho + th - 1) / th) * ((a.Wo + tw - 1) / tw) * (a.Cout / (16 * tn));
    return (unsigned)((tiles + 3) / 4);
}

hipError_t launch_gconv3(const GConvArgs &a, int S, int blocks, hipStream_t s)
{
    const int th = blocks > 1 ? 8 : 4, tw = blocks > 2 ? 8 : 4, SO = S * (a.Cout / a.groups), tn = SO % 32 ? 1 : 2;
    const void *k = a.dtype == DT_BF16 ? patch::kernel_of<bf16_t>(tn, a.stride, blocks) : patch::kernel_of<f16_t>(tn, a.stride, blocks);
    const uint16_t *x = (const uint16_t *)a.x, *w = (const uint16_t *)a.w;
    const int tiles_x = (a.Wo + tw - 1) / tw, tiles_y = (a.Ho + th - 1) / th, n_cols = a.Cout / (16 * tn);
    int tiles = a.B * tiles_x * tiles_y * n_cols;
    Magic cols = magic_of((unsigned)n_cols), image = magic_of((unsigned)(tiles_x * tiles_y)), row = magic_of((unsigned)tiles_x);
    unsigned packed = cols.shift << 2 | image.shift << 7 | row.shift << 12 | (unsigned)__builtin_ctz((unsigned)(SO / (16 * tn))) << 17;
    unsigned hw = (unsigned)a.H | (unsigned)a.W << 16, px = (unsigned)a.Cin * 2u;
    Conv3Rest p{};
    p.bias = (const uint16_t *)a.bias; p.res = (const uint16_t *)a.res; p.y = a.y;
    p.bias_bytes = a.bias ? (unsigned)a.Cout * 2u : 0u;
    p.y_bytes = (unsigned)(a.B * a.Ho * a.Wo) * (unsigned)a.Cout * 2u;
    p.res_bytes = a.res ? p.y_bytes : 0u;
    p.ldy = a.Cout; p.act = a.act; p.Ho = a.Ho; p.Wo = a.Wo;
    void *args[] = {&x, &w, &packed, &tiles, &cols.d, &cols.mul, &hw, &px, &image.d, &image.mul, &row.d, &row.mul, &p};
    return hipLaunchKernel(k, dim3((gconv3_workgroups(a, S, blocks) + 7u) & ~7u), dim3(256), args, 0, s);
}

#endif

}  // namespace eclip
