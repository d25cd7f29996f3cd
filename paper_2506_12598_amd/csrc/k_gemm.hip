// Implicit-GEMM convolution / linear layer on the gfx950 matrix cores.
//
//   y[m][n] = act( sum_k A[m][k] * w[n][k] + bias[n] + res[m][n] )
//   m = (b, oh, ow)  row of the output in channels-last order
//   k = (kh, kw, ci) with ci innermost, so that 8 consecutive k are 16 contiguous bytes of the
//       input whenever Cin % 8 == 0 (the loader pads the 3-channel network input to 8)
//   A[m][k] = x[b][oh*stride-pad+kh][ow*stride-pad+kw][ci], zero outside the image
//
// A linear layer is the case KH = KW = 1, H = W = 1 (or W = sequence length).
//
// Tiling: one 256-thread workgroup (4 wavefronts of 64) owns a BM x BN output tile and walks K in
// steps of BK through a two-slot LDS ring.  Global loads run two steps ahead of the MFMAs: while step t
// is multiplied out of LDS slot t%2, the registers already hold step t+1 and the loads of step t+2 are
// in flight, so one barrier per step suffices and a load has two steps to arrive.  Each wavefront owns
// a (BM/WM) x (BN/WN) sub-tile made of 16x16 blocks, one v_mfma_f32_16x16x32 per block and 32 k.  The
// weight tile is fed as the MFMA's row operand and the im2col tile as its column operand, so a lane
// ends up with 4 consecutive output channels of one output pixel: 8 contiguous bytes of y.
//
// Batch-1 inference leaves most layers with a few dozen tiles and a long K.  Those are cut along K
// into `splits` slices, one workgroup each, which write float partial sums to a workspace; a second,
// tiny kernel adds the slices in slice order (the sum does not depend on scheduling) and applies the
// epilogue.  The kernel boundary is what makes the partial sums visible: a device-wide fence inside the
// GEMM would have to write back the whole L2 of the issuing XCD, which costs far more than a launch.
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "gemm_tile.h"

namespace eclip {

namespace {

// y = act(sum_z ws[z] + bias + res): one thread per 4 consecutive channels (one channel when N % 4 != 0).
// The slices are read eight at a time so that their loads overlap; the additions keep slice order.
template <typename T>
__global__ __launch_bounds__(64) void splitk_reduce_kernel(const float *ws, int splits, int M, int N, const uint16_t *bias,
                                                           const uint16_t *res, uint16_t *y, float *y32, int act, int ldy)
{
    const bool vec = ((N & 3) == 0);
    const int per_row = vec ? N / 4 : N;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)M * per_row) return;
    const int m = (int)((unsigned)idx / (unsigned)per_row);
    const int n = (int)((unsigned)idx % (unsigned)per_row) * (vec ? 4 : 1);
    const long slice = (long)M * N;
    const float *src = ws + (long)m * N + n;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (vec) {
        for (int z0 = 0; z0 < splits; z0 += 8) {
            float4 q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                q[u] = (z0 + u < splits) ? *reinterpret_cast<const float4 *>(src + (long)(z0 + u) * slice) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < 8; ++u) { s[0] += q[u].x; s[1] += q[u].y; s[2] += q[u].z; s[3] += q[u].w; }
        }
    } else {
        for (int z = 0; z < splits; ++z) s[0] += src[z * slice];
    }
#define EPI(A) epilogue_store<T, A>(bias, res, y, y32, M, N, m, n, s, vec ? 4 : 1, ldy)
    ECLIP_ACT_SWITCH(act, EPI)
#undef EPI
}

constexpr PPTile kPlainTiles[] = {{0, 128, 128, 32, 2, LOOP_PLAIN}, {1, 64, 64, 64, 4, LOOP_PLAIN}};
constexpr PPTile tile_of_id(int id) { return id == 0 || id == 1 ? kPlainTiles[id] : pp_tile(id); }

template <typename T>
hipError_t launch_pp_split(const GemmDev &d, const GemmPlan &pl, hipStream_t s, hipError_t e);

template <typename T>
hipError_t launch_t(const GemmDev &d, const GemmPlan &pl, SeDeal deal, hipStream_t s)
{
    const dim3 grid(se_deal_grid(deal, (uint32_t)pl.tiles), (unsigned)pl.splits);
    switch (pl.variant) {
    case 0: hipLaunchKernelGGL((conv_gemm_kernel<T, 128, 128, 32, 2, 2, 2>), grid, dim3(256), lds_bytes(128, 128, 32), s, d, deal); break;
    case 1: hipLaunchKernelGGL((conv_gemm_kernel<T, 64, 64, 64, 2, 2, 4>), grid, dim3(256), lds_bytes(64, 64, 64), s, d, deal); break;
#define X(ID, BM, BN, BK, RS, LP) \
    case ID:                                                                                                                    \
        if constexpr (LP == LOOP_DMA)                                                                                           \
            if (gemm_pools(d)) return launch_pp_pool<ID>(d, deal, std::is_same<T, bf16_t>::value ? DT_BF16 : DT_F16, grid, s);  \
        return launch_pp_split<T>(d, pl, s, launch_pp<ID>(d, deal, std::is_same<T, bf16_t>::value ? DT_BF16 : DT_F16, grid, s));
        ECLIP_PP_TILES(X)
#undef X
    default: return hipErrorInvalidValue;
    }
    return launch_pp_split<T>(d, pl, s, hipGetLastError());
}

// second launch of a layer whose K is cut over the grid: the slice sum
template <typename T>
hipError_t launch_pp_split(const GemmDev &d, const GemmPlan &pl, hipStream_t s, hipError_t e)
{
    if (e != hipSuccess || pl.splits == 1) return e;
    const long threads = (long)d.M * ((d.N & 3) == 0 ? d.N / 4 : d.N);
    hipLaunchKernelGGL((splitk_reduce_kernel<T>), dim3((unsigned)((threads + 63) / 64)), dim3(64), 0, s, d.ws, pl.splits, d.M, d.N,
                       d.bias, d.res, d.y, d.y32, d.act, d.ldy);
    return hipGetLastError();
}

}  // namespace

hipError_t conv_gemm_init()
{
    hipError_t e;
#define X(ID, BM, BN, BK, RS, LP) \
    if ((e = init_pp<ID>()) != hipSuccess) return e;                      \
    if constexpr (LP == LOOP_DMA)                                         \
        if ((e = init_pp_pool<ID>()) != hipSuccess) return e;
    ECLIP_PP_TILES(X)
#undef X
    return hipSuccess;
}

void conv_gemm_tile(int variant, int *bm, int *bn, int *bk)
{
    const PPTile t = tile_of_id(variant);
    *bm = t.bm;
    *bn = t.bn;
    *bk = t.bk;
}

const char *conv_gemm_kernel_name(int variant) { return tile_of_id(variant).loop == LOOP_DMA ? "conv_gemm_dma_kernel" : "conv_gemm_kernel"; }
int conv_gemm_threads(int variant) { return tile_of_id(variant).loop == LOOP_DMA || tile_of_id(variant).loop == LOOP_PLAIN ? 256 : 512; }

static long cdiv(long a, long b) { return (a + b - 1) / b; }

// Large un-split problems are launched on the 8 x 4 block raster: the grid grows to whole blocks, 8 at a time.
static void set_raster(GemmPlan &pl, long M, long N)
{
    int bm, bn, bk;
    conv_gemm_tile(pl.variant, &bm, &bn, &bk);
    const long tm = cdiv(M, bm), tn = cdiv(N, bn);
    if (tm * tn < 256 || pl.splits != 1) {
        // fewer tiles than CUs (or K slices in grid.y): deal whole tile columns or rows to the XCDs when they divide
        // evenly, so that each L2 holds 1/8 of one operand instead of all of both.  (Uneven ranges of tiles per XCD were
        // slower than the plain order: ResNet-50's 64 x 128 tiles at batch 1, 13 tile rows, 2 us per launch in the chain.)
        if (tn >= 8 && tn % 8 == 0) pl.raster = 2;
        else if (tm >= 8 && tm % 8 == 0) pl.raster = 3;
        pl.tiles = (int)(tn * tm);
        return;
    }
    if (tn < 4) {
        // 8 x 4 blocks of a matrix with one to three tile columns are mostly empty, and an empty workgroup of 512 threads is
        // not free to launch: bands of tile rows per XCD instead, which pads the grid to 8 rows only
        // (VGG-16 conv1_2 at batch 8, one tile column: 12544 workgroups of which 3136 have a tile, 69 -> 63 us)
        pl.raster = 3;
        pl.tiles = (int)xcd_range_blocks((uint32_t)(tm * tn));
        return;
    }
    const long blocks = cdiv(tm, 8) * cdiv(tn, 4);
    pl.raster = 1;
    pl.tiles = (int)(cdiv(blocks, 8) * 8 * 32);
}

// Wave-split-K tiles are dealt to the 8 XCDs along one dimension when that dimension has enough tiles to keep the
// XCDs evenly loaded (a multiple of 8 tiles): along N when N >= M (the weights,
// N x K, are then the larger operand; the im2col operand is at most M x K), else along M; the other dimension is the
// second choice.  (The lean form deals its tiles itself where this leaves them in plain order, see launch_wsk_lean.)
static void set_xcd_split(GemmPlan &pl, long M, long N)
{
    int bm, bn;
    conv_wsk_tile(pl.variant, &bm, &bn);
    const long tm = cdiv(M, bm), tn = cdiv(N, bn);
    auto fits = [](long t) { return t >= 8 && t % 8 == 0; };
    const bool n_first = N >= M;                      // W is N x K, the im2col operand at most M x K
    const int order[2] = {n_first ? 2 : 3, n_first ? 3 : 2};
    for (int r : order) {
        const long t = r == 2 ? tn : tm, other = r == 2 ? tm : tn;
        if (fits(t)) {
            pl.raster = r;
            pl.tiles = (int)(8 * cdiv(t, 8) * other);
            return;
        }
    }
}

// Cost of the wave-split-K kernel (us, without the launch), 1e30 when the combination does not exist.  A compute
// unit pulls the im2col rows as 64-byte runs (slow) and the weights as contiguous 1 KB blocks (fast), or is bound by
// its matrix instructions when the tile is large; its workgroups run one after another; each wavefront needs
// ceil(steps / depth) round trips to memory; the partial tiles of the nw wavefronts are summed through LDS.
static double wsk_cost(long M, long N, long K, int n_cu, int v, int nw)
{
    const double ra = 2.676e4, rw = 4.635e5;         // bytes per us per CU: activation rows, weight blocks
    const double rm = 1.539e6;                       // multiply-adds per us per CU with 8 or more wavefronts
    const double lat = 0.04896, c_out = 3.14e-6, c_red = 1.248e-5, l2 = 9.238e7, c_wg = 0.02628;
    if (conv_wsk_lds_bytes(v, nw) > 128 * 1024) return 1e30;
    int bm, bn;
    conv_wsk_tile(v, &bm, &bn);
    const int depth = (bm + bn) <= 32 ? 8 : (bm + bn) <= 48 ? 6 : (bm + bn) <= 80 ? (nw == 16 ? 3 : 4) : (bm + bn) <= 96 ? (nw == 16 ? 2 : 3) : 2;
    const double t = (double)(cdiv(M, bm) * cdiv(N, bn));
    const double per_cu = (double)cdiv((long)t, n_cu), frac = t / n_cu > 1.0 ? t / n_cu : 1.0;
    const double a_b = (double)(M < bm ? M : bm) * K * 2.0, w_b = (double)(N < bn ? N : bn) * K * 2.0;
    const double loads = a_b / ra + w_b / rw;
    const double macs = (double)(M < bm ? M : bm) * bn * K / rm / (nw < 8 ? nw / 8.0 : 1.0);
    const double cu = per_cu * (loads > macs ? loads : macs) + frac * c_wg + frac * bm * bn * (c_out + c_red * nw);
    const double all = t * (a_b + w_b) / l2;
    const double cost = (cu > all ? cu : all) + lat * (double)cdiv(cdiv(cdiv(K, 32), nw), depth);
    // what the model above leaves unexplained per (tile, wavefront count), fitted last: cost * scale + offset
    static const struct { double scale, offset; } kAdjust[CONV_WSK_VARIANTS][3] = {
        {{1.0, 0.0}, {1.0, 0.0}, {1.0, -0.1}},  {{0.95, 0.2}, {1.0, 0.0}, {0.95, 0.0}}, {{1.2, 0.0}, {1.0, 0.0}, {1.0, 0.0}},
        {{1.0, 0.0}, {1.0, 0.0}, {1.0, 0.0}},   {{1.0, 0.0}, {0.9, 0.1}, {1.05, 0.0}},  {{0.9, 0.0}, {1.0, 0.0}, {1.0, 0.0}}};
    const auto &adj = kAdjust[v][nw == 4 ? 0 : nw == 8 ? 1 : 2];
    return cost * adj.scale + adj.offset;
}

// wsk_cost on the scale of the LDS tiles' costs: what every wave-split-K launch pays before and after its loop, and what
// each further round of workgroups on a compute unit pays again (same fit as the LDS tiles' table).  The fit priced the shape that
// wsk_cost picks, and only there does it hold: it decides between that shape and the LDS tiles, not among the wave-split-K
// shapes.  Picking those by it too makes 64 x 64 tiles win wherever they save a round: 160 kinds of request (12 networks, batch 1 to
// 8, 64 to 256 compute units) took 5.7 % longer, VGG-16 at batch 8 on 160 CUs 1141 us instead of 755.
static double wsk_whole_cost(long M, long N, long K, int n_cu, int v, int nw)
{
    int bm, bn;
    conv_wsk_tile(v, &bm, &bn);
    const double rounds = (double)(cdiv(M, bm) * cdiv(N, bn)) / n_cu;
    return wsk_cost(M, N, K, n_cu, v, nw) + 2.0 + (rounds > 1.0 ? rounds - 1.0 : 0.0);
}

// The same for the lean form (k_wsk_lean.hip), on the scale of the LDS tiles' costs and to pick by as well as to price by.  A compute unit
// takes in activations and weights at one rate each, a workgroup needs `lat` per round trip of its slices, and the partial tiles
// cost their summation; `offset` holds what that leaves unexplained per (tile, wavefront count).  Least-squares fit to 253 layers of
// the networks here (batch 1 to 8) x 17 shapes on 256 CUs, in chains whose weights no L2 holds, each time taken 1.25-fold, which
// is by how much the LDS tiles' table prices the small copied tiles of that measurement too high.  Of all plans the picks cost 5.3 % more than the
// best on average (7.3 % with the general form's constants) and 24 % at worst (48 %); the host submits a launch in 2.5 us,
// which blurs the shortest.  64 x 64 tiles carry 0.8 us that the fit does not ask for: where it errs, it errs towards them.
// With 256 CUs few of those layers had a second round.  On 64 and 96 CUs 32 x 64 tiles of 8 wavefronts take 0.6 us more for each (up to three) than
// the rest of the model knows (2304 x 768 by 64 rows on 64 CUs, 72 workgroups: 7.5 us; with 4 wavefronts, which it takes now, 6.6).
static double wsk_lean_cost(long M, long N, long K, int n_cu, int v, int nw)
{
    const double ra = 8.348e4, rw = 1.332e5, rm = 2.791e6, lat = 0.368, c_out = 2.165e-6, c_red = 1.1165e-4, l2 = 9.0e7, c_wg = 0.014, base = 0.324;
    if (conv_wsk_lds_bytes(v, nw) > 128 * 1024) return 1e30;
    int bm, bn;
    conv_wsk_tile(v, &bm, &bn);
    const int depth = conv_wsk_lean_depth(v, nw);
    const double t = (double)(cdiv(M, bm) * cdiv(N, bn));
    const double per_cu = (double)cdiv((long)t, n_cu), frac = t / n_cu > 1.0 ? t / n_cu : 1.0;
    const double a_b = (double)(M < bm ? M : bm) * K * 2.0, w_b = (double)(N < bn ? N : bn) * K * 2.0;
    const double loads = a_b / ra + w_b / rw;
    const double macs = (double)(M < bm ? M : bm) * bn * K / rm / (nw < 8 ? nw / 8.0 : 1.0);
    const double cu = per_cu * (loads > macs ? loads : macs) + (frac - 1.0) * c_wg + frac * bm * bn * (c_out + c_red * nw);
    const double all = t * (a_b + w_b) / l2;
    static const double offset[CONV_WSK_VARIANTS][3] = {{0.0, -0.324, -1.127}, {-0.347, -1.156, -2.773}, {0.21, -1.517, 0.0},
                                                        {0.582, 0.529, 0.356}, {0.336, 0.166, -0.264},   {0.01, -0.333, -1.203}};
    const double again = v == 1 && nw == 8 && per_cu > 1.0 ? 0.6 * ((per_cu < 4.0 ? per_cu : 4.0) - 1.0) : 0.0;
    return (cu > all ? cu : all) + lat * (double)cdiv(cdiv(cdiv(K, 32), nw), depth) + base + offset[v][nw == 4 ? 0 : nw == 8 ? 1 : 2] + again;
}

// What the planner compares the general form's shapes by, for a first layer that reads the caller's planes among others (tile `v`, `nw`
// wavefronts; the lean form is compared by wsk_lean_cost).
double conv_wsk_cost_estimate(long M, long N, long K, int n_cu, int v, int nw) { return wsk_cost(M, N, K, n_cu, v, nw); }

// Grouped convolutions: 4 or 8 wavefronts, all tiles but 64 x 64.
GemmPlan conv_wsk_plan_columns(long M, long N, long K, int n_cu, int columns)
{
    GemmPlan pl{1, 3, 1, 0, 4, 0};
    double best = 1e30;
    for (int v = 0; v < CONV_WSK_VARIANTS; ++v)
        for (int nw = 4; nw <= 8; nw *= 2) {
            int bm, bn;
            conv_wsk_tile(v, &bm, &bn);
            if (bm * bn > 32 * 64 || (columns && columns % bn)) continue;
            const double c = wsk_lean_cost(M, N, K, n_cu, v, nw);
            if (c < best) { best = c; pl = GemmPlan{1, v, 1, (int)(cdiv(M, bm) * cdiv(N, bn)), nw, 0}; }
        }
    set_xcd_split(pl, M, N);
    return pl;
}

// Every plan worth timing for a problem (eclip_model_tune): all wave-split-K tiles and wavefront counts that fit LDS, and
// every 8-wavefront or copied LDS tile whole and with K cut in two or four where the workspace allows (the plain tiles were best on
// none of 900 problems).  Tiles far larger than the problem are left out (a 256-row tile for a 64-row problem only wastes
// the measurement).
std::vector<GemmPlan> conv_gemm_candidates(long M, long N, long K, int n_cu, size_t ws_floats, const GemmTraits &traits)
{
    std::vector<GemmPlan> out;
    for (int v = 0; traits.conv3 && v < CONV3_VARIANTS; ++v)
        for (int nw = 2; nw <= 16; nw *= 2)
            if (conv3_launchable(v, nw, traits, (int)N)) out.push_back(GemmPlan{2, v, 1, (int)conv3_tiles(v, traits.B, traits.Ho, traits.Wo, (int)N), nw, 0});
    for (int v = 0; v < CONV_WSK_VARIANTS; ++v)
        for (int nw = 4; nw <= 16; nw *= 2) {
            if (conv_wsk_lds_bytes(v, nw) > 128 * 1024) continue;
            int bm, bn;
            conv_wsk_tile(v, &bm, &bn);
            if (cdiv(M, bm) * cdiv(N, bn) > 65536 * 4) continue;
            GemmPlan pl{1, v, 1, (int)(cdiv(M, bm) * cdiv(N, bn)), nw, 0};
            set_xcd_split(pl, M, N);
            out.push_back(pl);
        }
    for (const PPTile &t : kPPTiles) {
        const int v = t.id, bm = t.bm, bn = t.bn, bk = t.bk;
        if (bm > 2 * M + 32 || bn > 2 * N + 32 || (pp_fast_forms_only(v) && !traits.copied)) continue;
        const long KT = cdiv(K, bk);
        for (long sp = 1; sp <= 4; sp *= 2) {
            if (sp > 1 && (K < 512 * sp || (size_t)(sp * M * N) > ws_floats)) continue;
            GemmPlan pl{0, v, 1, (int)(cdiv(M, bm) * cdiv(N, bn)), 4, 0};
            pl.splits = (int)cdiv(KT, cdiv(KT, sp));
            if (sp > 1 && pl.splits == 1) continue;
            set_raster(pl, M, N);
            out.push_back(pl);
        }
    }
    (void)n_cu;
    return out;
}

// Tiles of the XCD that the block raster (set_raster) gives the most: whole blocks of 8 x 4 are dealt out, 9 of them as 2 to one and 1 to seven
static long heaviest_xcd(long tm, long tn)
{
    const long rows = cdiv(tm, 8), cols = cdiv(tn, 4), blocks = rows * cols;
    long most = 0;
    for (long x = 0; x < 8; ++x) {
        long n = 0;
        for (long b = x; b < blocks; b += 8) n += std::min(8l, tm - b % rows * 8) * std::min(4l, tn - b / rows * 4);
        most = std::max(most, n);
    }
    return most;
}

// conv_gemm_plan; *cost receives the modelled time of the plan (us, without the launch)
static GemmPlan plan_with_cost(long M, long N, long K, int n_cu, size_t ws_floats, const GemmTraits &traits, double *cost_out)
{
    *cost_out = 0.0;
    const bool lean = traits.lean;
    // wave-split-K launches are not dealt to the shader engines (se_deal.h); LDS tiles are where they need to be
    const int even_cu = traits.even_cu > 0 ? traits.even_cu : n_cu;
    auto tiles = [&](int v) { int bm, bn, bk; conv_gemm_tile(v, &bm, &bn, &bk); return cdiv(M, bm) * cdiv(N, bn); };
    auto wsk_tiles = [&](int v) { int bm, bn; conv_wsk_tile(v, &bm, &bn); return cdiv(M, bm) * cdiv(N, bn); };
    GemmPlan pl{0, 1, 1, 0, 4, 0};
    // tuning aid: ECLIP_GEMM_FORCE="kind,variant,n" overrides the heuristic; n = K splits (kind 0, clamped to the
    // workspace) or wavefronts per workgroup (kind 1: 4, 8 or 16); ids without a tile leave the choice to the planner
    const char *force = getenv("ECLIP_GEMM_FORCE");
    int f_kind = -1, f_variant = -1, f_n = -1;
    if (force) sscanf(force, "%d,%d,%d", &f_kind, &f_variant, &f_n);
    if (f_kind == 1 && f_variant >= 0 && f_variant < CONV_WSK_VARIANTS && (f_n == 4 || f_n == 8 || f_n == 16) &&
        conv_wsk_lds_bytes(f_variant, f_n) <= 128 * 1024) {
        pl.kind = 1; pl.variant = f_variant; pl.nw = f_n; pl.tiles = (int)wsk_tiles(f_variant);
        set_xcd_split(pl, M, N);
        return pl;
    }
    if (f_kind == 2 && traits.conv3 && conv3_launchable(f_variant, f_n, traits, (int)N))
        return GemmPlan{2, f_variant, 1, (int)conv3_tiles(f_variant, traits.B, traits.Ho, traits.Wo, (int)N), f_n, 0};
    if (f_kind == 0 && tile_of_id(f_variant).id >= 0 && (traits.copied || !pp_fast_forms_only(f_variant))) {
        pl.variant = f_variant;
        pl.tiles = (int)tiles(pl.variant);
        int bm, bn, bk;
        conv_gemm_tile(pl.variant, &bm, &bn, &bk);
        const long KT = cdiv(K, bk);
        long s = f_n < 1 ? 1 : f_n;
        if (s > KT) s = KT;
        while (s > 1 && (size_t)(s * M * N) > ws_floats) --s;
        const long kt_per = cdiv(KT, s);
        pl.splits = (int)cdiv(KT, kt_per);
        set_raster(pl, M, N);
        return pl;
    }
    // Every candidate is priced with a small cost model fitted to timings (below).  Times in microseconds, without the launch.
    double best = 1e30;
    for (int v = 0; v < CONV_WSK_VARIANTS; ++v)
        for (int nw = 4; nw <= 16; nw *= 2) {
            const double cost = lean ? wsk_lean_cost(M, N, K, even_cu, v, nw) : wsk_cost(M, N, K, even_cu, v, nw);
            if (cost < best) { best = cost; pl = GemmPlan{1, v, 1, (int)wsk_tiles(v), nw, 0}; }
        }
    if (!lean) best = wsk_whole_cost(M, N, K, even_cu, pl.variant, pl.nw);
    const bool long_sums = traits.copied && M >= 512 && K >= 768;        // copied_long, below
    if (long_sums && traits.gelu) best += (pl.nw == 4 ? 0.3 + 1.4e-5 * M * N / even_cu : 6.2e-5 * M * N / even_cu);
    // LDS-tiled kernels, optionally with K cut into slices (second launch: its cost plus the traffic of the partial sums).
    // A tile costs `fixed` us once (fill of the pipeline, epilogue) and `step` us per K step of its own depth when it has a
    // compute unit to itself; every further round of workgroups on a compute unit pays the steps again and `more` us; where two
    // workgroups fit a compute unit and hide each other's latencies, the two cost `two` times one; a full machine slows every
    // step by about 15 % (shared L2 and vector caches).  Times are without the 2.5 us launch cost that all single-launch
    // candidates share (as in wsk_cost).  Constants fitted, together with wsk_whole_cost's, to 440 problems x 36 plans (40 linear layers of 128 to
    // 1536 rows, 70 convolutions of ResNet, VGG and MobileNet shapes at batch 1, 3 and 8, each on 64, 96, 160 and 256 compute units), every
    // plan timed in a chain of four to eight layers with weights of their own, so that no layer finds its weights in an L2.
    // `bench.py --plans` repeats that measurement for linear layers.  eclip_model_tune closes what is left by measurement.
    // Shares whose shader engines hold unequal numbers of CUs (160 in granules of 16: 8, 8, 2 and 2 per XCD): LDS tiles are dealt to them
    // (se_deal.h).  That costs 1.1 us (the note read from memory, the surplus workgroups) in one round of the share, and in more rounds
    // up to 1.7 on the most uneven one (144: 8, 8, 1, 1), little from 192 on and nothing on 224 and 240: 1400 timed launches against the row's
    // price.  Wave-split-K launches are not dealt and priced by the CUs that the smallest engine leaves them (CuShare::even_cu).
    // Over 88 layers (65 linear, 23 convolutions), replayed from a graph with weights that no L2 holds, the picks cost on 144, 160, 176, 192, 208, 224 and
    // 240 CUs 3.0, 5.7, 2.9, 2.7, 2.2, 3.3 and 3.6 % more than the best plan; with all kernels priced as if the mask were even 30, 16, 6, 10, 17,
    // 13 and 4 % (1176 x 128 in nine taps of 128 on 144 CUs 22.0 us, now 8.0).
    // (A further 1.2 us on every tile, for inputs that the layer before has just written, made the 160 kinds of request above
    // 1.1 % slower, none faster by more than 1.5 % and ResNeXt at batch 8 on 160 CUs 651 us instead of 589; 2.4 us another 1.5 %.)
    // (13 carries 0.2 us more than it was fitted at: the copied tiles next to it have a shorter prologue since, 784 x 512 x 128 on 64 CUs takes
    // 4.6 us on it and 3.6 on 27.)
    // (17 lost 5 us of each launch to spilled registers when the rest was fitted.  Its rows, one for the layers of conv_gemm_is_copied and one for all
    // others, are set against 3, which has the same tile: 1536 x 4096 on 96 CUs, K = 128, 256, 512, 1024, 2048, 4096: 13.4, 16.1, 21.4, 32.1, 49.8,
    // 89.6 us on 3 and 14.0, 16.5, 21.3, 31.5, 46.7, 82.7 on 17, on 48 CUs 23.1, 28.1, 38.8, 60.2, 92.9, 168.8 and 24.3, 28.7, 38.7, 59.6, 87.5, 157.6;
    // in its general address form K = 264, 1032, 2056: 18.7, 38.6, 62.5 and 19.8, 38.7, 60.7.  With 4092 columns it is the faster one
    // at every K (256: 42.0 and 33.6), which the second row does not say.)
    // Layers that the copied tiles take in their fast form, of at least 512 rows and with sums of at least 768, have a table of their own, set by what gets
    // picked: 441 problems (linear layers of 512 to 3072 rows with and without GELU, 3 x 3 convolutions of 1568 to 50176 pixels; 48 to 256 CUs) x 15
    // tiles in chains with weights of their own (13, 15, 22, 23, 26 and 27 kept their rows).  Its picks took 2.3 % more than the best tile on the geometric mean and 56 % at worst, the other
    // table's, which has no 29 to 31, 4.1 and 90 % (1536 x 4096 x 1024 with GELU on 96 CUs 32.2 us, now 29.2, on 64 49.0, now 42.1; 2048 x 2304 x 768 on
    // 64 39.8, now 30.1; a 3 x 3 window of 50176 x 128 x 1152 on 96 49.2, now 45.5).  Shorter sums were not among them: with this table for all, three
    // co-located CNNs and encoders on 32 to 80 CUs took 2.3 % longer.  Of 29 to 31 a compute unit runs two at a time, in `two` times one's steps, and an odd
    // one alone.
    // GELU is priced there too: per 1000 outputs of a tile, `gelu` for the first workgroup of a compute unit and `gelu_more` for each further one.
    // It is 0.063 us per 1000 outputs wherever nothing runs beside a tile's epilogue; of workgroups that share a unit all but the first hide it under the others' K
    // loops.  Fitted to what GELU adds to 16 linear layers (512 to 3072 rows, sums of 768 to 3072) on 48, 64, 96, 128 and 256 CUs, 0.2 to 1.1 us rms of 0.5 to
    // 4.9.  (Six small tiles had paid nothing, which drew GELU layers to them: 768 x 3072 x 768 on 256 CUs 12.5 us on 26, 10.6 on 20.)
    // K in slices pays it in the launch that sums them (1.7 us on average over those layers), wave-split-K tiles by their wavefronts (0.3 to 2.8 us).
    // With GELU the picks for the 16 layers on eight shares (160, 176 and 192 too) take 1.3 % more than the best tile, without it 1.4.  Over 56 layers (44 linear ones of 512
    // to 3072 rows, 12 convolutions) x 8 or 13 shares without it the picks of this table take 2.3 % more than the best of 18 tiles and 50 % at worst, those of the
    // other one 4.4 and 84 %; of the 91 that differ 69 are faster by more than 3 %, 9 slower, by 8 % at worst (1536 x 4096 x 1024 on 160 CUs 23.7 us on 25, 25.8 on 24).
    struct LdsTile { int variant; double step, fixed, more, two, gelu, gelu_more; };
    static const LdsTile copied_256 = {17, 0.515, 9.7, 16.75, 0};
    static const std::vector<LdsTile> any = {
        {0, 0.509, 4.049, 7.322, 1.373}, {3, 0.568, 8.784, 16.049, 0}, {5, 0.595, 8.271, 16.021, 0}, {8, 0.525, 5.267, 9.068, 0},
        {13, 0.312, 2.898, 4.535, 1.656}, {15, 0.278, 3.194, 5.868, 1.418}, {16, 0.483, 4.611, 5.981, 0}, {17, 0.512, 10.9, 16.4, 0},
        {18, 0.552, 6.313, 10.504, 0}, {19, 0.579, 6.094, 8.303, 0}, {20, 0.337, 4.272, 6.499, 0}, {21, 0.444, 5.202, 8.054, 0},
        {22, 0.267, 3.021, 6.171, 1.444}, {23, 0.257, 3.012, 4.226, 1.544}, {24, 0.406, 8.399, 13.526, 0}, {25, 0.409, 8.333, 11.372, 0},
        {26, 0.176, 2.682, 3.32, 1.565}, {27, 0.177, 2.781, 4.298, 1.491}, {28, 0.222, 3.505, 5.135, 1.609}};
    static const std::vector<LdsTile> copied_long = {
        {13, 0.312, 2.898, 4.535, 1.656, 0.061, 0.000}, {15, 0.278, 3.194, 5.868, 1.418, 0.092, 0.002}, {16, 0.483, 4.611, 5.981, 0, 0.094, 0.033},
        {17, 0.515, 9.7, 7.009, 0, 0.065, 0.053}, {18, 0.558, 6.215, 5.632, 0, 0.056, 0.088}, {19, 0.545, 6.852, 5.409, 0, 0.056, 0.087},
        {20, 0.337, 4.272, 4.836, 0, 0.053, 0.085}, {21, 0.409, 5.709, 6.58, 0, 0.057, 0.086}, {22, 0.267, 3.021, 6.171, 1.444, 0.083, 0.010},
        {23, 0.257, 3.012, 4.226, 1.544, 0.077, 0.008}, {24, 0.372, 8.17, 8.751, 0, 0.064, 0.061}, {25, 0.35, 9.163, 8.532, 0, 0.061, 0.056},
        {26, 0.176, 2.682, 3.32, 1.565, 0.106, 0.007}, {27, 0.177, 2.781, 4.298, 1.491, 0.057, 0.000}, {28, 0.234, 4.367, 5.066, 1.549, 0.055, 0.001},
        {29, 0.3, 6.339, 4.349, 1.754, 0.059, 0.000}, {30, 0.286, 4.895, 4.854, 1.539, 0.058, 0.003}, {31, 0.291, 4.786, 5.235, 1.587, 0.057, 0.006}};
    for (const LdsTile &row : long_sums ? copied_long : any) {
        const LdsTile &c = row.variant == copied_256.variant && traits.copied && !long_sums ? copied_256 : row;
        if (c.fixed >= best) continue;                                   // planned anew for every launch: what cannot win is not worked out
        int bm, bn, bk;
        conv_gemm_tile(c.variant, &bm, &bn, &bk);
        const long KT = cdiv(K, bk), mn = cdiv(M, bm) * cdiv(N, bn);
        const bool dealt = mn > even_cu;
        // Dealing brings a shader engine's workgroups and its surplus in one row, and with room for two on a compute unit two may sit on one next to an idle one: 29 to
        // 31 take 0.9 to 1.8 times their price there, and which cannot be told from the sizes (160 tiles on 160 CUs 13.0 us, 176 on 176 29.8).  On 280 layers x
        // shares of 144 to 224 CUs their picks took 1.29 times as long as the next best's (30 for 1024 x 4096 x 1024 on 176 29.8, 18 17.3; 29 for
        // 3072 x 4096 x 1024 on 192 47.8, 17 30.4), by which the table was slower there than the other one, 3.4 % over the best tile instead of 2.7.
        if (pp_fast_forms_only(c.variant) && dealt && even_cu < n_cu) continue;
        for (long sp = 1; sp <= 4; sp *= 2) {
            if (sp > 1 && (K < 512 * sp || (size_t)(sp * M * N) > ws_floats)) break;
            // the table for long sums counts a launch on the block raster as eight times its heaviest XCD: 24 x 12 tiles of 128 x 256 (9 blocks) on 96 CUs
            // take 65.0 us, 24 x 9 (9 blocks as well, but 216 tiles, which are dealt in rows) 35.8
            const long wgs = long_sums && sp == 1 && mn >= 256 && cdiv(N, bn) >= 4 ? 8 * heaviest_xcd(cdiv(M, bm), cdiv(N, bn)) : mn * sp;
            const int cus = dealt || wgs <= even_cu ? n_cu : even_cu;            // few tiles in many slices: not dealt
            const double load = wgs >= cus ? 1.0 : (double)wgs / cus;
            double rounds = (double)cdiv(wgs, cus);
            const double per_cu = rounds;
            if (pp_fast_forms_only(c.variant)) rounds = (double)(cdiv(wgs, cus) / 2) * c.two + (double)(cdiv(wgs, cus) % 2);
            else if (c.two > 0.0 && rounds >= 2.0) rounds = c.two * ((double)wgs / cus > 2.0 ? (double)wgs / (2.0 * cus) : 1.0);
            double cost = c.fixed + (rounds - 1.0) * c.more + rounds * (double)cdiv(KT, sp) * c.step * (1.0 + 0.15 * load * load);
            if (dealt && even_cu < n_cu) cost += wgs <= n_cu ? 1.1 : even_cu < 0.8 * n_cu ? 3.0 * (0.8 - (double)even_cu / n_cu) : 0.0;
            if (sp > 1) cost += 15.48 + (double)M * N * (4.0 * sp + 2.0) / 4.243e6;
            if (long_sums && traits.gelu) cost += sp > 1 ? 5.2e-5 * M * N / n_cu : (c.gelu + (per_cu - 1.0) * c.gelu_more) * 1e-3 * bm * bn;
            if (cost < best) {
                best = cost;
                pl = GemmPlan{0, c.variant, 1, (int)mn, 4, 0};
                const long kt_per = cdiv(KT, sp);
                pl.splits = (int)cdiv(KT, kt_per);
            }
        }
    }
    // The patch kernel is not dealt either.  On the more uneven shares, beyond eight blocks of 16 x 16 outputs for every CU that the share counts as, the
    // dealt tiles are the safer choice: 28 x 28 x 128 at batch 3 and 8 8.1 and 10.5 us on 144 CUs, 10.6 and 23.0 here; 7.6 and 11.3 on 160, 7.1 and 13.0
    // here.  On 208 CUs (counted as 160) 56 x 56 x 64 at batch 4 takes 6.4 on the tiles and 5.2 here, on 112 (96) 7.0 and 6.0, 14 x 14 x 256 on 208 8 and 5.4.
    if (traits.conv3 && (even_cu >= 0.75 * n_cu || cdiv(M, 16) * cdiv(N, 16) <= 8l * even_cu))
        for (int v = 0; v < CONV3_VARIANTS; ++v)
            for (int nw = 2; nw <= 16; nw *= 2) {
                if (!conv3_launchable(v, nw, traits, (int)N)) continue;
                const double cost = conv3_cost(v, nw, traits, N, even_cu);
                if (cost < best) { best = cost; pl = GemmPlan{2, v, 1, (int)conv3_tiles(v, traits.B, traits.Ho, traits.Wo, (int)N), nw, 0}; }
            }
    if (pl.kind == 0) set_raster(pl, M, N);
    else if (pl.kind == 1) set_xcd_split(pl, M, N);
    *cost_out = pl.cost = best;
    return pl;
}
bool conv_gemm_is_copied(int KH, int KW, int Cin, int Cout) { return Cin % 32 == 0 && KH * KW <= 32 && Cout % 8 == 0; }

GemmPlan conv_gemm_plan(long M, long N, long K, int n_cu, size_t ws_floats, const GemmTraits &traits)
{
    double cost;
    return plan_with_cost(M, N, K, n_cu, ws_floats, traits, &cost);
}

// Two independent layers in one launch of the wave-split-K kernel: possible when both are planned on that kernel and
// one (tile, wavefront count) serves both at a modelled extra cost below what the second launch would cost.
// Plan for a first layer that reads the caller's NCHW tensor itself (see conv_wsk_kernel): the cheapest of the tile
// shapes that exist in that form, if it costs at most `stage_us` (the separate re-layout kernel it saves) more than
// the unrestricted plan.  (Shape by wsk_cost, as everywhere: ResNet-18 at batch 1 on 160 CUs 181 us, by wsk_whole_cost 188.)
bool conv_gemm_plan_stem(long M, long N, long K, int n_cu, size_t ws_floats, double stage_us, GemmPlan *out, int even_cu)
{
    if (getenv("ECLIP_GEMM_FORCE") || getenv("ECLIP_NO_PAIRS")) return false;
    if (even_cu <= 0) even_cu = n_cu;
    double any_cost;
    (void)plan_with_cost(M, N, K, n_cu, ws_floats, GemmTraits{false, even_cu}, &any_cost);
    double best = 1e30;
    int bv = -1;
    for (int v : {0, 1, 5}) {
        const double c = wsk_cost(M, N, K, even_cu, v, 4);
        if (c < best) { best = c; bv = v; }
    }
    if (bv < 0 || wsk_whole_cost(M, N, K, even_cu, bv, 4) > any_cost + stage_us) return false;
    int bm, bn;
    conv_wsk_tile(bv, &bm, &bn);
    GemmPlan pl{1, bv, 1, (int)(cdiv(M, bm) * cdiv(N, bn)), 4, 0};
    set_xcd_split(pl, M, N);
    *out = pl;
    return true;
}

bool conv_gemm_plan_pair(const GemmPlan &s0, long M0, long N0, long K0, int form0, const GemmPlan &s1, long M1, long N1, long K1, int form1, int n_cu,
                         GemmPlan *p0, GemmPlan *p1)
{
    if (getenv("ECLIP_GEMM_FORCE") || getenv("ECLIP_NO_PAIRS")) return false;
    if ((s0.kind != 1 && s0.cost <= 0.0) || (s1.kind != 1 && s1.cost <= 0.0)) return false;      // chosen by measurement: kept
    // all on the scale of the tiles' costs
    auto wsk = [&](bool lean, long M, long N, long K, int v, int nw) { return lean ? wsk_lean_cost(M, N, K, n_cu, v, nw) : wsk_whole_cost(M, N, K, n_cu, v, nw); };
    const double separate = (s0.kind == 1 ? wsk(form0 >= 0, M0, N0, K0, s0.variant, s0.nw) : s0.cost) +
                            (s1.kind == 1 ? wsk(form1 >= 0, M1, N1, K1, s1.variant, s1.nw) : s1.cost);
    const bool lean = conv_wsk_lean_pair_form(form0, form1) >= 0;      // the kernel that launch_conv_wsk_pair takes
    double best = 1e30;
    int bv = -1, bnw = 0;
    for (int v = 0; v < CONV_WSK_VARIANTS; ++v)
        for (int nw = 4; nw <= 16; nw *= 2) {
            const double c = wsk(lean, M0, N0, K0, v, nw) + wsk(lean, M1, N1, K1, v, nw);
            if (c < best) { best = c; bv = v; bnw = nw; }
        }
    const double launch_us = 2.5;                    // what a kernel costs as one more link of an in-order chain
    if (bv < 0 || best > separate + launch_us) return false;
    int bm, bn;
    conv_wsk_tile(bv, &bm, &bn);
    *p0 = GemmPlan{1, bv, 1, (int)(cdiv(M0, bm) * cdiv(N0, bn)), bnw, 0};
    *p1 = GemmPlan{1, bv, 1, (int)(cdiv(M1, bm) * cdiv(N1, bn)), bnw, 0};
    set_xcd_split(*p0, M0, N0);
    if (p0->tiles % 8 == 0) set_xcd_split(*p1, M1, N1);     // the second layer's workgroup b runs on XCD (tiles0 + b) % 8
    return true;
}

static GemmDev make_dev(const ConvGemmArgs &a, const GemmPlan &pl)
{
    GemmDev d;
    d.x = (const uint16_t *)a.x; d.w = (const uint16_t *)a.w; d.bias = (const uint16_t *)a.bias;
    d.res = (const uint16_t *)a.res; d.y = (uint16_t *)a.y; d.y32 = a.y32; d.ws = a.ws;
    d.B = a.B; d.H = a.H; d.W = a.W; d.Cin = a.Cin; d.Ho = a.Ho; d.Wo = a.Wo; d.KH = a.KH; d.KW = a.KW;
    d.stride = a.stride; d.pad = a.pad; d.act = a.act;
    d.M = a.B * a.Ho * a.Wo; d.N = a.Cout; d.K = a.KH * a.KW * a.Cin;
    d.nchw_c = a.nchw_c;
    d.ldx = a.ldx ? a.ldx : a.Cin;
    d.ldy = a.ldy ? a.ldy : a.Cout;
    d.x_bytes = (unsigned)((size_t)a.B * a.H * a.W * (a.nchw_c ? a.nchw_c : d.ldx) * 2);
    d.w_bytes = (unsigned)((size_t)((d.N + 15) / 16) * ((d.K + 31) / 32) * 1024);   // blocked layout, see ConvGemmArgs::w
    int bm, bn, bk = 32;
    if (pl.kind == 1) conv_wsk_tile(pl.variant, &bm, &bn);
    else conv_gemm_tile(pl.variant, &bm, &bn, &bk);
    d.KT = (d.K + bk - 1) / bk;
    d.splits = pl.splits;
    d.kt_per = (d.KT + pl.splits - 1) / pl.splits;
    d.tiles_m = (d.M + bm - 1) / bm;
    d.tiles_n = (d.N + bn - 1) / bn;
    d.raster = pl.raster;
    d.howo = magic_of((unsigned)(a.Ho * a.Wo >> (a.pool ? 2 : 0)));
    d.wo = magic_of((unsigned)(a.Wo >> (a.pool ? 1 : 0)));
    d.fast = magic_of((unsigned)(pl.raster == 3 ? d.tiles_n : d.tiles_m));
    return d;
}

// The patch kernel (whole windows lie in its blocks of 4 x 4 pixels) and the copied tiles with K in one piece, whose pooling form is compiled for windows
// over channels of whole K steps and for ReLU.
bool conv_gemm_pools(const ConvGemmArgs &a, const GemmPlan &pl)
{
    if (a.res || a.y32 || a.nchw_c || a.Ho % 2 || a.Wo % 2 || a.act != ACT_RELU) return false;
    if (pl.kind == 2) return true;
    if (pl.kind != 0 || pl.splits != 1 || a.Cout % 8 || a.KH * a.KW == 1 || tile_of_id(pl.variant).loop != LOOP_DMA) return false;
    return a.Cin % tile_of_id(pl.variant).bk == 0 && a.KH * a.KW <= 32;
}

hipError_t launch_conv_gemm(const ConvGemmArgs &a, const GemmPlan &pl, const SeDeal &deal, hipStream_t s, uint32_t *n_launched)
{
    if (a.pool && !conv_gemm_pools(a, pl)) return hipErrorInvalidValue;
    if ((a.ldx && (a.ldx % 8 || a.ldx < a.Cin || a.nchw_c)) || (a.ldy && (a.ldy % 8 || a.ldy < a.Cout || a.res || a.y32 || ((uintptr_t)a.y & 15))))
        return hipErrorInvalidValue;
    if (n_launched) *n_launched += pl.splits > 1 ? 2 : 1;
    if (pl.kind == 2) return launch_conv3(a, pl.variant, pl.nw, s);
    const GemmDev d = make_dev(a, pl);
    if (pl.kind == 1) return launch_conv_wsk(d, a.dtype, pl.variant, pl.nw, pl.tiles, s);
    if (a.dtype == DT_BF16) return launch_t<bf16_t>(d, pl, deal, s);
    return launch_t<f16_t>(d, pl, deal, s);
}

hipError_t launch_conv_gemm_pair(const ConvGemmArgs &a0, const GemmPlan &p0, const ConvGemmArgs &a1, const GemmPlan &p1, hipStream_t s,
                                 uint32_t *n_launched)
{
    if (p0.kind != 1 || p1.kind != 1 || p0.variant != p1.variant || p0.nw != p1.nw || a0.dtype != a1.dtype) return hipErrorInvalidValue;
    for (const ConvGemmArgs *a : {&a0, &a1})
        if ((a->ldx && (a->ldx % 8 || a->ldx < a->Cin || a->nchw_c)) || (a->ldy && (a->ldy % 8 || a->ldy < a->Cout || a->res || a->y32 || ((uintptr_t)a->y & 15))))
            return hipErrorInvalidValue;
    if (n_launched) *n_launched += 1;
    return launch_conv_wsk_pair(make_dev(a0, p0), p0.tiles, make_dev(a1, p1), p1.tiles, a0.dtype, p0.variant, p0.nw, s);
}

}  // namespace eclip
