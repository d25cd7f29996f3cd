// The LDS-tiled matrix-core kernel whose operand tiles are copied straight from memory into LDS (implicit-GEMM convolution /
// linear layer; same contraction, weights layout and epilogue as conv_gemm_kernel in gemm_tile.h).
//
// What bounds this class of kernel is the path into a compute unit, not its matrix pipes: conv_gemm_kernel brings the weights
// of a tile column in once per wavefront that needs them and moves the activations through registers, and its 128 x 128 tile
// takes 0.47-0.67 us per K step of 64 where the matrix instructions need 0.21.  Here both operands cross that path once,
// land in LDS without passing registers (buffer_load_dwordx4 ... lds), several K steps ahead, and four wavefronts with
// square sub-tiles read every LDS byte as rarely as a workgroup tile allows:
//   - a ring of ST stages of BK = 64 or 32; the loads of K step t + ST go out as soon as every wavefront has read step t;
//   - fragments are read half a step ahead of the matrix instructions that use them, and loads, LDS reads and matrix
//     instructions are interleaved one by one: a SIMD has one wavefront, so nothing else would fill its gaps;
//   - LDS positions: the weights in the order of their 1 KB blocks (a fragment is 1 KB in a row); a row of the activation
//     tile is 128 (64) bytes, its 16-byte chunk c at position c ^ (row / 2 % 8) (c ^ (row / 4 % 4)), so that 16 lanes reading
//     one chunk of 16 consecutive rows touch all banks once, while the lanes that load a row still read it in one piece.
#pragma once
#include "gemm_tile.h"

// The compiler calls m0 reserved and warns of every statement that names it; it does take the name as a definition of m0.
#pragma clang diagnostic ignored "-Winline-asm"

namespace eclip {

// Copies 16 bytes per lane from `rsrc` (byte offset voff + soff; zeros beyond its end) to LDS byte lds + AT + 16 * lane.  Written out
// because the compiler would otherwise wait for every such load before any later LDS read; the waits are explicit.  m0 holds the
// LDS address of the copy and belongs to the compiler, which uses it too: it is named as overwritten.
template <unsigned AT>
__device__ __forceinline__ void dma_lds16(u32x4 rsrc, unsigned voff, unsigned soff, unsigned lds)
{
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff), "n"(AT) : "memory", "m0", "scc");
}

// Waits until at most VM of this wavefront's memory accesses and (LGKM) none of its LDS accesses are outstanding, then for all
// wavefronts of the workgroup.  To the compiler s_barrier itself touches no memory, so an LDS read of what another wavefront copies
// could be moved in front of a bare one: the wait and the barrier are one statement that reads of memory do not pass.
template <int VM, bool LGKM = true> __device__ __forceinline__ void wait_and_meet()
{
    if constexpr (LGKM) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(VM) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(VM) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Accumulators that leave no room for the rest in the 256 vector registers go to the accumulation registers (one wavefront
// per SIMD has both files).  The matrix instruction is then written out: left to itself the compiler copies accumulators
// between registers around every instruction.
// They have to fit there (dma_acc_fit): accumulators that the compiler moves between the files next to such an instruction are read before they are written.
// Two wavefronts on a SIMD have 128 accumulation registers each, which is less than any such tile needs; one has 256.
constexpr bool dma_acc_in_agprs(int bm, int bn, int waves) { return bm * bn / waves > 128 * 64; }
constexpr int dma_per_cu(int bm, int bn, int bk, int stages) { return dma_lds_bytes(bm, bn, bk, stages) > 80 * 1024 ? 1 : 2; }      // workgroups that the registers are for
constexpr bool dma_acc_fit(int bm, int bn, int bk, int stages, int waves)
{
    return !dma_acc_in_agprs(bm, bn, waves) || (bm * bn / waves <= 256 * 64 && waves * dma_per_cu(bm, bn, bk, stages) <= 4);
}
template <typename T> __device__ __forceinline__ void mma_agpr(uint4 a, uint4 b, f32x4 &c)
{
    const u32x4 va = {a.x, a.y, a.z, a.w}, vb = {b.x, b.y, b.z, b.w};
    if constexpr (std::is_same<T, bf16_t>::value) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(va), "v"(vb));
    else asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(va), "v"(vb));
}

// Accumulators of two blocks (of one) for an epilogue.  Those in accumulation registers are fetched by statements of their own: left to
// the compiler, with two epilogues to choose from, it moves them to vector registers before the branch and spills what does not fit
// (60 registers of the 256 x 256 tile, whose every launch paid for it whichever epilogue ran).  The compiler does not see that
// v_permlane16_swap, which follows, must stay clear of them.
template <bool AGPR> __device__ __forceinline__ void acc_pair(const f32x4 &a, const f32x4 &b, unsigned (&v)[8])
{
    if constexpr (AGPR) {
        asm volatile("v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\tv_accvgpr_read_b32 %2, %10\n\tv_accvgpr_read_b32 %3, %11\n\t"
                     "v_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\tv_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15\n\ts_nop 3"
                     : "=v"(v[0]), "=v"(v[1]), "=v"(v[2]), "=v"(v[3]), "=v"(v[4]), "=v"(v[5]), "=v"(v[6]), "=v"(v[7])
                     : "a"(a[0]), "a"(a[1]), "a"(a[2]), "a"(a[3]), "a"(b[0]), "a"(b[1]), "a"(b[2]), "a"(b[3]));
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) { v[c] = __float_as_uint(a[c]); v[4 + c] = __float_as_uint(b[c]); }
    }
}
__device__ __forceinline__ uint4 acc_agpr(const f32x4 &a)
{
    uint4 v;
    asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7"
                 : "=v"(v.x), "=v"(v.y), "=v"(v.z), "=v"(v.w) : "a"(a[0]), "a"(a[1]), "a"(a[2]), "a"(a[3]));
    return v;
}

// Forms of the kernel (conv_gemm_dma_kernel)
enum { DMA_PLAIN, DMA_F32, DMA_POOL };

// Epilogue for outputs of the storage type, or (DMA_F32) float ones, or (DMA_POOL) their maxima over windows, with N a multiple of 8 (the rest goes through tile_epilogue).  One wavefront per SIMD
// has nobody to hide behind, so this one is kept short and straight: buffer stores that drop what lies beyond M or N instead
// of a branch per store, accumulators taken block row by block row.
// (256 x 192 tile: 5.5 us with
// the general epilogue, 5.0 with this one.  Passing the accumulators through LDS to a short rolled loop was slower, 7 us.)
template <typename T, int BM, int BN, int WM, int WN, int TM, int TN, int ACT, bool RES, bool EARLY, int FORM>
__device__ __forceinline__ void dma_epilogue(const GemmDev &p, f32x4 (&acc)[TM][TN], const u32x4 (&bq)[TN / 2], int m_base, int n_base, int wm, int wn)
{
    static_assert(TN % 2 == 0, "pairs of blocks");
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63, q = lane >> 4;
    const int m0 = m_base + wm * (BM / WM) + (lane & 15), n0 = n_base + wn * (BN / WN) + 16 * (q & 1) + 8 * (q >> 1);   // see tile_epilogue_impl
    constexpr unsigned OOB = 0xffffffffu;
    constexpr bool F32 = FORM == DMA_F32;
    constexpr int WIN = FORM == DMA_POOL ? 4 : 1;                      // rows of the tile per row of y
    const unsigned bytes = (unsigned)(((size_t)(p.M / WIN - 1) * p.ldy + p.N) * 2);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(F32 ? (void *)p.y32 : (void *)p.y, 0, (int)(F32 ? 2u * bytes : bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)(RES ? p.res : p.y), 0, (int)bytes, 0x00020000);
    unsigned off[TN / 2];
    float bv[TN / 2][8];
    static_for<TN / 2>([&](auto jc) {
        constexpr int jp = decltype(jc)::value;
        off[jp] = n0 + 32 * jp < p.N ? ((unsigned)(m0 / WIN) * (unsigned)p.ldy + (unsigned)(n0 + 32 * jp)) * 2u : OOB;
#pragma unroll
        for (int e = 0; e < 8; ++e) bv[jp][e] = 0.f;
        if constexpr (EARLY) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { bv[jp][2 * e] = Cvt<T>::from_bits(bq[jp][e] & 0xffffu); bv[jp][2 * e + 1] = Cvt<T>::from_bits(bq[jp][e] >> 16); }
        } else if (p.bias && n0 + 32 * jp < p.N) Pack<T, 8>::load(reinterpret_cast<const T *>(p.bias) + n0 + 32 * jp, bv[jp]);
    });
    const unsigned row16 = 32u / WIN * (unsigned)p.ldy;
    u32x4 rq[2][TN / 2];
    auto load_res = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (RES && i < TM)
            static_for<TN / 2>([&](auto jc) {
                constexpr int jp = decltype(jc)::value;
                rq[i & 1][jp] = __builtin_amdgcn_raw_buffer_load_b128(rr, m0 + 16 * i < p.M ? off[jp] : OOB, (int)(row16 * i), 0);
            });
    };
    load_res(std::integral_constant<int, 0>{});
    static_for<TM>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        load_res(std::integral_constant<int, i + 1>{});
        static_for<TN / 2>([&](auto jc) {
            constexpr int jp = decltype(jc)::value;
            float o[8];
            unsigned ab[8];
            acc_pair<!EARLY>(acc[i][2 * jp], acc[i][2 * jp + 1], ab);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const u32x2 sw = __builtin_amdgcn_permlane16_swap(ab[c], ab[4 + c], false, false);
                o[c] = __uint_as_float(sw[0]);
                o[4 + c] = __uint_as_float(sw[1]);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += bv[jp][e];
            if constexpr (RES) {
                const u32x4 w = rq[i & 1][jp];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[2 * e] += Cvt<T>::from_bits(w[e] & 0xffffu);
                    o[2 * e + 1] += Cvt<T>::from_bits(w[e] >> 16);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = apply_act_c<ACT>(o[e]);
            if constexpr (FORM == DMA_POOL) {                          // lanes 4 w .. 4 w + 3 hold window w
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    o[e] = fmaxf(o[e], __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(o[e]), 0xb1, 0xf, 0xf, true)));        // quad_perm 1 0 3 2
                    o[e] = fmaxf(o[e], __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(o[e]), 0x4e, 0xf, 0xf, true)));        // quad_perm 2 3 0 1
                }
            }
            // The row's offset goes into the vector offset here, not into the scalar one: with a scalar-register offset the compiler
            // leaves no gap between a 16-byte store and the next write of its data registers, and on this GPU the store then
            // now and then takes the new values (only with several workgroups on the CU).
            const bool ok = m0 + 16 * i < p.M && n0 + 32 * jp < p.N && (WIN == 1 || (lane & 3) == 0);
            u32x4 v;
            if constexpr (F32) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(o[4 * h + e]);
                    __builtin_amdgcn_raw_buffer_store_b128(v, ry, ok ? 2u * (off[jp] + row16 * i) + 16u * h : OOB, 0, 0);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = Cvt<T>::pack2(o[2 * e], o[2 * e + 1]);
                __builtin_amdgcn_raw_buffer_store_b128(v, ry, ok ? off[jp] + row16 * i : OOB, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    });
}

// What dma_epilogue does not take (N not a multiple of 8, slices of K), for the tiles whose accumulators fill the
// accumulation registers.  tile_epilogue, made for tiles with registers to spare, cost the 256 x 256 tile 60 spilled ones:
// here half the sub-tile goes through the wavefront's own part of LDS to one short loop.  With acc_pair, 1536 x 4096 x 1024 on 96 CUs:
// 32.0 -> 27.0 us on 256 x 256 tiles, 1536 x 3072 x 1024 24.3 -> 23.2 on 256 x 192, 26.3 -> 25.7 on 192 x 256.
template <typename T, int BM, int BN, int WM, int WN, int TM, int TN>
__device__ __forceinline__ void dma_epilogue_rest(const GemmDev &p, f32x4 (&acc)[TM][TN], uint16_t *smem, int m_base, int n_base, int wm, int wn, int z)
{
    static_assert(TM % 2 == 0, "two halves");
    constexpr int ROWS = TM * 8, COLS = TN * 16, SP = COLS + 4;
    const int lane = threadIdx.x & 63;
    float *stage = reinterpret_cast<float *>(smem) + (wm * WN + wn) * (ROWS * SP);
    __syncthreads();                                                   // everyone is done with the ring
    static_for<2>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        static_for<TM / 2>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            static_for<TN>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const f32x4 a = acc[h * (TM / 2) + i][j];
                *reinterpret_cast<uint4 *>(&stage[(i * 16 + (lane & 15)) * SP + j * 16 + (lane >> 4) * 4]) = acc_agpr(a);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_s_waitcnt(0xc07f);                            // lgkmcnt(0): this wavefront's LDS writes have landed
#pragma unroll 1
        for (int t = lane; t < ROWS * (COLS / 4); t += 64) {
            const int r = t / (COLS / 4), c = (t - r * (COLS / 4)) * 4;
            const int m = m_base + wm * (BM / WM) + h * ROWS + r, n = n_base + wn * (BN / WN) + c;
            const float4 q = *reinterpret_cast<const float4 *>(&stage[r * SP + c]);
            const f32x4 v = {q.x, q.y, q.z, q.w};
            if (p.splits != 1) {
                if (m >= p.M || n >= p.N) continue;
                float *dst = p.ws + ((long)z * p.M + m) * p.N + n;
                if ((p.N & 3) == 0) {
                    *reinterpret_cast<float4 *>(dst) = q;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < p.N) dst[e] = v[e];
                }
            } else {
#define EPI(A) epilogue_store<T, A>(p.bias, p.res, p.y, p.y32, p.M, p.N, m, n, v, 4, p.ldy)
                ECLIP_ACT_SWITCH(p.act, EPI)
#undef EPI
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_s_waitcnt(0xc07f);                            // reads done before the second half overwrites the buffer
    });
}

// Touches one 128-byte line per lane (4 bytes each go to LDS bytes lds .. lds + 255, which nobody reads).
__device__ __forceinline__ void dma_touch(u32x4 rsrc, unsigned voff, unsigned soff, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}

// Raster, from bit 8 on the shift of the division by the tiles of the walk's first dimension, and two flags: pixel m is row m (stride 1,
// no padding; asked for 1 x 1 windows), the workgroups are dealt (se_deal.h).
enum : unsigned { DMA_ROWS = 1u << 16, DMA_DEALT = 1u << 17 };
inline unsigned dma_walk(const GemmDev &d, const SeDeal &deal)
{
    return (unsigned)d.raster | d.fast.shift << 8 | (d.stride == 1 && d.pad == 0 ? DMA_ROWS : 0u) | (deal.level ? DMA_DEALT : 0u);
}

// Layers that take the F32 form of their tile (conv_gemm_dma_kernel).
inline bool dma_writes_floats(const GemmDev &d) { return d.y32 && d.splits == 1 && d.N % 8 == 0; }

// A position in the ring of stages: a constant, or a number carried in a register.
template <typename S> struct RingPos {
    static constexpr unsigned fixed = S::value;
    __device__ static __forceinline__ unsigned moving(S) { return 0u; }
};
template <> struct RingPos<unsigned> {
    static constexpr unsigned fixed = 0u;
    __device__ static __forceinline__ unsigned moving(unsigned s) { return s; }
};

// n bits (0 to 32) from bit `at` on
__device__ __forceinline__ unsigned bits_run(int at, int n) { return (n >= 32 ? ~0u : (1u << n) - 1u) << (at & 31); }

// DMA_F32: the form of the tiles whose accumulators fill the accumulation registers for layers that write floats (dma_writes_floats).  It is a kernel of
// its own: as one more branch its epilogues cost the launches that do not take them 0.5 % of the stress mix, with no instruction more
// executed but the code further apart.  (Through dma_epilogue_rest, whose short loop waits for its bias on every turn, requests of one layer with
// float outputs took: 3000 x 4096 x 1024 on 96 CUs 97 us, now 74, on 64 CUs 136, now 98; 1536 x 3000 x 1024 on 96 48, now 39; 1005 x 3072 x 768 on 64
// 43, now 33.)
// DMA_POOL (A_UNIFORM, ReLU): the rows of the tile are the pixels of 2 x 2 windows, window by window, so that four neighbouring lanes hold a window and its
// maximum costs two lane exchanges: the pool's launch goes, and three quarters of the stores (gemm_pools).
template <typename T, int BM, int BN, int BK, int WM, int WN, int ST, int AMODE, int FORM = DMA_PLAIN>
__global__ __launch_bounds__(WM * WN * 64, dma_per_cu(BM, BN, BK, ST)) void conv_gemm_dma_kernel(const uint16_t *x, const uint16_t *w, unsigned x_bytes, int M, int N, int K, int ldx, int kt_per, unsigned walk, unsigned tiles,
                          unsigned fast_d, unsigned fast_mul, GemmDev p, SeDeal deal)
{
    // What the first copies need comes as 14 words of separate arguments, which the hardware puts into scalar registers before the
    // wavefront starts (dma_walk packs the last things); what the other forms need beyond that is fetched together.
    p.x = x; p.w = w; p.x_bytes = x_bytes; p.M = M; p.N = N; p.K = K; p.ldx = ldx; p.kt_per = kt_per; p.KT = (K + BK - 1) / BK;
    p.raster = (int)(walk & 255u);
    p.fast = Magic{fast_d, fast_mul, walk >> 8 & 255u};
    p.w_bytes = (unsigned)((N + 15) >> 4) * (unsigned)((K + 31) >> 5) * 1024u;
    if constexpr (AMODE != A_MATRIX)
        asm volatile("" : "+s"(p.H), "+s"(p.W), "+s"(p.Cin), "+s"(p.KH), "+s"(p.KW), "+s"(p.stride), "+s"(p.pad), "+s"(p.howo.d), "+s"(p.howo.mul),
                     "+s"(p.howo.shift), "+s"(p.wo.d), "+s"(p.wo.mul), "+s"(p.wo.shift));
    constexpr int NW = WM * WN, KS = BK / 32;                           // KS: matrix instructions along K per step and block
    static_assert(KS == 1 || KS == 2, "K step of 32 or 64");
    static_assert(dma_acc_fit(BM, BN, BK, ST, NW), "accumulators fit the accumulation registers");
    constexpr int TM = BM / WM / 16, TN = BN / WN / 16, NM = TM * TN;
    constexpr int RPC = 16 / KS, CPR = 4 * KS;                          // rows per 1 KB copy of the activations, 16-byte chunks per row
    constexpr int AI = BM / RPC / NW, BI = BN / 16 * KS / NW;           // 1 KB copies per wavefront and step
    static_assert(AI * RPC * NW == BM && BI * 16 * NW == BN * KS && TM * 16 * WM == BM && TN * 16 * WN == BN, "whole copies and blocks per wavefront");
    constexpr int TOUCH = AMODE == A_MATRIX && dma_touches(BM, BN, BK, ST) ? 1 : 0;
    constexpr unsigned STAGE = (BM + BN) * BK * 2u;                        // bytes: activations, then weights
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    int tile_m, tile_n;
    const uint32_t bid = walk & DMA_DEALT ? se_dealt_block(deal, blockIdx.x) : blockIdx.x;
    if (bid == 0xffffffffu || !gemm_tile_of(p, tiles, bid, tile_m, tile_n)) return;
    const int m_base = tile_m * BM, n_base = tile_n * BN;
    constexpr unsigned OOB = 0xffffffffu;
    u32x4 rx, rw;
    rx.x = (unsigned)(uintptr_t)p.x; rx.y = (unsigned)((uintptr_t)p.x >> 32) & 0xffffu; rx.z = p.x_bytes; rx.w = 0x00020000u;
    rw.x = (unsigned)(uintptr_t)p.w; rw.y = (unsigned)((uintptr_t)p.w >> 32) & 0xffffu; rw.z = p.w_bytes; rw.w = 0x00020000u;

    // ---- per-lane addressing that does not change along K: copy i of this wavefront is rows RPC (AI * wave + i) .. of the tile
    const int KB = (p.K + 31) >> 5, NB = (p.N + 15) >> 4;
    const bool rows = walk & DMA_ROWS;                                // A_MATRIX: row m of the operand is pixel m
    bool a_ok[AI];
    unsigned a_off[AI];                      // byte offset of this lane's chunk at window tap (0, 0), channel 0 (modulo 2^32 when padded)
    int a_ih0[AI], a_iw0[AI];
    // position of chunk c of a row: c ^ swizzle(row).  (A_GENERAL with 128-byte rows: the same chunk in every copy of a lane)
    auto swizzle = [](int row) { return KS == 1 ? (row >> 2) & 3 : AMODE == A_GENERAL ? row & 7 : (row >> 1) & 7; };
    int kc = 0;                              // A_GENERAL: first k of this lane's chunk within a step (the same in every copy)
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        const int row = (AI * wave + i) * RPC + lane / CPR, m = m_base + row;
        const int chunk = lane % CPR ^ swizzle(row);
        if (AMODE == A_GENERAL) kc = chunk * 8;
        a_ok[i] = m < p.M;
        const int mm = a_ok[i] ? m : 0;
        if (AMODE == A_MATRIX && rows) {
            a_off[i] = (unsigned)mm * (unsigned)p.ldx * 2u;
        } else {
            const int win = FORM == DMA_POOL ? mm >> 2 : mm;
            const int b = (int)div_by((unsigned)win, p.howo), r = win - b * (int)p.howo.d;
            int oh = (int)div_by((unsigned)r, p.wo), ow = r - oh * (int)p.wo.d;
            if constexpr (FORM == DMA_POOL) {
                oh = 2 * oh + (mm >> 1 & 1);
                ow = 2 * ow + (mm & 1);
            }
            a_ih0[i] = oh * p.stride - p.pad;
            a_iw0[i] = ow * p.stride - p.pad;
            a_off[i] = (unsigned)((b * p.H + a_ih0[i]) * p.W + a_iw0[i]) * (unsigned)p.ldx * 2u;
        }
        if (AMODE != A_GENERAL) a_off[i] += (unsigned)chunk * 16u;
        if (AMODE == A_MATRIX && !a_ok[i]) a_off[i] = OOB;
    }
    // A_UNIFORM: bit t of a_out says that the row has no pixel under tap t = kh * KW + kw (at most 32 taps, see gemm_amode), so that
    // a copy's offset costs three vector instructions; tests of the borders go through scalar masks, and a lone wavefront
    // waits out every hop between its vector and scalar halves (128 x 128 tile, 3 x 3 window, 72 K steps: 36.6 -> 33.0 us).
    unsigned a_out[AI];
    if (AMODE == A_UNIFORM) {
        unsigned starts = 0;                                            // the first tap of every window row
#pragma unroll 1
        for (int h = 0; h < p.KH; ++h) starts |= 1u << (h * p.KW);
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            // taps of columns lo_w .. and rows lo_h .. lie inside the image: a run of bits repeated in a run of rows
            const int lo_w = max(-a_iw0[i], 0), n_w = max(min(p.W - a_iw0[i], p.KW) - lo_w, 0);
            const int lo_h = max(-a_ih0[i], 0), n_h = max(min(p.H - a_ih0[i], p.KH) - lo_h, 0);
            a_out[i] = a_ok[i] ? ~(bits_run(lo_w, n_w) * (starts & bits_run(lo_h * p.KW, n_h * p.KW))) : ~0u;
        }
    }
    unsigned b_off[BI];                      // copy i: weight block (row block (BI * wave + i) / KS, k block (BI * wave + i) % KS of the step)
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int blk = BI * wave + i, nb = (n_base >> 4) + blk / KS;
        b_off[i] = nb < NB ? ((unsigned)(nb * KB + blk % KS) * 64u + (unsigned)lane) * 16u : OOB;
    }

    // ---- position along K of the step copied next
    const int kt_begin = blockIdx.y * p.kt_per, kt_end = min(p.KT, kt_begin + p.kt_per);
    int kt_run = kt_begin;
    int k_run = kt_begin * BK + kc, kh = 0, kw = 0, ci = AMODE == A_GENERAL ? k_run : kt_begin * BK;   // uniform but for A_GENERAL
    if (AMODE != A_MATRIX && p.KH * p.KW != 1) {
        const int tap = ci / p.Cin;
        ci -= tap * p.Cin;
        kh = tap / p.KW;
        kw = tap - kh * p.KW;
    }
    unsigned tap_off = (unsigned)((kh * p.W + kw) * p.ldx + ci) * 2u;
    int tap = kh * p.KW + kw;                                         // A_UNIFORM (uniform)
    const int k_lim = min(p.K, kt_end * BK), kb_lim = min(KB, kt_end * KS);
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)smem;
    // Copies beyond the end of the slice read nothing: the descriptors are emptied when the slice ends, so the loads in flight stay
    // countable.  LDS positions are a scalar per wavefront and a constant.
    const unsigned lds_a = lds0 + (unsigned)(AI * wave) * 1024u, lds_b = lds0 + BM * BK * 2u + (unsigned)(BI * wave) * 1024u;
    unsigned a_soff = (unsigned)kt_begin * (BK * 2u), b_soff = (unsigned)kt_begin * (KS * 1024u);
    auto copy_a = [&](auto ic, auto slot) {
        constexpr int i = decltype(ic)::value;
        unsigned v = a_off[i], s = 0;
        if (AMODE == A_MATRIX) s = a_soff;
        else if (AMODE == A_UNIFORM) v = (v + tap_off) | (unsigned)((int)(a_out[i] << (31 - tap)) >> 31);
        else {
            const int ok = (int)a_ok[i] & (int)((unsigned)(a_ih0[i] + kh) < (unsigned)p.H) & (int)((unsigned)(a_iw0[i] + kw) < (unsigned)p.W) &
                           (int)(k_run < k_lim);
            v = ok ? v + tap_off : OOB;
        }
        dma_lds16<RingPos<decltype(slot)>::fixed + i * 1024u>(rx, v, s, lds_a + RingPos<decltype(slot)>::moving(slot));
    };
    auto copy_b = [&](auto ic, auto slot) {
        constexpr int i = decltype(ic)::value;
        u32x4 r = rw;
        if (AMODE == A_GENERAL) r.z = kt_run * KS + (BI * wave + i) % KS < kb_lim ? p.w_bytes : 0u;
        const unsigned soff = AMODE == A_GENERAL ? (unsigned)__builtin_amdgcn_readfirstlane((int)b_soff) : b_soff;   // (of 128 x 64 x 32 it lands in a vector register)
        dma_lds16<RingPos<decltype(slot)>::fixed + i * 1024u>(r, b_off[i], soff, lds_b + RingPos<decltype(slot)>::moving(slot));
    };
    // The weights of a large model are in no cache: the workgroups that share a tile column (and an L2) take turns touching the
    // lines of the step PD steps ahead of the copies (BERT-large FFN2 on 96 CUs, served: 36 -> 31 us; with the weights in the
    // last-level cache it costs 1 us of 28).
    constexpr int PD = 6, LINES = BN * BK / 64;                         // 128-byte lines of a step's weights
    const int share = p.raster == 2 ? p.tiles_m : (p.tiles_m + 7) >> 3, part = p.raster == 2 ? tile_m : tile_m >> 3;
    const unsigned t_line = (unsigned)(wave * 64 + lane), t_blk = t_line / (8 * KS);
    const unsigned t_off = t_line < LINES ? ((unsigned)((n_base >> 4) + (int)t_blk) * (unsigned)KB * 1024u + (t_line % (8 * KS)) * 128u) : OOB;
    int turn = kt_begin + part + PD < kt_end ? part : 1 << 30;        // steps until this workgroup's next turn
    const u32x4 rw_all = rw, rw_none = {rw.x, rw.y, 0u, rw.w};
    auto touch_b = [&]() {
        if (--turn < 0) {
            dma_touch(rw_all, t_off, b_soff + PD * (KS * 1024u), lds0 + ST * STAGE);
            turn = kt_run + share + PD < kt_end ? share - 1 : 1 << 30;
        } else {
            dma_touch(rw_none, t_off, 0, lds0 + ST * STAGE);          // as many accesses in flight as in the other branch
        }
    };
    auto advance = [&]() {
        ++kt_run;
        a_soff += BK * 2u;
        b_soff += KS * 1024u;
        if (AMODE != A_GENERAL && kt_run == kt_end) {
            asm volatile("");                                          // a branch: as selects the descriptors would move every step
            rx.z = rw.z = 0u;
        }
        if (AMODE == A_UNIFORM) {
            ci += BK;
            if (ci >= p.Cin) {
                ci = 0;
                ++tap;
                if (++kw == p.KW) { kw = 0; ++kh; }
            }
        } else if (AMODE == A_GENERAL) {
            k_run += BK;
            ci += BK;
#pragma unroll
            for (int u = 0; u < BK / 8; ++u) {       // Cin >= 8
                const int wrap = ci >= p.Cin;
                ci -= wrap ? p.Cin : 0;
                kw += wrap;
                const int wrap2 = kw == p.KW;
                kw = wrap2 ? 0 : kw;
                kh += wrap2;
            }
        }
        if (AMODE != A_MATRIX) tap_off = (unsigned)((kh * p.W + kw) * p.ldx + ci) * 2u;
    };

    // ---- fragments: half ks of a step
    const int r15 = lane & 15;
    const unsigned a_rd0 = (unsigned)(wm * (BM / WM) + r15) * (BK * 2u) + (unsigned)((lane >> 4) ^ swizzle(r15)) * 16u;
    const unsigned b_rd0 = BM * BK * 2u + (unsigned)(wn * (BN / WN) / 16) * (KS * 1024u) + (unsigned)lane * 16u;
    uint4 fa[2][TM], fb[2][TN];
    const char *lds_c = reinterpret_cast<const char *>(smem);
    auto read_one = [&](auto qc, auto setc, auto slot) {            // q-th of the TM + TN fragments of half step ks into register set `set`
        constexpr int q = decltype(qc)::value, set = decltype(setc)::value, ks = KS == 2 ? set : 0;
        if constexpr (q < TN) fb[set][q] = *reinterpret_cast<const uint4 *>(lds_c + slot + b_rd0 + q * (KS * 1024) + ks * 1024);
        else fa[set][q - TN] = *reinterpret_cast<const uint4 *>(lds_c + slot + (a_rd0 ^ (ks * 64u)) + (q - TN) * (BK * 32));
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // copies per step; with two half steps the last L - L2 of them go out in the first half of the next one
    constexpr int L = AI + BI + TOUCH, L2 = KS == 2 ? L / 2 : L, R = TM + TN;
    auto copy = [&](auto qc, auto slot) {
        constexpr int q = decltype(qc)::value;
        if constexpr (q < AI) copy_a(qc, slot);
        else if constexpr (q < AI + BI) copy_b(std::integral_constant<int, q - AI>{}, slot);
        else touch_b();
    };
    // The matrix instructions of register set `set`, copies C0 .. C0 + C - 1 of a step and the reads of the other register set, spread
    // evenly: a burst of copies fills the queue towards memory (64 bytes per clock), and a wavefront waiting to issue a copy
    // issues no matrix instructions either (128 x 128 tile, K step of 64: 0.40 us with the copies in one half, 0.35 spread).
    auto half_step = [&](auto setc, auto c0c, auto cc, auto copy_slot, auto read_slot) {
        constexpr int set = decltype(setc)::value, C0 = decltype(c0c)::value, C = decltype(cc)::value, Q = C + R;
        static_for<NM>([&](auto mc) {
            constexpr int m = decltype(mc)::value, i = m / TN, j = m % TN;
            if constexpr (dma_acc_in_agprs(BM, BN, NW)) mma_agpr<T>(fb[set][j], fa[set][i], acc[i][j]);
            else acc[i][j] = Mma<T>::run(fb[set][j], fa[set][i], acc[i][j]);
            constexpr int q0 = m * Q / NM, q1 = (m + 1) * Q / NM;
            static_for<q1 - q0>([&](auto dc) {
                constexpr int q = q0 + decltype(dc)::value, c0 = q * C / Q, c1 = (q + 1) * C / Q;
                if constexpr (c1 > c0) copy(std::integral_constant<int, C0 + c0>{}, copy_slot);
                else read_one(std::integral_constant<int, q - c0>{}, std::integral_constant<int, 1 - set>{}, read_slot);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using IL2 = std::integral_constant<int, L2>;
    using IL1 = std::integral_constant<int, L - L2>;
    // The bias of this wavefront's channels is on its way before the first operand, where the registers allow: the epilogue
    // starts with the accumulators, not with a trip to memory.
    constexpr bool EARLY = !dma_acc_in_agprs(BM, BN, NW);
    u32x4 bq[TN / 2];
    if constexpr (EARLY) {
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias, 0, p.bias ? p.N * 2 : 0, 0x00020000);
        const int n0 = n_base + wn * (BN / WN) + 16 * ((lane >> 4) & 1) + 8 * (lane >> 5);
#pragma unroll
        for (int jp = 0; jp < TN / 2; ++jp) bq[jp] = __builtin_amdgcn_raw_buffer_load_b128(rb, n0 + 32 * jp < p.N ? (unsigned)(n0 + 32 * jp) * 2u : OOB, 0, 0);
    }
    static_for<ST>([&](auto sc) {
        constexpr int st = decltype(sc)::value;
        static_for<(st == ST - 1 ? L2 : L)>([&](auto qc) { copy(qc, std::integral_constant<unsigned, st * STAGE>{}); });
        if constexpr (st < ST - 1 || KS == 1) advance();
    });
    wait_and_meet<(ST - 2) * L + L2, false>();
    static_for<R>([&](auto qc) { read_one(qc, I0{}, std::integral_constant<unsigned, 0u>{}); });

    // Every wavefront has read all of the current step and its copies of the next one have landed; after the barrier so have everyone's
    auto meet = [&]() { wait_and_meet<(ST - 2) * L>(); };
    int kt = kt_begin;
    if constexpr (dma_acc_in_agprs(BM, BN, NW)) {
        // the largest tiles carry the stage in a register: their matrix instructions leave time for it, and unrolled over the ring
        // they would spill 80 registers
        auto after = [&](unsigned slot) { return slot + STAGE == ST * STAGE ? 0u : slot + STAGE; };
        static_assert(KS == 1, "two steps per turn");
        unsigned slot = 0;
        for (; kt < kt_end; kt += 2) {                                 // a step beyond the slice multiplies zeros
            meet();
            unsigned next = after(slot);
            half_step(I0{}, I0{}, IL2{}, slot, next);
            advance();
            slot = next;
            meet();
            next = after(slot);
            half_step(I1{}, I0{}, IL2{}, slot, next);
            advance();
            slot = next;
        }
    } else {
        // Unrolled over the ring, so that every LDS position is a constant: a lone wavefront issues one instruction in four to five
        // cycles, and carrying the stage and rebuilding descriptors cost 15 to 20 of them per step.  1568 x 512 x 4608 on 64 x 64 x 64
        // tiles 18.5 -> 15.8 us (256 CUs), 6272 x 512 x 4608 on 128 x 128 x 64 32.9 -> 30.3, 1536 x 1024 x 4096 on 96 CUs 28.4 -> 27.7; the
        // prologue (divisions by multiplier, arguments in registers, window masks without loops, bias fetched first) is the
        // other part: 1536 x 1024 x 1024 on 64 x 128 x 64 8.4 -> 7.6, 25088 x 64 x 256 5.3 -> 4.6.
        constexpr int TURNS = KS == 2 || ST % 2 == 0 ? ST : 2 * ST;    // steps until stage and register set repeat
        bool more = true;
        do {
            static_for<TURNS>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                using Prev = std::integral_constant<unsigned, (u + ST - 1) % ST * STAGE>;    // stage of step kt - 1 (= kt + ST - 1)
                using Slot = std::integral_constant<unsigned, u % ST * STAGE>;
                using Next = std::integral_constant<unsigned, (u + 1) % ST * STAGE>;
                if (more) {
                    if constexpr (KS == 2) {
                        half_step(I0{}, IL2{}, IL1{}, Prev{}, Slot{});
                        advance();
                        meet();
                        half_step(I1{}, I0{}, IL2{}, Slot{}, Next{});
                    } else {
                        meet();
                        half_step(std::integral_constant<int, u % 2>{}, I0{}, IL2{}, Slot{}, Next{});
                        advance();
                    }
                    more = ++kt < kt_end;
                }
            });
        } while (more);
    }
    asm volatile("s_nop 15");                                          // the compiler does not see the latency of mma_agpr
    wait_and_meet<0>();
    if constexpr (FORM == DMA_POOL) {
        dma_epilogue<T, BM, BN, WM, WN, TM, TN, ACT_RELU, false, EARLY, DMA_POOL>(p, acc, bq, m_base, n_base, wm, wn);
        return;
    }
    if constexpr (FORM == DMA_F32) {
#define EPI(A) p.res ? dma_epilogue<T, BM, BN, WM, WN, TM, TN, A, true, EARLY, DMA_F32>(p, acc, bq, m_base, n_base, wm, wn) \
                     : dma_epilogue<T, BM, BN, WM, WN, TM, TN, A, false, EARLY, DMA_F32>(p, acc, bq, m_base, n_base, wm, wn)
        ECLIP_ACT_SWITCH(p.act, EPI)
#undef EPI
        return;
    }
    if (p.splits == 1 && p.y && (p.N & 7) == 0) {
#define EPI(A) p.res ? dma_epilogue<T, BM, BN, WM, WN, TM, TN, A, true, EARLY, DMA_PLAIN>(p, acc, bq, m_base, n_base, wm, wn) \
                     : dma_epilogue<T, BM, BN, WM, WN, TM, TN, A, false, EARLY, DMA_PLAIN>(p, acc, bq, m_base, n_base, wm, wn)
        ECLIP_ACT_SWITCH(p.act, EPI)
#undef EPI
        return;
    }
    if constexpr (dma_acc_in_agprs(BM, BN, NW)) {
        static_assert(4 * (TM * 8) * (TN * 16 + 4) * 4 <= dma_lds_bytes(BM, BN, BK, ST), "half the sub-tiles fit");
        dma_epilogue_rest<T, BM, BN, WM, WN, TM, TN>(p, acc, smem, m_base, n_base, wm, wn, blockIdx.y);
    } else tile_epilogue<T, BM, BN, WM, WN, TM, TN>(p, acc, smem, m_base, n_base, blockIdx.y);
}

}  // namespace eclip
