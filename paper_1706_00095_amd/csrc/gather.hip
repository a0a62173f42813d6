// Implicit-GEMM kernels that gather their operands into LDS.
//
// igemm_kernel computes C[m][n] = sum_k A(m,k) * B(n,k) for every dense contraction of
// the iteration: convolution forward, backward-data and backward-weight, and the three
// fully-connected passes.  Operand elements are addressed through index maps (cg_internal.h),
// so the im2col matrix is never materialised: a tile of it is gathered straight from the NCHW
// tensor into LDS, with zero padding folded into the load address.
//
// Work decomposition: a block of 4 waves owns an MT x 128 tile of C; each wave owns TM x TN
// sub-tiles of 32x32, accumulated by v_mfma_f32_32x32x2_f32.  The K loop advances KT = 16 at a
// time through a ring of NST LDS stages.  Operand tiles travel global memory -> LDS directly
// (buffer loads with the LDS modifier: no register round trip, no LDS store instructions), and an
// element that is zero padding, lies beyond the tile's rows or beyond K gets an offset outside the
// buffer descriptor's range, for which the hardware writes 0.  The loads of tile it+NST-1 are
// issued while tile it is multiplied; one s_barrier per K-tile.
//
// split_gemm.hip holds the other kernel for these problems; igemm.hip says which of the two a
// problem gets, and why.
#include <atomic>
#include <cstdio>
#include <type_traits>
#include <utility>
#include "cg_internal.h"
#include "igemm_device.h"

// This file is compiled three times.  CG_MATH = 0 (the default) multiplies in fp32 and also holds the
// band kernel.  CG_MATH = 1 and 2 build the gathered kernel and its launcher once more, for the bf16
// matrix instructions: the tiles travel
// and lie in LDS as fp32 exactly as before, a lane rounds its fragments to bf16 (nearest even)
// and one v_mfma_f32_32x32x16_bf16 per accumulator multiplies a whole K-tile of 16.
//   1 (CG_MATH_BF16):   a*b with a, b rounded to bf16, accumulated in fp32.
//   2 (CG_MATH_BF16X3): a = ah + al, b = bh + bl (ah = bf16(a), al = bf16(a - ah)), three products
//                       al*bh + ah*bl + ah*bh: what is dropped is al*bl, about 2^-16 of a product.
#ifndef CG_MATH
#define CG_MATH 0
#endif

namespace cg {

namespace {

constexpr int KT = 16;                       // reduction indices per LDS stage (a ring of NST stages)
constexpr int NPART = KT / 2;                // MFMA steps per tile = parts the loads of a tile are issued in


// The eight fp32 fragment values a lane holds of a K-tile (k = 8*ks + 4*h + t, ks = 0..1, t = 0..3)
// as the bf16 operand vector of v_mfma_f32_32x32x16_bf16, whose lane half h supplies k slots
// 8h..8h+7: slot 4*ks + t.  Which k sits in which slot is immaterial as long as A and B agree.
template <bool SPLIT>
__device__ __forceinline__ void to_bf16(const float (&f)[KT / 8][4], bf16x8 &hi, bf16x8 &lo)
{
#pragma unroll
    for (int ks = 0; ks < KT / 8; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float x = f[ks][t];
            const __bf16 xh = (__bf16)x;
            hi[4 * ks + t] = xh;
            if (SPLIT) lo[4 * ks + t] = (__bf16)(x - (float)xh);
        }
}

// 64 lanes x 4 bytes, global memory -> LDS: lane l's element lands at lds + 4*l.  `lds` and `soff`
// are wave-uniform.  Written as assembly so that the waits stay under this file's control: the
// kernel below waits for exactly the tile it is about to read (s_waitcnt vmcnt(n)), whereas the
// compiler, told that a load writes LDS, drains every load in flight before each LDS read.
// The hazard recognizer does not look inside assembly: a scalar register written by a preceding
// vector instruction (a readfirstlane, or a v_readlane that restores a spilled register, the buffer
// descriptor included) may not be read by a vector-memory instruction for five wait states (one for
// M0), so the s_mov and the s_nop 3 of this form supply them.  The short forms below (s_nop 0) are
// for kernels that spill no scalar register, which the build checks (build.py).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(BufferRsrc rsrc, const float *lds, uint32_t voff, uint32_t soff)
{
    const uint32_t lds_addr = (uint32_t)(size_t)(const lds_float *)lds;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(soff))
                 : "memory", "m0");
}
// The same without a scalar offset: no scalar register a vector instruction may just have written is
// read, and the one wait state M0 needs is enough.  A load with its set-up costs the matrix pipeline
// about 6 % of a four-MFMA step with four wait states and 4 % with one (measured on a loop of MFMAs).
__device__ __forceinline__ void load_to_lds(BufferRsrc rsrc, const float *lds, uint32_t voff)
{
    const uint32_t lds_addr = (uint32_t)(size_t)(const lds_float *)lds;
#if CG_MATH == 0
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 ::"s"(lds_addr), "v"(voff), "s"(rsrc) : "memory", "m0");
#else   // the bf16 instances of the gathered kernel spill scalar registers: the long form throughout
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 ::"s"(lds_addr), "v"(voff), "s"(rsrc) : "memory", "m0");
#endif
}
// 64 lanes x 16 bytes: lane l's four elements land at lds + 16*l.
constexpr int kShortWS = CG_MATH == 0 ? 1 : 4;
template <int WS = kShortWS>
__device__ __forceinline__ void load4_to_lds(BufferRsrc rsrc, const float *lds, uint32_t voff)
{
    const uint32_t lds_addr = (uint32_t)(size_t)(const lds_float *)lds;
    if constexpr (WS == 1)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     ::"s"(lds_addr), "v"(voff), "s"(rsrc) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     ::"s"(lds_addr), "v"(voff), "s"(rsrc) : "memory", "m0");
}
#pragma clang diagnostic pop

// ---- tile loaders -------------------------------------------------------------------------------
// A loader brings one R x KT operand tile into an LDS stage and says where the MFMA fragment of a
// lane lives there.  One load instruction moves 64 elements that land contiguously in LDS, so the
// lanes run along whichever index is contiguous in memory:
//   RowsLoader: lanes = 64 consecutive rows at one k.  Stage layout [k][RS], RS = 64*chunks + 8.
//               Row offsets (and window origins) live in registers for the whole K loop; the k part
//               is wave-uniform and travels in the scalar offset of the load.
//   KLoader:    lanes = 4 rows x 16 consecutive k.  Stage layout [row/4][68] with row%4 and k inside
//               the 64-float group.  The k part is computed per lane once per tile.
// In both, lane (i = lane&31, h = lane>>5) of a wave fetches for one 8-wide k step the four values
// k = 8*ks + 4h + t, t = 0..3 of row i; MFMA number t of the step consumes value t.  Which k a
// lane half holds is immaterial as long as A and B agree.  The paddings (8, 4) put the two lane
// halves, and neighbouring row groups, on different LDS banks.
// Wave w of the block issues the loads of k = 4w..4w+3 (RowsLoader) or of rows R/4*w.. (KLoader).

template <int R, bool CHECK> struct RowsLoader {
    static constexpr int NCH = (R + 63) / 64;
    static constexpr int RS = NCH * 64 + 8;
    static constexpr int SZ = KT * RS;
    static constexpr int LPT = 4 * NCH;          // load instructions per tile and wave
    uint32_t roff[NCH];
    int32_t ra[NCH], rb[NCH];

    __device__ __forceinline__ void init(const Operand &op, uint32_t row0, uint32_t nrows, int, int lane)
    {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const uint32_t rl = (uint32_t)(c * 64 + lane), row = row0 + rl;
            const Info q = map_info(op.row, row);
            roff[c] = (rl < (uint32_t)R && row < nrows) ? (uint32_t)q.off * 4u : OOB_ROW;
            ra[c] = q.a; rb[c] = q.b;
        }
    }
    // scalar info of the k this wave is loading (set by the part that issues chunk 0 of that k)
    Info kq;
    uint32_t ksoff;

    // The loads of one tile are cut into NPART parts so that the K loop can place one part behind
    // each MFMA step: part P issues loads [P*LPT/NPART, (P+1)*LPT/NPART), load i = (t, chunk).
    template <int P>
    __device__ __forceinline__ void issue_part(BufferRsrc rsrc, float *stage, const Operand &op, uint32_t k0,
                                               uint32_t kend, int wave, int)
    {
#pragma unroll
        for (int i = P * LPT / NPART; i < (P + 1) * LPT / NPART; ++i) {
            const int t = i / NCH, c = i % NCH;
            const uint32_t kl = (uint32_t)(4 * wave + t), k = k0 + kl;       // wave-uniform
            if (c == 0) {
                kq = map_info(op.k, k);
                ksoff = (k < kend && (op.k.r1_lim == 0 || kq.r1 < op.k.r1_lim)) ? (uint32_t)kq.off * 4u : OOB_K;
            }
            uint32_t voff = roff[c];
            if (CHECK) {
                const bool ok = (uint32_t)(ra[c] + kq.a) < op.limA && (uint32_t)(rb[c] + kq.b) < op.limB;
                voff = ok ? voff : OOB_ROW;
            }
            load_to_lds(rsrc, stage + kl * RS + c * 64, voff, ksoff);
        }
    }
    __device__ __forceinline__ static void frag(const float *stage, int row, int ks, int h, float out[4])
    {
#pragma unroll
        for (int t = 0; t < 4; ++t) out[t] = stage[(8 * ks + 4 * h + t) * RS + row];
    }
};

template <int R, bool CHECK> struct KLoader {
    static_assert(R % 16 == 0, "four waves, four rows per load");
    static constexpr int NI = R / 4;             // load instructions per tile
    static constexpr int NJ = NI / 4;            // ... and wave
    static constexpr int GS = 68;
    static constexpr int SZ = NI * GS;
    static constexpr int LPT = NJ;
    uint32_t roff[NJ];
    int32_t ra[NJ], rb[NJ];

    __device__ __forceinline__ void init(const Operand &op, uint32_t row0, uint32_t nrows, int wave, int lane)
    {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t row = row0 + (uint32_t)(4 * (wave * NJ + j) + (lane >> 4));
            const Info q = map_info(op.row, row);
            roff[j] = row < nrows ? (uint32_t)q.off * 4u : OOB_ROW;
            ra[j] = q.a; rb[j] = q.b;
        }
    }
    Info kq;              // this lane's k of the tile being loaded (set by part 0)
    uint32_t koff;

    template <int P>
    __device__ __forceinline__ void issue_part(BufferRsrc rsrc, float *stage, const Operand &op, uint32_t k0,
                                               uint32_t kend, int wave, int lane)
    {
        if (P == 0) {
            const uint32_t k = k0 + (uint32_t)(lane & 15);
            kq = map_info(op.k, k);
            koff = (k < kend && (op.k.r1_lim == 0 || kq.r1 < op.k.r1_lim)) ? (uint32_t)kq.off * 4u : OOB_K;
        }
#pragma unroll
        for (int j = P * LPT / NPART; j < (P + 1) * LPT / NPART; ++j) {
            uint32_t voff = roff[j] + koff;
            if (CHECK) {
                const bool ok = (uint32_t)(ra[j] + kq.a) < op.limA && (uint32_t)(rb[j] + kq.b) < op.limB;
                voff = ok ? voff : OOB_ROW;
            }
            load_to_lds(rsrc, stage + (wave * NJ + j) * GS, voff);
        }
    }
    __device__ __forceinline__ static void frag(const float *stage, int row, int ks, int h, float out[4])
    {
        const float4 q = *reinterpret_cast<const float4 *>(stage + (row >> 2) * GS + (row & 3) * 16 + 8 * ks + 4 * h);
        out[0] = q.x; out[1] = q.y; out[2] = q.z; out[3] = q.w;
    }
};

// KLoader4: for an operand in which every aligned group of four reduction indices is four
// consecutive floats in memory (a row-major matrix; or runs of pixels, one run per image, the run
// length padded to a multiple of four in the index space).  One load moves 16 rows x 16 k: lane l
// fetches quad (l&3) ^ ((row>>2)&3) of row l>>2, so that the four quads of a row sit in its 64-byte
// LDS line in an order that spreads a fragment read of 16 rows over all banks.  Addresses need
// only 4-byte alignment, and the range check is per float: a quad that reaches beyond K, a run or
// the tensor delivers the floats that exist and zeros (or the neighbouring row's values) for the
// rest, which meet zeros of operand B.
template <int R, int WS = kShortWS> struct KLoader4 {       // WS: wait states behind the M0 set-up of a load (1 or 4)
    static constexpr int NJ = (R + 63) / 64;     // load instructions per tile and wave
    static constexpr int SZ = 4 * NJ * 256;      // rows beyond R are loaded as zeros
    static constexpr int LPT = NJ;
    uint32_t roff[NJ];
    uint32_t kq4;                                // first k of this lane's quad inside the tile
    uint32_t koff;                               // byte offset of that quad (set by part 0 of a tile)

    __device__ __forceinline__ void init(const Operand &op, uint32_t row0, uint32_t nrows, int wave, int lane)
    {
        const uint32_t r = (uint32_t)lane >> 2;
        kq4 = 4u * (((uint32_t)lane & 3u) ^ ((r >> 2) & 3u));
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t rl = (uint32_t)(16 * (wave * NJ + j)) + r, row = row0 + rl;
            const Info q = map_info(op.row, row);
            roff[j] = (rl < (uint32_t)R && row < nrows) ? (uint32_t)q.off * 4u : OOB_ROW;
        }
    }
    template <int P>
    __device__ __forceinline__ void issue_part(BufferRsrc rsrc, float *stage, const Operand &op, uint32_t k0,
                                               uint32_t kend, int wave, int)
    {
        if (P == 0) {
            const uint32_t k = k0 + kq4;
            // a plain matrix (wave-uniform test) needs no index arithmetic: its k is its offset
            const uint32_t off = op.k.d1.d == 1 ? k + (uint32_t)op.k.o0 : (uint32_t)map_info(op.k, k).off;
            koff = k < kend ? off * 4u : OOB_K;
        }
#pragma unroll
        for (int j = P * LPT / NPART; j < (P + 1) * LPT / NPART; ++j)
            load4_to_lds<WS>(rsrc, stage + (wave * NJ + j) * 256, roff[j] + koff);
    }
    __device__ __forceinline__ static void frag(const float *stage, int row, int ks, int h, float out[4])
    {
        const int unit = row * 4 + ((2 * ks + h) ^ ((row >> 2) & 3));
        const float4 q = *reinterpret_cast<const float4 *>(stage + unit * 4);
        out[0] = q.x; out[1] = q.y; out[2] = q.z; out[3] = q.w;
    }
};

}  // namespace

template <int WM, int WN, int TM, int TN, int NST, class LA, class LB, int MATH>
__global__ __launch_bounds__(256, 2) void igemm_kernel(const IgemmProblem p)
{
    static_assert(WM * WN == 4, "four waves");
    constexpr int MT = WM * TM * 32, NT = WN * TN * 32;
    constexpr int STAGE = LA::SZ + LB::SZ;
    constexpr int LPT = LA::LPT + LB::LPT;
    static_assert((NST - 1) * LPT <= 63, "the vector-memory counter holds 63 loads");

    extern __shared__ __attribute__((aligned(16))) float smem[];     // [NST][LA::SZ + LB::SZ]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const uint32_t m0 = blockIdx.y * MT, n0 = blockIdx.x * NT;
    const uint32_t g = blockIdx.z / p.splits, sp = blockIdx.z % p.splits;
    const uint32_t kbeg = sp * p.k_per_split;
    const uint32_t kend = min(p.K, kbeg + p.k_per_split);
    const int n_iter = (int)((kend - kbeg + KT - 1) / KT);

    const BufferRsrc rsrcA = operand_rsrc(p.A, g), rsrcB = operand_rsrc(p.B, g);
    LA la;
    LB lb;
    la.init(p.A, m0, p.M, wave, lane);
    lb.init(p.B, n0, p.N, wave, lane);

    // Tiles past the end of the K range are all padding: they cost no memory traffic and keep the
    // count of outstanding loads the same in every iteration.
    auto issue_part = [&](auto PC, int tile) {
        constexpr int P = decltype(PC)::value;
        float *st = smem + (tile % NST) * STAGE;
        const uint32_t k0 = kbeg + (uint32_t)tile * KT;
        la.template issue_part<P>(rsrcA, st, p.A, k0, kend, wave, lane);
        lb.template issue_part<P>(rsrcB, st + LA::SZ, p.B, k0, kend, wave, lane);
    };

    const int wm = wave / WN, wn = wave % WN;
    const int h = lane >> 5, li = lane & 31;
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
    for (int d = 0; d < NST - 1; ++d) static_for<0, NPART>([&](auto PC) { issue_part(PC, d); });

    for (int it = 0; it < n_iter; ++it) {
        // This wave's loads of tile `it` have landed (all but the NST-2 newer tiles are complete);
        // behind the barrier that holds for every wave, and everyone is done reading tile it-1,
        // whose stage the loads issued below overwrite.
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NST - 2) * LPT) : "memory");
        const float *a_s = smem + (it % NST) * STAGE, *b_s = a_s + LA::SZ;
        if constexpr (MATH != 0) {
            // bf16 matrix instructions: all fragments of the tile, rounded (and split), one MFMA per
            // accumulator and product, then the next tile's loads
            float af[TM][KT / 8][4], bf[TN][KT / 8][4];
#pragma unroll
            for (int ks = 0; ks < KT / 8; ++ks) {
#pragma unroll
                for (int i = 0; i < TM; ++i) LA::frag(a_s, (wm * TM + i) * 32 + li, ks, h, af[i][ks]);
#pragma unroll
                for (int j = 0; j < TN; ++j) LB::frag(b_s, (wn * TN + j) * 32 + li, ks, h, bf[j][ks]);
            }
            bf16x8 ah[TM], al[TM], bh[TN], bl[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) to_bf16<MATH == 2>(af[i], ah[i], al[i]);
#pragma unroll
            for (int j = 0; j < TN; ++j) to_bf16<MATH == 2>(bf[j], bh[j], bl[j]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (MATH == 2) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
                    }
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
                }
            static_for<0, NPART>([&](auto PC) { issue_part(PC, it + NST - 1); });
            continue;
        }
        float af[KT / 8][TM][4], bf[KT / 8][TN][4];
        // the fragments of the tile's first eight k now, those of the second eight behind the first
        // MFMA step: half the reads are waited for at the start of a tile
#pragma unroll
        for (int i = 0; i < TM; ++i) LA::frag(a_s, (wm * TM + i) * 32 + li, 0, h, af[0][i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) LB::frag(b_s, (wn * TN + j) * 32 + li, 0, h, bf[0][j]);
        __builtin_amdgcn_sched_barrier(0);
        // One part of the next tile's loads behind each MFMA step: the address pipeline and the
        // matrix pipeline both stay fed, instead of taking turns.
        static_for<0, NPART>([&](auto PC) {
            constexpr int P = decltype(PC)::value, ks = P / 4, s4 = P % 4;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[ks][i][s4], bf[ks][j][s4], acc[i][j], 0, 0, 0);
            if constexpr (P == 0) {
#pragma unroll
                for (int ks2 = 1; ks2 < KT / 8; ++ks2) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) LA::frag(a_s, (wm * TM + i) * 32 + li, ks2, h, af[ks2][i]);
#pragma unroll
                    for (int j = 0; j < TN; ++j) LB::frag(b_s, (wn * TN + j) * 32 + li, ks2, h, bf[ks2][j]);
                }
            }
            issue_part(PC, it + NST - 1);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    // the padding tiles still in flight write into this block's LDS: let them finish before it is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();            // every wave has read its last fragments: the stages are free for the epilogue
    // (scattered rows: strided backward-data, whose columns are an image's cells under a window)
    store_tile<TM, TN, std::is_same_v<LB, RowsLoader<NT, true>>>(p, acc, g, sp, m0 + (uint32_t)(wm * TM * 32), n0 + (uint32_t)(wn * TN * 32), p.N, lane,
                       smem + wave * EpiLds<TN>::FLOATS);
}

#if CG_MATH == 0
// ---- band kernel: backward-weight with the input staged as raw padded rows ------------------------
//
//   dw[m][(c,kh,kw)] = sum over pixels (n,oh,ow) of dy[n][m][oh][ow] * x[n][c][oh*s-p+kh][ow*s-p+kw]
//
// The gathered kernel fetches x once per filter tap and column tile.  Here the reduction walks
// "units" = (image, band of output rows); for a unit a block keeps the zero-padded source rows of
// the CPB input channels its 128 columns (c,kh,kw) belong to in LDS (loaded once per unit), and
// the B fragment of column (c,kh,kw) at pixel (r,ow) of the band is
//   patch[c - c0][ (r*s + kh)*Wp + ow*s + kw ] = patch[colbase(lane) + sigma(pixel)],
// colbase fixed per lane for the whole kernel, sigma computed per K-tile for the eight pixels a
// lane half multiplies.  dy arrives in K-tiles of 16 consecutive pixels of the band (aligned quads;
// what a quad reads beyond the band's last pixel meets B values forced to zero).  Pipeline and
// waits: A ring of NSTA stages as in igemm_kernel, the patch double buffered, the next
// unit's patch loads issued during the current unit's first K-tile (a unit has >= 5 K-tiles).

template <int WM, int WN, int TM, int TN, int NSTA, int CPB, int NSL>
__global__ __launch_bounds__(256, 2) void igemm_wgrad_kernel(const IgemmProblem p)
{
    static_assert(WM * WN == 4 && WN * TN == 4, "four waves, 128 columns per block");
    static_assert(CPB % 4 == 0, "whole channels per wave");
    constexpr int MT = WM * TM * 32, NT = 128;
    using LA = KLoader4<MT, 4>;
    constexpr int LAW = LA::LPT;
    constexpr int CS = NSL * 64 + 1;            // odd: the channels of one tap fall on different banks
    constexpr int BUF = CPB * CS;
    constexpr int NB = CPB / 4 * NSL;           // patch load instructions per wave and unit
    static_assert((NSTA - 1) * LAW + NB <= 63, "the vector-memory counter holds 63 loads");

    extern __shared__ __attribute__((aligned(16))) float smem[];     // [NSTA][LA::SZ] then [2][BUF]
    float *const sB = smem + NSTA * LA::SZ;

    const WgradGeom &wg = p.wgrad;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t m0 = blockIdx.y * MT, n0 = blockIdx.x * NT;
    const uint32_t g = blockIdx.z / p.splits, sp = blockIdx.z % p.splits;
    const int KK = wg.KH * wg.KW, P = wg.OH * wg.OW, HW = wg.H * wg.W;
    const int u0 = (int)sp * wg.units_per_split, u1 = min(wg.units, u0 + wg.units_per_split);

    const BufferRsrc rsrcA = operand_rsrc(p.A, g);
    BufferRsrc rsrcX;
    {
        const int64_t first = (int64_t)g * wg.Cg * HW;
        const uint64_t base = (uint64_t)reinterpret_cast<uintptr_t>(wg.x) + (uint64_t)(first * 4);
        rsrcX.x = __builtin_amdgcn_readfirstlane((uint32_t)base);
        rsrcX.y = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
        rsrcX.z = __builtin_amdgcn_readfirstlane((uint32_t)(((int64_t)wg.x_elems - first) * 4));
        rsrcX.w = 0x00020000u;
    }
    LA la;
    la.init(p.A, m0, p.M, wave, lane);

    const int wm = wave / WN, wn = wave % WN;
    const int h = lane >> 5, li = lane & 31;
    const uint32_t c0 = fdiv(n0, wg.divKK);                  // first input channel of this block's columns
    int32_t colbase[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const uint32_t n = n0 + (uint32_t)((wn * TN + j) * 32 + li);
        int32_t cb = 0;
        if (n < p.N) {
            const uint32_t c = fdiv(n, wg.divKK), tap = n - c * (uint32_t)KK;
            const uint32_t kh = fdiv(tap, wg.divKW), kw = tap - kh * (uint32_t)wg.KW;
            cb = (int32_t)(c - c0) * CS + (int32_t)kh * wg.Wp + (int32_t)kw;
        }
        colbase[j] = cb;
    }

    // a unit's band: first output row, number of output rows, pixels, K-tiles
    auto band_of = [&](int u, int &img, int &oy0, int &rows) {
        img = u / wg.nb;
        const int jb = u - img * wg.nb;
        oy0 = jb * wg.Rb;
        rows = min(wg.Rb, wg.OH - oy0);
    };
    int n_iter = 0;
    for (int u = u0; u < u1; ++u) {
        int img, oy0, rows;
        band_of(u, img, oy0, rows);
        n_iter += (rows * wg.OW + KT - 1) / KT;
    }

    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // ---- patch loads of unit u (a burst, issued in NPART parts) -----------------------------------
    uint32_t pvoff[NSL];
    auto patch_offsets = [&](int u) {          // global byte offset of every slot this lane loads, or out of range
        int img, oy0, rows;
        band_of(u, img, oy0, rows);
        const int prow = (rows - 1) * wg.s + wg.KH, sy0 = oy0 * wg.s - wg.pad_h;
#pragma unroll
        for (int e = 0; e < NSL; ++e) {
            const uint32_t jslot = (uint32_t)(e * 64 + lane);
            const uint32_t r = fdiv(jslot, wg.divWp), cc = jslot - r * (uint32_t)wg.Wp;
            const int sy = sy0 + (int)r, sx = (int)cc - wg.pad_w;
            const bool ok = (int)r < prow && (uint32_t)sy < (uint32_t)wg.H && (uint32_t)sx < (uint32_t)wg.W;
            pvoff[e] = ok ? (uint32_t)(sy * wg.W + sx) * 4u : OOB_ROW;
        }
    };
    auto issue_patch_part = [&](auto PC, int u) {
        constexpr int Pn = decltype(PC)::value;
        if (Pn == 0) patch_offsets(u);
        const int img = u / wg.nb;
        float *buf = sB + (u & 1) * BUF;
#pragma unroll
        for (int q = Pn * NB / NPART; q < (Pn + 1) * NB / NPART; ++q) {
            const int cl = wave + 4 * (q / NSL), e = q % NSL;
            const uint32_t c = c0 + (uint32_t)cl;
            const uint32_t soff = c < (uint32_t)wg.Cg ? (uint32_t)((img * wg.C + (int)c) * HW) * 4u : OOB_K;
            load_to_lds(rsrcX, buf + cl * CS + e * 64, pvoff[e], soff);
        }
    };
    // ---- A loads of the K-tile t of unit u: 16 consecutive pixels of dy ---------------------------
    auto issue_a_part = [&](auto PC, int tile, int u, int t) {
        constexpr int Pn = decltype(PC)::value;
        if (Pn == 0) {
            int img, oy0, rows;
            band_of(u, img, oy0, rows);
            const uint32_t k = (uint32_t)(oy0 * wg.OW + t * KT) + la.kq4;            // pixel of this lane's quad in its image
            la.koff = tile < n_iter ? ((uint32_t)(img * wg.M) * (uint32_t)P + k) * 4u : OOB_K;
        }
#pragma unroll
        for (int j = Pn * LAW / NPART; j < (Pn + 1) * LAW / NPART; ++j)
            load4_to_lds<4>(rsrcA, smem + (tile % NSTA) * LA::SZ + (wave * LA::NJ + j) * 256, la.roff[j] + la.koff);
    };
    auto tiles_of = [&](int u) {
        int img, oy0, rows;
        band_of(u, img, oy0, rows);
        return (rows * wg.OW + KT - 1) / KT;
    };

    // prologue: the first unit's patch, then A tiles 0..NSTA-2
    static_for<0, NPART>([&](auto PC) { issue_patch_part(PC, u0); });
    int iu = u0, it_ = 0, itiles = tiles_of(u0);        // (unit, tile) of the next A tile to issue
    auto advance_issue = [&]() {
        if (++it_ == itiles) { it_ = 0; ++iu; itiles = iu < u1 ? tiles_of(iu) : 1 << 30; }
    };
#pragma unroll
    for (int d = 0; d < NSTA - 1; ++d) {
        static_for<0, NPART>([&](auto PC) { issue_a_part(PC, d, iu, it_); });
        advance_issue();
    }

    int cu = u0, ct = 0, ctiles = tiles_of(u0);         // (unit, tile) being multiplied
    for (int it = 0; it < n_iter; ++it) {
        const bool burst = cu + 1 < u1;                 // this unit issues the next one's patch in its tile 0
        if (burst && ct >= 1 && ct <= NSTA - 2)
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NSTA - 2) * LAW + NB) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NSTA - 2) * LAW) : "memory");
        const float *a_s = smem + (it % NSTA) * LA::SZ;
        const float *b_s = sB + (cu & 1) * BUF;
        int img, oy0, rows;
        band_of(cu, img, oy0, rows);
        const int npix = rows * wg.OW;
        float af[KT / 8][TM][4], bf[KT / 8][TN][4];
#pragma unroll
        for (int ks = 0; ks < KT / 8; ++ks) {
#pragma unroll
            for (int i = 0; i < TM; ++i) LA::frag(a_s, (wm * TM + i) * 32 + li, ks, h, af[ks][i]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int pix = ct * KT + 8 * ks + 4 * h + t;
                const uint32_t r = fdiv((uint32_t)pix, wg.divOW), ox = (uint32_t)pix - r * (uint32_t)wg.OW;
                const int sg = (int)(r * (uint32_t)wg.s) * wg.Wp + (int)(ox * (uint32_t)wg.s);
                const bool live = pix < npix;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const float vv = b_s[live ? colbase[j] + sg : 0];
                    bf[ks][j][t] = live ? vv : 0.f;
                }
            }
        }
        const bool do_patch = burst && ct == 0;
        static_for<0, NPART>([&](auto PC) {
            constexpr int Pn = decltype(PC)::value, ks = Pn / 4, s4 = Pn % 4;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[ks][i][s4], bf[ks][j][s4], acc[i][j], 0, 0, 0);
            issue_a_part(PC, it + NSTA - 1, iu, it_);
            if (do_patch) issue_patch_part(PC, cu + 1);
            __builtin_amdgcn_sched_barrier(0);
        });
        advance_issue();
        if (++ct == ctiles) { ct = 0; ++cu; ctiles = cu < u1 ? tiles_of(cu) : 1 << 30; }
    }
    // the padding tiles still in flight write into this block's LDS: let them finish before it is released
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();            // every wave has read its last fragments: the stages are free for the epilogue
    store_tile<TM, TN, false>(p, acc, g, sp, m0 + (uint32_t)(wm * TM * 32), n0 + (uint32_t)(wn * TN * 32), p.N, lane,
                       smem + wave * EpiLds<TN>::FLOATS);
}

#endif  // CG_MATH == 0

namespace {

template <int WM, int WN, int TM, int TN, int NST, class LA, class LB>
int launch_cfg(const IgemmProblem &p, const char *modes, hipStream_t stream)
{
    constexpr int MT = WM * TM * 32, NT = WN * TN * 32;
    dim3 grid((p.N + NT - 1) / NT, (p.M + MT - 1) / MT, p.groups * p.splits);
    if (grid.y > 65535u || grid.z > 65535u) return CG_EUNSUPPORTED;
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, CG_MATH == 0 ? "igemm_kernel<%dx%d,%s>" : CG_MATH == 1 ? "igemm_kernel<%dx%d,%s,bf16>" : "igemm_kernel<%dx%d,%s,bf16x3>", MT, NT, modes);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    constexpr size_t lds = (size_t)NST * (LA::SZ + LB::SZ) * sizeof(float);
    static_assert(lds >= 4 * EpiLds<TN>::FLOATS * sizeof(float), "the epilogue turns the tile around in the stages' LDS");
    static_assert(2 * lds <= 160 * 1024, "two blocks of this tile do not fit the LDS of a compute unit");
    static std::atomic<bool> attr_set{false};      // raising the dynamic-LDS limit: once per kernel (repeating it is harmless)
    if (!attr_set.load(std::memory_order_acquire)) {
        CG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&igemm_kernel<WM, WN, TM, TN, NST, LA, LB, CG_MATH>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((igemm_kernel<WM, WN, TM, TN, NST, LA, LB, CG_MATH>), grid, dim3(256), lds, stream, p);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

// How an operand's tile is fetched: rows along the lanes, k along the lanes, or aligned quads of k.
enum { LD_ROWS = 0, LD_K = 1, LD_K4 = 2 };
template <int MODE, int R, bool CHECK>
using LoaderOf = std::conditional_t<MODE == LD_K4, KLoader4<R>,
                                    std::conditional_t<MODE == LD_K, KLoader<R, CHECK>, RowsLoader<R, CHECK>>>;

template <int AM, int BM, bool BC>
int launch_modes(const IgemmProblem &p, int mt, hipStream_t stream)
{
    static const char modes[4] = {"rk4"[AM], "rk4"[BM], BC ? 'c' : '-', 0};
    switch (mt) {
    case 256: return launch_cfg<2, 2, 4, 2, 3, LoaderOf<AM, 256, false>, LoaderOf<BM, 128, BC>>(p, modes, stream);
    case 192: return launch_cfg<2, 2, 3, 2, 3, LoaderOf<AM, 192, false>, LoaderOf<BM, 128, BC>>(p, modes, stream);
    case 128: return launch_cfg<2, 2, 2, 2, 4, LoaderOf<AM, 128, false>, LoaderOf<BM, 128, BC>>(p, modes, stream);
    case 96: return launch_cfg<1, 4, 3, 1, 4, LoaderOf<AM, 96, false>, LoaderOf<BM, 128, BC>>(p, modes, stream);
    case 64: return launch_cfg<1, 4, 2, 1, 4, LoaderOf<AM, 64, false>, LoaderOf<BM, 128, BC>>(p, modes, stream);
    default: return launch_cfg<1, 4, 1, 1, 4, LoaderOf<AM, 32, false>, LoaderOf<BM, 128, BC>>(p, modes, stream);
    }
}

}  // namespace

// am, bm: how an operand's tile is fetched, 0 rows along the lanes, 1 k along the lanes, 2 aligned quads of k
#define CG_CAT_(a, b) a##b
#define CG_CAT(a, b) CG_CAT_(a, b)
int CG_CAT(gather_launch_, CG_MATH)(const IgemmProblem &p, int mt, int am, int bm, hipStream_t stream)
{
    const bool bc = p.B.check != 0;
    if (am == LD_K4 && bm == LD_ROWS) return bc ? launch_modes<LD_K4, LD_ROWS, true>(p, mt, stream) : launch_modes<LD_K4, LD_ROWS, false>(p, mt, stream);
    if (am == LD_K4 && bm == LD_K4) return launch_modes<LD_K4, LD_K4, false>(p, mt, stream);
    if (am == LD_K4 && bm == LD_K) return bc ? launch_modes<LD_K4, LD_K, true>(p, mt, stream) : launch_modes<LD_K4, LD_K, false>(p, mt, stream);
    if (am == LD_K && bm == LD_ROWS) return bc ? launch_modes<LD_K, LD_ROWS, true>(p, mt, stream) : launch_modes<LD_K, LD_ROWS, false>(p, mt, stream);
    if (am == LD_K && (bm == LD_K || bm == LD_K4)) return bc ? launch_modes<LD_K, LD_K, true>(p, mt, stream) : launch_modes<LD_K, LD_K, false>(p, mt, stream);
    if (am == LD_ROWS && bm == LD_ROWS && !bc) return launch_modes<LD_ROWS, LD_ROWS, false>(p, mt, stream);
    return CG_EUNSUPPORTED;
}

#if CG_MATH == 0
namespace {

template <int TM, int NSTA, int CPB, int NSL>
int launch_wgrad_cfg(const IgemmProblem &p, hipStream_t stream)
{
    constexpr int MT = 2 * TM * 32;
    using LA = KLoader4<MT>;
    dim3 grid((p.N + 127) / 128, (p.M + MT - 1) / MT, p.groups * p.splits);
    if (grid.y > 65535u || grid.z > 65535u) return CG_EUNSUPPORTED;
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, "igemm_wgrad_kernel<%dx128,%d,%d>", MT, CPB, NSL);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    constexpr size_t lds = ((size_t)NSTA * LA::SZ + 2 * CPB * (NSL * 64 + 1)) * sizeof(float);
    static_assert(lds >= 4 * EpiLds<2>::FLOATS * sizeof(float), "the epilogue turns the tile around in the stages' LDS");
    static_assert(2 * lds <= 160 * 1024, "two blocks of this tile do not fit the LDS of a compute unit");
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        CG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&igemm_wgrad_kernel<2, 2, TM, 2, NSTA, CPB, NSL>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((igemm_wgrad_kernel<2, 2, TM, 2, NSTA, CPB, NSL>), grid, dim3(256), lds, stream, p);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

int wgrad_mt(uint32_t M) { return M > 128 && (M + 191) / 192 * 192 <= (M + 127) / 128 * 128 ? 192 : M > 64 ? 128 : 64; }

}  // namespace

int wgrad_launch(const IgemmProblem &p, hipStream_t stream)
{
    const int mt = wgrad_mt(p.M);
    if (p.wgrad.cpb == 16) {
        if (mt == 192) return launch_wgrad_cfg<3, 3, 16, 4>(p, stream);
        if (mt == 128) return launch_wgrad_cfg<2, 4, 16, 4>(p, stream);
        return launch_wgrad_cfg<1, 4, 16, 4>(p, stream);
    }
    if (mt == 192) return launch_wgrad_cfg<3, 3, 8, 8>(p, stream);
    if (mt == 128) return launch_wgrad_cfg<2, 4, 8, 8>(p, stream);
    return launch_wgrad_cfg<1, 4, 8, 8>(p, stream);
}

static std::atomic<uint32_t> g_wgrad_enabled{0};
void wgrad_set_enabled(int on) { g_wgrad_enabled.store(on ? 1 : 0, std::memory_order_relaxed); }

bool wgrad_plan(WgradGeom &g, uint32_t M, uint32_t N, uint32_t groups, uint32_t images, uint32_t *splits)
{
    g.cpb = g.nsl = 0;
    const int KK = g.KH * g.KW;
    if (!g_wgrad_enabled.load(std::memory_order_relaxed) || KK < 9 || g.s <= 0 || g.Cg <= 0 || images == 0) return false;
    if (g.x_elems * 4 > kMaxBufferBytes || (uint64_t)images * g.M * g.OH * g.OW * 4 > kMaxBufferBytes) return false;
    g.Wp = (g.OW - 1) * g.s + g.KW;
    // channels a block of 128 columns can touch: at most 127/KK + 2
    const int chans = 127 / KK + 2;
    const int cpb = chans > 8 ? 16 : 8, nsl = cpb == 16 ? 4 : 8;
    if (chans > 16) return false;
    const int max_prow = nsl * 64 / g.Wp;                   // padded source rows that fit the staging
    const int max_rows = (max_prow - g.KH) / g.s + 1;       // output rows per band
    if (max_prow < g.KH || max_rows < 1) return false;
    g.nb = (g.OH + max_rows - 1) / max_rows;
    g.Rb = (g.OH + g.nb - 1) / g.nb;
    // every unit needs at least five K-tiles of 16 pixels (the patch of the next unit lands during four)
    const int last_rows = g.OH - (g.nb - 1) * g.Rb;
    if (last_rows < 1 || last_rows * g.OW < 5 * KT) return false;
    if ((uint64_t)images * g.nb >= (1u << 30)) return false;
    g.units = (int32_t)(images * (uint32_t)g.nb);
    g.divOW = make_fastdiv((uint32_t)g.OW);
    g.divWp = make_fastdiv((uint32_t)g.Wp);
    g.divKK = make_fastdiv((uint32_t)KK);
    g.divKW = make_fastdiv((uint32_t)g.KW);
    // K slices: at most kSplitBlocks blocks, whole units per slice
    const int mt = wgrad_mt(M);
    const uint64_t tiles = (uint64_t)((M + mt - 1) / mt) * ((N + 127) / 128) * groups;
    uint64_t want = kSplitBlocks / tiles;
    if (want > (uint64_t)g.units) want = (uint64_t)g.units;
    if (want < 1) want = 1;
    if (want > 4096) want = 4096;
    g.units_per_split = (int32_t)(((uint64_t)g.units + want - 1) / want);
    *splits = (uint32_t)(((uint64_t)g.units + g.units_per_split - 1) / g.units_per_split);
    if ((uint64_t)*splits * groups * M * N >= (1ull << 31)) return false;
    g.cpb = cpb; g.nsl = nsl;
    return true;
}

#endif

}  // namespace cg
