// Planning of the dense contractions: which kernel, which tile, how many K slices; the kernels that
// add the slices and the bias gradient; and the fp32 band kernel for backward-weight.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include "cg_internal.h"
#include "igemm_device.h"

namespace cg {


namespace {

// Blocks a split-K launch aims at, from below: two blocks are resident per compute unit, so up to
// 512 blocks start together and finish together.  A few blocks more than a whole number of such
// rounds run an extra round on a nearly empty GPU (1040 blocks took 19 % longer than 1000 on the
// backward-weight shapes of the benchmark), and one round measured faster than two or three.
#ifndef CG_SPLIT_BLOCKS
#define CG_SPLIT_BLOCKS 512
#endif
constexpr uint64_t kSplitBlocks = CG_SPLIT_BLOCKS;
// Blocks of the matrix kernels the GPU keeps resident at once: two per compute unit of the current
// device (512 on the 256 units of an MI355X), unless a test has set a lower count.
static std::atomic<uint32_t> g_resident_override{0};
uint32_t resident_blocks()
{
    const uint32_t o = g_resident_override.load(std::memory_order_relaxed);
    if (o) return o;
    static std::atomic<uint32_t> cached{0};
    uint32_t c = cached.load(std::memory_order_relaxed);
    if (!c) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
            c = 2u * (uint32_t)cus;
        else
            c = 512;
        cached.store(c, std::memory_order_relaxed);
    }
    return c;
}

constexpr int KT = 16;                       // reduction indices per LDS stage (a ring of NST stages)
constexpr int NPART = KT / 2;                // MFMA steps per tile = parts the loads of a tile are issued in
// 64 lanes x 4 bytes, global memory -> LDS: lane l's element lands at lds + 4*l.  `lds` and `soff`
// are wave-uniform.  Written as assembly so that the waits stay under this file's control: the
// kernel below waits for exactly the tile it is about to read (s_waitcnt vmcnt(n)), whereas the
// compiler, told that a load writes LDS, drains every load in flight before each LDS read.
// The hazard recognizer does not look inside assembly: a scalar register written by a preceding
// vector instruction (a readfirstlane, or a v_readlane that restores a spilled register, the buffer
// descriptor included) may not be read by a vector-memory instruction for five wait states (one for
// M0), so the s_mov and the s_nop 3 supply them.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(BufferRsrc rsrc, const float *lds, uint32_t voff, uint32_t soff)
{
    const uint32_t lds_addr = (uint32_t)(size_t)(const lds_float *)lds;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(soff))
                 : "memory", "m0");
}
// 64 lanes x 16 bytes: lane l's four elements land at lds + 16*l.
__device__ __forceinline__ void load4_to_lds(BufferRsrc rsrc, const float *lds, uint32_t voff)
{
    const uint32_t lds_addr = (uint32_t)(size_t)(const lds_float *)lds;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 ::"s"(lds_addr), "v"(voff), "s"(rsrc) : "memory", "m0");
}
#pragma clang diagnostic pop

// ---- tile loader of the band kernel -------------------------------------------------------------
// KLoader4: for an operand in which every aligned group of four reduction indices is four
// consecutive floats in memory (a row-major matrix; or runs of pixels, one run per image, the run
// length padded to a multiple of four in the index space).  One load moves 16 rows x 16 k: lane l
// fetches quad (l&3) ^ ((row>>2)&3) of row l>>2, so that the four quads of a row sit in its 64-byte
// LDS line in an order that spreads a fragment read of 16 rows over all banks.  Addresses need
// only 4-byte alignment, and the range check is per float: a quad that reaches beyond K, a run or
// the tensor delivers the floats that exist and zeros (or the neighbouring row's values) for the
// rest, which meet zeros of operand B.
template <int R> struct KLoader4 {
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
            load4_to_lds(rsrc, stage + (wave * NJ + j) * 256, roff[j] + koff);
    }
    __device__ __forceinline__ static void frag(const float *stage, int row, int ks, int h, float out[4])
    {
        const int unit = row * 4 + ((2 * ks + h) ^ ((row >> 2) & 3));
        const float4 q = *reinterpret_cast<const float4 *>(stage + unit * 4);
        out[0] = q.x; out[1] = q.y; out[2] = q.z; out[3] = q.w;
    }
};

}  // namespace

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
// waits as in the patch kernel above: A ring of NSTA stages, the patch double buffered, the next
// unit's patch loads issued during the current unit's first K-tile (a unit has >= 5 K-tiles).

template <int WM, int WN, int TM, int TN, int NSTA, int CPB, int NSL>
__global__ __launch_bounds__(256, 2) void igemm_wgrad_kernel(const IgemmProblem p)
{
    static_assert(WM * WN == 4 && WN * TN == 4, "four waves, 128 columns per block");
    static_assert(CPB % 4 == 0, "whole channels per wave");
    constexpr int MT = WM * TM * 32, NT = 128;
    using LA = KLoader4<MT>;
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
            load4_to_lds(rsrcA, smem + (tile % NSTA) * LA::SZ + (wave * LA::NJ + j) * 256, la.roff[j] + la.koff);
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
    store_tile<TM, TN>(p, acc, g, sp, m0 + (uint32_t)(wm * TM * 32), n0 + (uint32_t)(wn * TN * 32), p.N, lane,
                       smem + wave * EpiLds<TN>::FLOATS);
}


namespace {

// every aligned group of four reduction indices is four consecutive floats: k is unit-stride, either
// throughout or inside runs whose padded length is a multiple of four
bool quad_ok(const Operand &o, uint32_t)
{
    if (!o.lanes_k || o.check) return false;
    const bool linear = o.k.d1.d == 1 && o.k.d2.d == 1 && o.k.s1 == 1;
    const bool runs = o.k.d1.d % 4 == 0 && o.k.d2.d == 1 && o.k.s2 == 1;
    return linear || runs;
}

// Row-tile height for a problem.  A taller tile gathers the B operand (the costly one: one load
// instruction per 64 elements) fewer times, but leaves fewer blocks to spread over the 256 compute
// units, two resident per unit.  The cost model is the number of blocks the busiest unit runs (an
// odd one out runs alone and a little slower than a pair) times a block's duration, rows + a fixed
// per-block part; problems with few tiles are cut along K afterwards, which fills the chip for any
// tile height, so there only the per-block efficiency counts.
int pick_mt(uint32_t M, uint32_t N, uint32_t groups, uint32_t K = 0)
{
    const int cand[6] = {256, 192, 128, 96, 64, 32};
    int best = 32;
    double best_cost = 1e300;
    for (int c : cand) {
        const uint64_t tiles = (uint64_t)((M + c - 1) / c) * ((N + 127) / 128) * groups;
        double cost;
        if (tiles < 512 && K && K / 128 < kSplitBlocks / tiles) {
            // a short reduction cannot be cut into enough slices to fill the chip: the blocks all run
            // at once (or two to a unit), and what counts is how long one of them takes, in the same
            // unit as below (block duration per K-tile of the whole reduction, blocks per unit)
            const uint64_t splits = K / 128 >= 2 ? K / 128 : 1;
            const uint64_t kt = (K + KT - 1) / KT, kt_per = (kt + splits - 1) / splits;
            cost = (double)((tiles * splits + 255) / 256) * (c + 50) * (double)kt_per / (double)kt;
        } else if (tiles < 512) {
            cost = (double)tiles * (c + 50) / 256.0;                  // cut along K afterwards into one round of resident blocks
        } else {
            const uint64_t n = (tiles + 255) / 256;
            cost = ((n & 1) ? (double)(n - 1) + 1.2 : (double)n) * (c + 50);
        }
        if (cost < best_cost * 0.999) { best_cost = cost; best = c; }   // ties keep the larger tile
    }
    return best;
}

// Row-tile height of split_gemm_kernel: the same model for its tiles.  What a step costs whatever its
// height (fetching, cutting and storing 128 columns, the barrier) is worth 154 rows: 11x11 windows over
// 227x227, one column of blocks of 128 / 64 / 32 / 16 rows took 508 / 393 / 357 / 314 us.
int gemm_mt(uint32_t M, uint32_t N, uint32_t groups, uint32_t K)
{
    const int cand[4] = {128, 64, 32, 16};
    int best = 16;
    double best_cost = 1e300;
    for (int c : cand) {
        const uint64_t tiles = (uint64_t)((M + c - 1) / c) * ((N + 127) / 128) * groups;
        const double t = c + 154;
        double cost;
        if (tiles < kSplitBlocks && K / 128 < kSplitBlocks / tiles) {
            const uint64_t splits = K / 128 >= 2 ? K / 128 : 1;
            const uint64_t st = (K + 31) / 32, st_per = (st + splits - 1) / splits;
            cost = (double)((tiles * splits + 255) / 256) * t * (double)st_per / (double)st;
        } else if (tiles < kSplitBlocks) {
            cost = (double)tiles * t / 256.0;
        } else {
            const uint64_t n = (tiles + 255) / 256;
            cost = ((n & 1) ? (double)(n - 1) + 1.2 : (double)n) * t;
        }
        if (cost < best_cost * 0.999) { best_cost = cost; best = c; }
    }
    return best;
}

// lower bound of a map's offsets over its index range
int64_t map_min_off(const IndexMap &m)
{
    if (m.count == 0) return m.o0;
    const int64_t q1max = (m.count - 1) / m.d1.d;
    const int64_t q2max = (int64_t)((m.count - 1 < m.d1.d - 1 ? m.count - 1 : m.d1.d - 1)) / m.d2.d;
    const int64_t r2max = (int64_t)m.d2.d - 1;
    int64_t lo = m.o0;
    if (m.s1 < 0) lo += q1max * m.s1;
    if (m.s2 < 0) lo += q2max * m.s2;
    if (m.s3 < 0) lo += r2max * m.s3;
    return lo;
}
int64_t map_max_off(const IndexMap &m)
{
    if (m.count == 0) return m.o0;
    const int64_t q1max = (m.count - 1) / m.d1.d;
    const int64_t q2max = (int64_t)((m.count - 1 < m.d1.d - 1 ? m.count - 1 : m.d1.d - 1)) / m.d2.d;
    const int64_t r2max = (int64_t)m.d2.d - 1;
    int64_t hi = m.o0;
    if (m.s1 > 0) hi += q1max * m.s1;
    if (m.s2 > 0) hi += q2max * m.s2;
    if (m.s3 > 0) hi += r2max * m.s3;
    return hi;
}

// Moves the most negative part of both maps' offsets into the base pointer and checks that the
// buffer descriptor of every group, and every offset the kernel can form, fit 31 bits of bytes.
int normalise_operand(Operand &o, uint32_t groups)
{
    if (!o.ptr || !aligned16(o.ptr) || o.row.count == 0 || o.k.count == 0 || o.elems == 0) return CG_EINVAL;
    const int64_t lo_r = map_min_off(o.row), lo_k = map_min_off(o.k);
    o.row.o0 -= (int32_t)lo_r;
    o.k.o0 -= (int32_t)lo_k;
    o.shift = lo_r + lo_k;
    const int64_t span = (int64_t)o.elems - o.shift;          // floats behind the shifted base of group 0
    if (span <= 0 || (uint64_t)span * 4 > kMaxBufferBytes) return CG_EUNSUPPORTED;
    if ((uint64_t)(map_max_off(o.row) + 1) * 4 > kMaxBufferBytes || (uint64_t)(map_max_off(o.k) + 1) * 4 > kMaxBufferBytes)
        return CG_EUNSUPPORTED;
    if ((int64_t)(groups - 1) * o.gstride + o.shift >= (int64_t)o.elems) return CG_EINVAL;
    return CG_OK;
}

}  // namespace

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

}  // namespace

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

void patch_set_resident_blocks(uint32_t b) { g_resident_override.store(b, std::memory_order_relaxed); }
uint32_t igemm_resident_blocks() { return resident_blocks(); }
int igemm_pick_mt(uint32_t M, uint32_t N, uint32_t groups) { return pick_mt(M, N, groups); }

FastDiv make_fastdiv(uint32_t d)
{
    // mul = ceil(2^(31+L) / d) with L = ceil(log2 d): exact quotients for all n < 2^31.
    FastDiv f;
    f.d = d ? d : 1;
    uint32_t L = 0;
    while ((1ull << L) < f.d) ++L;
    f.sh = 31 + L;
    f.mul = (uint32_t)(((1ull << f.sh) + f.d - 1) / f.d);
    return f;
}

IndexMap linear_map(uint32_t count, int32_t stride)
{
    IndexMap m{};
    m.count = count;
    m.d1 = make_fastdiv(1);
    m.d2 = make_fastdiv(1);
    m.s1 = stride;
    return m;
}

IndexMap split_map(uint32_t count, uint32_t d, int32_t sq, int32_t sr)
{
    IndexMap m{};
    m.count = count;
    m.d1 = make_fastdiv(d);
    m.d2 = make_fastdiv(1);
    m.s1 = sq;
    m.s2 = sr;
    return m;
}

void igemm_host_element(const Operand &op, uint32_t row, uint32_t k, int64_t *off, int *valid)
{
    const Info r = map_info(op.row, row), q = map_info(op.k, k);
    *valid = (uint32_t)(r.a + q.a) < op.limA && (uint32_t)(r.b + q.b) < op.limB &&
             (op.k.r1_lim == 0 || q.r1 < op.k.r1_lim);
    *off = (int64_t)r.off + q.off + op.shift;
}


int igemm_launch(const IgemmProblem &p0, hipStream_t stream)
{
    if (p0.use_patch) return split_patch_launch(p0, stream);
    if (p0.use_band) return split_wgrad_launch(p0, stream);
    if (p0.math != CG_MATH_FP32 && p0.math != CG_MATH_BF16 && p0.math != CG_MATH_BF16X3) return CG_EINVAL;
    IgemmProblem p = p0;
    if (!p.c_ptr || !aligned16(p.c_ptr)) return CG_EINVAL;
    if (p.M == 0 || p.N == 0 || p.K == 0 || p.groups == 0 || p.splits == 0) return CG_EINVAL;
    if (p.M >= (1u << 30) || p.N >= (1u << 30) || p.K >= (1u << 30)) return CG_EUNSUPPORTED;
    if (p.bias_mode && !p.bias) return CG_EINVAL;
    if (p.use_wgrad) {         // K slices are whole units here, not k ranges
        if (p.math != CG_MATH_FP32) return CG_EUNSUPPORTED;      // the band kernel multiplies in fp32 only
        if (!p.wgrad.x || !aligned16(p.wgrad.x) || p.wgrad.cpb == 0 || p.A.check) return CG_EINVAL;
        p.A.shift = 0;
        const int rcw = normalise_operand(p.A, p.groups);
        if (rcw) return rcw;
        return wgrad_launch(p, stream);
    }
    if (p.splits > 1 && (p.k_per_split % KT != 0)) return CG_EINVAL;
    if ((uint64_t)p.k_per_split * p.splits < p.K || (uint64_t)p.k_per_split * (p.splits - 1) >= p.K) return CG_EINVAL;
    if (p.bias_mode && !p.bias) return CG_EINVAL;
    if (p.A.check) return CG_EUNSUPPORTED;
    p.A.shift = p.B.shift = 0;
    int rc = normalise_operand(p.A, p.groups);
    if (rc) return rc;
    if (p.A.row.count != p.M || p.B.row.count != p.N || p.A.k.count != p.K || p.B.k.count != p.K) return CG_EINVAL;
    rc = normalise_operand(p.B, p.groups);
    if (rc) return rc;
    if (!p.A.check) { p.A.limA = p.A.limB = 1; }
    if (!p.B.check) { p.B.limA = p.B.limB = 1; }

    const int mt = p.mt ? p.mt : gemm_mt(p.M, p.N, p.groups, p.K);
    // how an operand's elements are fetched: 0 rows along the lanes, 1 k along the lanes, 2 aligned quads of k
    const bool aq = quad_ok(p.A, p.K);
    int bm = quad_ok(p.B, p.K) ? 2 : p.B.lanes_k ? 1 : 0;
    // A quad that reaches beyond K, or into the padding of a run of reduction indices, delivers the
    // floats that follow in memory (the next row's first elements): harmless only if the other
    // operand delivers exact zeros there, which the loaders that check every element do and the quad
    // loader does not.  Quads on both sides need a reduction range without any such position.
    if (aq && bm == 2 && (p.K % 4 != 0 || p.A.k.r1_lim != 0 || p.B.k.r1_lim != 0)) bm = 1;
    if (!aq && p.A.lanes_k) return CG_EUNSUPPORTED;
    if (p.math == CG_MATH_BF16) return split_gemm_1(p, mt, aq, bm, stream);
    if (p.math == CG_MATH_BF16X3) return split_gemm_2(p, mt, aq, bm, stream);
    return split_gemm_3(p, mt, aq, bm, stream);
}

// ---- split-K: more blocks for problems whose C has few tiles ---------------------------------

namespace {

struct FinishArgs {
    const float *part;
    int64_t plane;            // floats between consecutive K slices: groups * M * N
    int splits;
    float *c_ptr;
    int32_t c_row_stride;
    IndexMap c_col;
    int c_scatter;
    IndexMap c_row;
    uint32_t c_limA, c_limB;
    int64_t c_gstride;
    const float *bias;
    int bias_mode;
    int32_t bias_gstride;
    uint32_t M, N;
    FastDiv divN, divMN;
    int accumulate, relu;
    const float *gate;
    uint32_t total;           // groups * M * N
    // a convolution's bias gradient riding in the same launch: blocks finish_blocks.. sum one channel each
    const float *r_dy;
    int rN, rM, rP;
    FastDiv r_divQP;
    float *r_db;
    uint32_t finish_blocks;
};

typedef float f4u_b __attribute__((ext_vector_type(4), aligned(4)));

// Sum of dy[n][m][0..P) over the images n_beg..n_end-1, by one block; thread 0 returns it.
// The (image, group of four pixels) pairs are spread over the threads, each moving 16 bytes
// (4-byte aligned: planes of an odd pixel count start anywhere) with four loads in flight.
__device__ __forceinline__ float bias_channel_sum(const float *__restrict__ dy, int M, int P, int m, int n_beg, int n_end,
                                                  FastDiv divQP)
{
    const uint32_t QP = divQP.d, total = (uint32_t)(n_end - n_beg) * QP;
    float s = 0.f;
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += 256 * 4) {
        f4u_b v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = i0 + u * 256;
            v[u] = f4u_b{0.f, 0.f, 0.f, 0.f};
            if (i < total) {
                const uint32_t n = fdiv(i, divQP), qd = i - n * QP;
                const float *src = dy + ((size_t)(n_beg + (int)n) * M + m) * P + 4 * qd;
                const int rem = P - 4 * (int)qd;
                if (rem >= 4) v[u] = __builtin_nontemporal_load(reinterpret_cast<const f4u_b *>(src));
                else {
                    v[u].x = src[0];
                    if (rem > 1) v[u].y = src[1];
                    if (rem > 2) v[u].z = src[2];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) s += (v[u].x + v[u].y) + (v[u].z + v[u].w);
    }
    __shared__ float red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

// C = (sum over the K slices) + bias, written through the problem's output map.  With few slices a
// thread adds them in slice order.  With many (ROWS = 8) a block owns 32 consecutive elements, its
// 8 thread rows add interleaved slices (row r: slices r, r+8, ...), and the 8 row sums are added
// in row order.  Either way the association is fixed by the number of slices alone, so the result
// does not depend on scheduling.
__device__ __forceinline__ void finish_store(const FinishArgs &a, uint32_t i, float s)
{
    const uint32_t g = fdiv(i, a.divMN), rem = i - g * a.divMN.d;
    const uint32_t m = fdiv(rem, a.divN), n = rem - m * a.divN.d;
    if (a.bias_mode == 1) s += a.bias[(int64_t)g * a.bias_gstride + m];
    else if (a.bias_mode == 2) s += a.bias[(int64_t)g * a.bias_gstride + n];
    if (a.relu) s = fmaxf(s, 0.f);
    const Info ci = map_info(a.c_col, n);
    int32_t in_group = (int32_t)m * a.c_row_stride + ci.off;
    if (a.c_scatter) {
        const Info ri = map_info(a.c_row, m);
        if (!((uint32_t)(ri.a + ci.a) < a.c_limA && (uint32_t)(ri.b + ci.b) < a.c_limB)) return;
        in_group = ri.off + ci.off;
    }
    const int64_t idx = (int64_t)g * a.c_gstride + in_group;
    if (a.gate && !(a.gate[idx] > 0.f)) s = 0.f;
    float *dst = a.c_ptr + idx;
    if (a.accumulate) s += *dst;
    *dst = s;
}

// AHEAD: a thread's next eight loads are in flight together (under a condition each, where fewer are left).  It pays
// where a thread has many; whole passes, us, plain / ahead: one thread per element, 2 slices 33.8 / 39.8, 3 slices
// 26.9 / 28.4, 7 slices 16.1 / 15.0, 13 slices 16.1 / 14.4; eight rows of threads, 32 slices 44.8 / 49.4, 49 slices 15.3 / 14.0,
// 64 slices 113.8 / 109.2, 512 slices 55.6 / 44.9.
template <int ROWS, bool AHEAD> __global__ __launch_bounds__(256) void splitk_finish_kernel(const FinishArgs a)
{
    if (a.r_dy && blockIdx.x >= a.finish_blocks) {       // a rider block: one channel of the bias gradient
        const int m = (int)(blockIdx.x - a.finish_blocks);
        const float s = bias_channel_sum(a.r_dy, a.rM, a.rP, m, 0, a.rN, a.r_divQP);
        if (threadIdx.x == 0) a.r_db[m] = s;
        return;
    }
    const uint32_t nblk = a.r_dy ? a.finish_blocks : gridDim.x;
    if (ROWS == 1) {
        for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < a.total; i += nblk * 256) {
            float s = a.part[i];
            if constexpr (!AHEAD)
                for (int k = 1; k < a.splits; ++k) s += a.part[(int64_t)k * a.plane + i];
            else for (int k0 = 1; k0 < a.splits; k0 += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = k0 + u < a.splits ? a.part[(int64_t)(k0 + u) * a.plane + i] : 0.f;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (k0 + u < a.splits) s += v[u];
            }
            finish_store(a, i, s);
        }
        return;
    }
    __shared__ float part[8][33];
    const int el = threadIdx.x & 31, r = threadIdx.x >> 5;
    for (uint32_t i0 = blockIdx.x * 32; i0 < a.total; i0 += nblk * 32) {
        const uint32_t i = i0 + el;
        float s = 0.f;
        if (i < a.total) {
            if constexpr (!AHEAD)
                for (int k = r; k < a.splits; k += 8) s += a.part[(int64_t)k * a.plane + i];
            else for (int k0 = r; k0 < a.splits; k0 += 64) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = k0 + 8 * u < a.splits ? a.part[(int64_t)(k0 + 8 * u) * a.plane + i] : 0.f;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (k0 + 8 * u < a.splits) s += v[u];
            }
        }
        part[r][el] = s;
        __syncthreads();
        if (r == 0 && i < a.total) {
            s = part[0][el];
#pragma unroll
            for (int k = 1; k < 8; ++k) s += part[k][el];
            finish_store(a, i, s);
        }
        __syncthreads();
    }
}

}  // namespace

// K slices for row tiles of mt rows: as many as make one round of resident blocks, at least 128
// reduction indices each.
static SplitPlan slices(uint32_t M, uint32_t N, uint32_t K, uint32_t groups, int mt)
{
    SplitPlan pl{1, K, 0, mt};
    const uint64_t tiles = (uint64_t)((M + mt - 1) / mt) * ((N + 127) / 128) * groups;
    if (tiles >= 512) return pl;
    uint64_t want = kSplitBlocks / tiles;
    const uint64_t max_by_k = K / 128;
    if (want > max_by_k) want = max_by_k;
    if (want > 512) want = 512;
    if (want < 2) return pl;
    if ((uint64_t)groups * M * N >= (1ull << 31)) return pl;
    uint64_t per = (K + want - 1) / want;
    per = (per + KT - 1) / KT * KT;
    pl.k_per_split = (uint32_t)per;
    pl.splits = (uint32_t)((K + per - 1) / per);
    if (pl.splits < 2) return SplitPlan{1, K, 0, mt};
    pl.ws_bytes = (size_t)pl.splits * groups * M * N * sizeof(float);
    return pl;
}

// A slice's sums are as long as its share of K, and their rounding error with them.  The tiles of up to
// 256 rows that pick_mt chooses from leave room for more slices than lower ones in one round; where a
// slice would get more than 4/3 as long, the blocks make two or more rounds instead (up to kOwnK terms the
// three-piece products round a sum 0.86 times as much as the fp32 instruction, so the error stays below its).
SplitPlan plan_split(uint32_t M, uint32_t N, uint32_t K, uint32_t groups)
{
    const int mt = gemm_mt(M, N, groups, K);
    SplitPlan pl = slices(M, N, K, groups, mt);
    const SplitPlan tall = slices(M, N, K, groups, pick_mt(M, N, groups, K));
    if (tall.splits < 2 || pl.splits * 4 >= tall.splits * 3) return pl;
    const uint64_t tiles = (uint64_t)((M + mt - 1) / mt) * ((N + 127) / 128) * groups;
    uint64_t want = 0;
    for (uint64_t rounds = 1; want * 4 < (uint64_t)tall.splits * 3; ++rounds) want = rounds * kSplitBlocks / tiles;
    if (want > tall.splits) want = tall.splits;
    const uint64_t per = ((K + want - 1) / want + KT - 1) / KT * KT;
    pl.k_per_split = (uint32_t)per;
    pl.splits = (uint32_t)((K + per - 1) / per);
    pl.ws_bytes = (size_t)pl.splits * groups * M * N * sizeof(float);
    return pl;
}

uint32_t tall_tile_splits(uint32_t M, uint32_t N, uint32_t K, uint32_t groups)
{
    return slices(M, N, K, groups, pick_mt(M, N, groups, K)).splits;
}

// What the caller is told to bring.  Never less than the tiles of up to 256 rows need that pick_mt
// chooses from: a size that a program has been told stays enough, and the entry point with a scratch
// array of a fixed size keeps refusing exactly the problems it refused.
size_t igemm_ws_bytes(const IgemmProblem &p)
{
    if (p.use_patch) return 0;
    if (p.use_wgrad) return p.splits > 1 ? (size_t)p.splits * p.groups * p.M * p.N * sizeof(float) : 0;
    const size_t a = p.use_band ? (p.splits > 1 ? (size_t)p.splits * p.groups * p.M * p.N * sizeof(float) : 0)
                                : plan_split(p.M, p.N, p.K, p.groups).ws_bytes;
    const size_t b = slices(p.M, p.N, p.K, p.groups, pick_mt(p.M, p.N, p.groups, p.K)).ws_bytes;
    return a > b ? a : b;
}

int igemm_run(const IgemmProblem &p0, void *ws, size_t ws_bytes, hipStream_t stream, const BiasRider *rider, bool *rider_taken)
{
    if (rider_taken) *rider_taken = false;
    const SplitPlan pl = p0.use_patch   ? SplitPlan{1, p0.K, 0, 0}
                         : p0.use_wgrad || p0.use_band ? SplitPlan{p0.splits, p0.K, (size_t)(p0.splits > 1 ? p0.splits : 0) * p0.groups * p0.M * p0.N * sizeof(float), 0}
                                        : plan_split(p0.M, p0.N, p0.K, p0.groups);
    if (pl.splits <= 1) {
        IgemmProblem p = p0;
        p.splits = 1; p.k_per_split = p.K; p.mt = pl.mt;
        return igemm_launch(p, stream);
    }
    if (!ws || ws_bytes < pl.ws_bytes) return CG_ENOSPC;
    if (!aligned16(ws) || !p0.c_ptr) return CG_EINVAL;
    if (p0.bias_mode && !p0.bias) return CG_EINVAL;
    IgemmProblem p = p0;
    p.c_ptr = static_cast<float *>(ws);
    p.c_row_stride = (int32_t)p0.N;
    p.c_col = linear_map(p0.N, 1);
    p.c_gstride = (int64_t)p0.M * p0.N;
    p.c_split_stride = (int64_t)p0.groups * p0.M * p0.N;
    p.c_scatter = 0;
    p.bias = nullptr; p.bias_mode = 0; p.accumulate = 0; p.relu = 0; p.gate = nullptr;
    p.splits = pl.splits; p.k_per_split = pl.k_per_split; p.mt = pl.mt;
    const int rc = igemm_launch(p, stream);
    if (rc) return rc;
    FinishArgs a{};
    a.part = static_cast<const float *>(ws);
    a.plane = p.c_split_stride;
    a.splits = (int)pl.splits;
    a.c_ptr = p0.c_ptr; a.c_row_stride = p0.c_row_stride; a.c_col = p0.c_col; a.c_gstride = p0.c_gstride;
    a.c_scatter = p0.c_scatter; a.c_row = p0.c_row; a.c_limA = p0.c_limA; a.c_limB = p0.c_limB;
    a.bias = p0.bias; a.bias_mode = p0.bias_mode; a.bias_gstride = p0.bias_gstride;
    a.M = p0.M; a.N = p0.N;
    a.divN = make_fastdiv(p0.N);
    a.divMN = make_fastdiv(p0.M * p0.N);
    a.accumulate = p0.accumulate; a.relu = p0.relu; a.gate = p0.gate;
    a.total = p0.groups * p0.M * p0.N;
    unsigned riders = 0;
    if (rider && rider->dy && rider->db && rider->M > 0 && rider->M <= 65536 &&
        (uint64_t)rider->N * (uint64_t)((rider->P + 3) / 4) < (1ull << 31)) {
        a.r_dy = rider->dy; a.rN = rider->N; a.rM = rider->M; a.rP = rider->P; a.r_db = rider->db;
        a.r_divQP = make_fastdiv((uint32_t)(rider->P + 3) / 4);
        riders = (unsigned)rider->M;
        if (rider_taken) *rider_taken = true;
    }
    if (pl.splits >= 16) {
        const unsigned blocks = (a.total + 31) / 32 < 65536 ? (a.total + 31) / 32 : 65536;
        a.finish_blocks = blocks;
        if (pl.splits >= 40) hipLaunchKernelGGL((splitk_finish_kernel<8, true>), dim3(blocks + riders), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((splitk_finish_kernel<8, false>), dim3(blocks + riders), dim3(256), 0, stream, a);
    } else {
        const unsigned blocks = (a.total + 255) / 256 < 16384 ? (a.total + 255) / 256 : 16384;
        a.finish_blocks = blocks;
        if (pl.splits >= 6) hipLaunchKernelGGL((splitk_finish_kernel<1, true>), dim3(blocks + riders), dim3(256), 0, stream, a);
        else hipLaunchKernelGGL((splitk_finish_kernel<1, false>), dim3(blocks + riders), dim3(256), 0, stream, a);
    }
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

// ---- bias gradient of a convolution: db[m] = sum over n and pixels of dy[n][m][pix] ------------

namespace {

// block (m, s) sums the samples of slice s; the slices are added afterwards in slice order.
// The (image, group of four pixels) pairs of the slice are spread over the threads, each moving
// 16 bytes (4-byte aligned: planes of an odd pixel count start anywhere) with four loads in flight.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

__global__ __launch_bounds__(256) void bias_grad_partial_kernel(const float *__restrict__ dy, int N, int M, int P,
                                                                int n_per, FastDiv divQP, float *__restrict__ part)
{
    const int m = blockIdx.x, sl = blockIdx.y;
    const int n_beg = sl * n_per, n_end = min(N, n_beg + n_per);
    const float s = bias_channel_sum(dy, M, P, m, n_beg, n_end, divQP);
    if (threadIdx.x == 0) part[(size_t)sl * M + m] = s;
}

__global__ __launch_bounds__(256) void bias_grad_finish_kernel(const float *__restrict__ part, int M, int S,
                                                               float *__restrict__ db)
{
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m >= M) return;
    float s = 0.f;
    for (int k = 0; k < S; ++k) s += part[(size_t)k * M + m];
    db[m] = s;
}

int bias_slices(int N, int M)
{
    int S = (2048 + M - 1) / M;
    if (S > N) S = N;
    return S < 1 ? 1 : S;
}

}  // namespace

size_t bias_grad_ws_bytes(int N, int M)
{
    return (size_t)bias_slices(N, M) * M * sizeof(float);
}

bool bias_grad_single_launch(int N, int P) { return (uint64_t)N * (uint64_t)P <= 32768; }

int bias_grad_launch(const float *dy, int N, int M, int P, float *db, void *ws, size_t ws_bytes,
                     hipStream_t stream)
{
    if (!dy || !db || N <= 0 || M <= 0 || P <= 0) return CG_EINVAL;
    if (!ws || ws_bytes < bias_grad_ws_bytes(N, M)) return CG_ENOSPC;
    // a small layer: one block per channel sums all images and writes db itself (one launch)
    const int S = bias_grad_single_launch(N, P) ? 1 : bias_slices(N, M);
    const int n_per = (N + S - 1) / S;
    const int S2 = (N + n_per - 1) / n_per;
    float *part = static_cast<float *>(ws);
    if ((uint64_t)n_per * (uint64_t)((P + 3) / 4) >= (1ull << 31)) return CG_EUNSUPPORTED;     // 32-bit pair index
    hipLaunchKernelGGL(bias_grad_partial_kernel, dim3(M, S2), dim3(256), 0, stream, dy, N, M, P, n_per,
                       make_fastdiv((uint32_t)(P + 3) / 4), S2 == 1 ? db : part);
    CG_HIP_TRY(hipGetLastError());
    if (S2 == 1) return CG_OK;
    hipLaunchKernelGGL(bias_grad_finish_kernel, dim3((M + 255) / 256), dim3(256), 0, stream, part, M, S2, db);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}


}  // namespace cg
