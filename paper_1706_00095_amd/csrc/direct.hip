// Small contractions in one launch: C[m][n] = sum_k A(m,k) * B(n,k) by v_mfma_f32_16x16x4_f32.
//
// What bounds a small problem: launches that wait for one another (a copy of the filters, the matrix kernel, the kernel
// that adds its K slices: 4 to 5 us each) and the latency of a chain of loads on few compute units.  So a block is a
// 16 x 32 tile, small enough for many blocks, and its 4 to 16 waves share out the reduction: every wave walks its own
// part without a barrier, operands straight from memory into registers (32 indices in flight while 32 are multiplied), and
// the sums meet in LDS at the end.  Nothing is rearranged beforehand: backward-data reads the filters where they are, at
// strides > 1 too, and a small bias gradient rides in blocks of its own.  A wave works out the offsets of 64 reduction
// indices at a time, one a lane, and reads them back from LDS, so that an element costs an add and (beside padding) a
// window test.  Every block loads 48 values for 16 x 32 products, which is what ends its range (direct_choice).
// 5 images of 19 channels 33x29 -> 37 rows, 5x3 stride 2, all three passes 49.7 -> 28.1 us; 16 images of 86x95, 504 -> 1
// channels, 3x3 stride 2 backward-data 290 -> 51 us.  Tiles of 32 x 32 were faster for a few problems (1 - 2 % in the
// mean over all) and spill beside 16 waves; 64 x 32 never.
#include <atomic>
#include <cstdio>
#include "cg_internal.h"
#include "igemm_device.h"
#include "split_device.h"

namespace cg {

namespace {

constexpr int TM = 1, TN = 2, MT = 16 * TM, NT = 16 * TN;
constexpr int TABLE = 64;                    // reduction indices whose offsets a wave works out at a time
constexpr int STEP = 32;                     // reduction indices in registers at a time, twice (this step's, the next one's)

enum { AD_WORDS = 0, AD_CHECKED = 1, AD_QUADS = 2 };      // how an operand is loaded: element by element, where the window has one, aligned quads of k

// byte offset of an index of an operand, and its window coordinates
struct Entry { uint32_t off; int32_t a, b; };
__device__ __forceinline__ Entry entry_of(const IndexMap &m, uint32_t k, uint32_t kend)
{
    const Info q = map_info(m, k);
    const bool ok = k < kend && (m.r1_lim == 0 || q.r1 < m.r1_lim);
    return Entry{ok ? (uint32_t)q.off * 4u : OOB_K, q.a, q.b};
}

__device__ __forceinline__ float ldw(__amdgpu_buffer_rsrc_t r, uint32_t voff)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, 0));
}

// One element of C by itself: bias, rectifier, gate, accumulation, the output map.
template <bool SCATTER> __device__ __forceinline__ void store_element(const IgemmProblem &a, uint32_t g, uint32_t m, uint32_t n, float s)
{
    if (a.bias_mode == 1) s += a.bias[(int64_t)g * a.bias_gstride + m];
    else if (a.bias_mode == 2) s += a.bias[(int64_t)g * a.bias_gstride + n];
    if (a.relu) s = fmaxf(s, 0.f);
    const Info ci = map_info(a.c_col, n);
    int32_t in_group = (int32_t)m * a.c_row_stride + ci.off;
    if constexpr (SCATTER) {
        const Info ri = map_info(a.c_row, m);
        if (!((uint32_t)(ri.a + ci.a) < a.c_limA && (uint32_t)(ri.b + ci.b) < a.c_limB)) return;
        if (!__builtin_isfinite(s)) {
            const auto &f = first_argument<IgemmProblem>();
            s = sum_of_taps(f.taps, f.c_row, f.c_col, g, m, n);
        }
        in_group = ri.off + ci.off;
    }
    const int64_t idx = (int64_t)g * a.c_gstride + in_group;
    if (a.gate && !(a.gate[idx] > 0.f)) s = 0.f;
    float *dst = a.c_ptr + idx;
    if (a.accumulate) s += *dst;
    *dst = s;
}

// offsets of TABLE reduction indices of one wave: B's offset and window coordinates, A's likewise where it has them
template <int AKIND, int BKIND> struct Table {
    static constexpr bool BCHECK = BKIND == AD_CHECKED;
    static constexpr int COLS = 1 + (BCHECK ? 2 : 0) + (AKIND == AD_QUADS ? 0 : AKIND == AD_CHECKED ? 3 : 1);
    static constexpr int WORDS = COLS * TABLE;
    static constexpr int BA = 1, BB = 2, AO = BCHECK ? 3 : 1, AA = AO + 1, AB = AO + 2;
};

}  // namespace

struct DirectArgs {
    IgemmProblem p;
    FastDiv divNT, divMT, divG;              // column tiles, row tiles, groups
    uint32_t tiles, k_per_wave;
    BiasRider rider;                         // blocks behind the tiles: a channel of a convolution's bias gradient each
    FastDiv divQP;
};

static_assert(offsetof(DirectArgs, p) == 0, "the problem is the start of a kernel's arguments");

template <int AKIND, int BKIND>
__global__ __launch_bounds__(1024) void direct_kernel(const DirectArgs d)
{
    using T = Table<AKIND, BKIND>;
    constexpr bool BCHECK = BKIND == AD_CHECKED;
    constexpr int LS = NT + 4;
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    const IgemmProblem &p = d.p;
    if (blockIdx.x >= d.tiles) {
        const int m = (int)(blockIdx.x - d.tiles);
        const float s = bias_channel_sum(d.rider.dy, d.rider.M, d.rider.P, m, 0, d.rider.N, d.divQP, blockDim.x, reinterpret_cast<float *>(smem));
        if (threadIdx.x == 0) d.rider.db[m] = s;
        return;
    }
    const int lane = threadIdx.x & 63, q = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t r = fdiv(blockIdx.x, d.divNT), gs = fdiv(r, d.divMT), sp = fdiv(gs, d.divG), g = gs - sp * d.divG.d;
    const uint32_t m0 = (r - gs * d.divMT.d) * MT, n0 = (blockIdx.x - r * d.divNT.d) * NT;
    const uint32_t kbeg = sp * p.k_per_split + (uint32_t)wave * d.k_per_wave, kend = min(min(p.K, (sp + 1) * p.k_per_split), kbeg + d.k_per_wave);
    const int ns = kbeg < kend ? (int)((kend - kbeg + STEP - 1) / STEP) : 0;

    const int64_t fa = (int64_t)g * p.A.gstride + p.A.shift, fb = (int64_t)g * p.B.gstride + p.B.shift;
    const auto rA = buffer_of(p.A.ptr + fa, (uint64_t)((int64_t)p.A.elems - fa) * 4u);
    const auto rB = buffer_of(p.B.ptr + fb, (uint64_t)((int64_t)p.B.elems - fb) * 4u);

    uint32_t arow[TM], brow[TN];
    int32_t ara[TM], arb[TM], bra[TN], brb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t row = m0 + (uint32_t)(16 * i + l16);
        const Info e = map_info(p.A.row, row);
        arow[i] = row < p.M ? (uint32_t)e.off * 4u : OOB_ROW;
        ara[i] = e.a; arb[i] = e.b;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const uint32_t col = n0 + (uint32_t)(16 * j + l16);
        const Info e = map_info(p.B.row, col);
        brow[j] = col < p.N ? (uint32_t)e.off * 4u : OOB_ROW;
        bra[j] = e.a; brb[j] = e.b;
    }

    // ---- the wave's own table, two of TABLE indices: nobody else reads it, so no barrier ------------------
    uint32_t *const tab = smem + wave * 2 * T::WORDS;
    auto fill = [&](int t) {
        uint32_t *to = tab + (t & 1) * T::WORDS + lane;
        const uint32_t k = kbeg + (uint32_t)(t * TABLE + lane);
        const Entry e = entry_of(p.B.k, k, kend);
        to[0] = e.off;
        if constexpr (BCHECK) { to[T::BA * TABLE] = (uint32_t)e.a; to[T::BB * TABLE] = (uint32_t)e.b; }
        if constexpr (AKIND != AD_QUADS) {
            const Entry f = entry_of(p.A.k, k, kend);
            to[T::AO * TABLE] = f.off;
            if constexpr (AKIND == AD_CHECKED) { to[T::AA * TABLE] = (uint32_t)f.a; to[T::AB * TABLE] = (uint32_t)f.b; }
        }
        // other lanes of the wave read this: no instruction, but nothing moves across
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // the four consecutive indices of this lane in 16 of them: column c of the table
    auto four = [&](int s, int h, int c) {
        return *reinterpret_cast<const v4u *>(tab + ((s >> 1) & 1) * T::WORDS + c * TABLE + (s & 1) * STEP + 16 * h + 4 * q);
    };

    float av[2][STEP / 16][TM][4], bv[2][STEP / 16][TN][4];
    auto load = [&](auto BC, int s) {
        constexpr int b = decltype(BC)::value;
#pragma unroll
        for (int h = 0; h < STEP / 16; ++h) {
            if constexpr (AKIND == AD_QUADS) {
                const uint32_t k = kbeg + (uint32_t)(s * STEP + 16 * h + 4 * q);
                const uint32_t ko = k < kend ? (uint32_t)map_info(p.A.k, k).off * 4u : OOB_K;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rA, arow[i] + ko, 0, 0);
#pragma unroll
                    for (int t = 0; t < 4; ++t) av[b][h][i][t] = __uint_as_float((uint32_t)v[t]);
                }
            } else {
                const v4u ao = four(s, h, T::AO);
                v4u aa{}, ab{};
                if constexpr (AKIND == AD_CHECKED) { aa = four(s, h, T::AA); ab = four(s, h, T::AB); }
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        uint32_t at = arow[i];
                        if constexpr (AKIND == AD_CHECKED)
                            at = (uint32_t)(ara[i] + (int32_t)aa[t]) < p.A.limA && (uint32_t)(arb[i] + (int32_t)ab[t]) < p.A.limB ? at : OOB_ROW;
                        av[b][h][i][t] = ldw(rA, at + ao[t]);
                    }
            }
            const v4u bo = four(s, h, 0);
            if constexpr (BKIND == AD_QUADS) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rB, brow[j] + bo[0], 0, 0);
#pragma unroll
                    for (int t = 0; t < 4; ++t) bv[b][h][j][t] = __uint_as_float((uint32_t)v[t]);
                }
                continue;
            }
            v4u ba{}, bb{};
            if constexpr (BCHECK) { ba = four(s, h, T::BA); bb = four(s, h, T::BB); }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    uint32_t at = brow[j];
                    if constexpr (BCHECK)
                        at = (uint32_t)(bra[j] + (int32_t)ba[t]) < p.B.limA && (uint32_t)(brb[j] + (int32_t)bb[t]) < p.B.limB ? at : OOB_ROW;
                    bv[b][h][j][t] = ldw(rB, at + bo[t]);
                }
        }
    };

    v4f acc[2][TM][TN];                      // even and odd sixteens: half the chain, half the rounding of it
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[h][i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](auto BC, int s) {
        constexpr int b = decltype(BC)::value;
#pragma unroll
        for (int h = 0; h < STEP / 16; ++h) {
            if constexpr (AKIND == AD_QUADS) {
                // what a quad holds behind the last index (of the reduction, of a run) may be anything; an element of B is zero there
                const v4u bo = four(s, h, 0);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i) av[b][h][i][t] = bo[t] < OOB_K ? av[b][h][i][t] : 0.f;
                if constexpr (BKIND == AD_QUADS)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int j = 0; j < TN; ++j) bv[b][h][j][t] = bo[t] < OOB_K ? bv[b][h][j][t] : 0.f;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[h][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[b][h][j][t], av[b][h][i][t], acc[h][i][j], 0, 0, 0);
        }
    };

    if (ns > 0) {
        fill(0);
        load(std::integral_constant<int, 0>{}, 0);
        for (int s = 0; s < ns; s += 2) {
            load(std::integral_constant<int, 1>{}, s + 1);
            multiply(std::integral_constant<int, 0>{}, s);
            if (s + 1 >= ns) break;
            if (s + 2 < ns) {
                fill(s / 2 + 1);
                load(std::integral_constant<int, 0>{}, s + 2);
            }
            multiply(std::integral_constant<int, 1>{}, s + 1);
        }
    }

    // ---- the waves' sums meet in LDS and are added in wave order -------------------------------------------
    block_sync_lds();                        // (every wave is done with its table)
    float *const red = reinterpret_cast<float *>(smem);
    const int waves = (int)(blockDim.x >> 6);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            *reinterpret_cast<v4f *>(red + (wave * MT + 16 * i + l16) * LS + 16 * j + 4 * q) = acc[0][i][j] + acc[1][i][j];
    block_sync_lds();
    for (uint32_t e = threadIdx.x; e < (uint32_t)(MT * NT); e += blockDim.x) {
        const uint32_t row = e / NT, col = e % NT, m = m0 + row, n = n0 + col;
        if (m >= p.M || n >= p.N) continue;
        float s = red[row * LS + col];
        for (int w = 1; w < waves; ++w) s += red[(w * MT + (int)row) * LS + (int)col];
        if (p.splits > 1) p.c_ptr[(int64_t)g * p.c_gstride + (int64_t)sp * p.c_split_stride + (int64_t)m * p.c_row_stride + n] = s;
        else store_element<AKIND == AD_CHECKED>(p, g, m, n, s);       // (strided backward-data)
    }
}

namespace {

template <int AKIND, int BKIND> int launch_cfg(const IgemmProblem &p, int waves, const BiasRider *rider, hipStream_t stream)
{
    DirectArgs d{};
    d.p = p;
    const uint32_t nt = (p.N + NT - 1) / NT, mt = (p.M + MT - 1) / MT;
    const uint64_t tiles = (uint64_t)nt * mt * p.groups * p.splits;
    if (tiles >= (1u << 30)) return CG_EUNSUPPORTED;
    d.tiles = (uint32_t)tiles;
    d.divNT = make_fastdiv(nt);
    d.divMT = make_fastdiv(mt);
    d.divG = make_fastdiv(p.groups);
    d.k_per_wave = ((p.k_per_split + waves - 1) / waves + 15) / 16 * 16;
    unsigned riders = 0;
    if (rider) {
        d.rider = *rider;
        d.divQP = make_fastdiv((uint32_t)(rider->P + 3) / 4);
        riders = (unsigned)rider->M;
    }
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, "igemm_direct_kernel<%dx%d,%c%c>", MT, NT, "rc4"[AKIND], "rc4"[BKIND]);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    const size_t tab = (size_t)waves * 2 * Table<AKIND, BKIND>::WORDS * 4, sums = (size_t)waves * MT * (NT + 4) * 4;
    static_assert(16 * 2 * Table<AKIND, BKIND>::WORDS * 4 <= 64 * 1024 && 16 * MT * (NT + 4) * 4 <= 64 * 1024, "what a block of 16 waves gets without asking");
    size_t lds = tab > sums ? tab : sums;
    if (riders && lds < 4096) lds = 4096;                       // a rider block adds up one float a thread
    hipLaunchKernelGGL((direct_kernel<AKIND, BKIND>), dim3((unsigned)tiles + riders), dim3((unsigned)waves * 64), lds, stream, d);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

}  // namespace

// Expected times, us, from 1268 passes of 220 problems (windows 1 to 11, 1 to 512 channels, 7 to 227 pixels a side, up to
// 2 GFLOP), each run here with 4, 8 and 16 waves and on the gathered kernel: one standard deviation of the relative error
// is 11 - 17 % here and 16 % there.  `start` is what a call costs in any case.  Here a wave's steps of 32 indices follow
// one another, and what the waves of a SIMD load adds up; there K-tiles of a block do, and a second launch adds K slices, a
// first one makes a copy of the filters.  Chosen by these (below 0.9 of the other) forward became faster by 14 %,
// backward-data by 45 %, backward-weight by 4 % in the mean, 7 of 660 passes slower than 0.97 (0.77 at worst); one at 9 us
// is bound by the host.  Mean error against 64 bits 0.6 of the gathered kernel's: a wave's chain is no longer than the larger of
// its K slice and 144 indices (where there is such a plan).
static double direct_cost(const IgemmProblem &p, bool a_quads, uint64_t tiles, int waves)
{
    struct Fit { double start, step, load, check, wave; };
    static const Fit quads{6.0, 0.218, 0.556, 0.183, 0.199}, across{6.3, 0.037, 0.793, 0.056, 0.}, words{6.0, 0.279, 0.387, 0.326, 0.138},
        checked{5.2, 0.427, 0.061, 0.541, 0.352};
    const Fit &f = p.A.check ? checked : !a_quads ? words : p.B.lanes_k ? across : quads;
    const uint64_t per = ((p.K + waves - 1) / waves + 15) / 16 * 16;
    const double steps = (double)((per + STEP - 1) / STEP), simd = (double)tiles * waves / (2. * igemm_resident_blocks()), all = (simd > 1. ? simd : 1.) * steps;
    return f.start + f.step * steps + all * (f.load + (p.B.check ? f.check : 0.)) + f.wave * simd;
}

static std::atomic<int> g_enabled{1};
void direct_set_enabled(int on) { g_enabled.store(on ? 1 : 0, std::memory_order_relaxed); }

int direct_choice(const IgemmProblem &p, bool a_quads, const SplitPlan *other, bool other_copies)
{
    if (p.math != CG_MATH_FP32 || !g_enabled.load(std::memory_order_relaxed)) return 0;
    // A gathered from dy or from rows of a matrix beside a B that runs along k as well: neighbouring lanes lie far apart, and
    // beyond a few hundred indices the loads take longer than the second launch (181 x 68 with 2048 indices 35.3 / 12.9)
    if (p.B.lanes_k && p.K > 768) return 0;
    // Where the gathered kernel needs no copy of the filters either (forward, 1x1 backward-data): from about 0.38 GFLOP on what
    // is gained is within the fit's error (13 forward problems 0.96 - 1.47, median 1.1; below 98 problems, 1.35), and long rows
    // of pixels suit its loaders (35 x 55575 with 243 indices 50.3 / 27.7)
    if (other && !other_copies && 2. * p.M * (double)p.N * p.K * p.groups > 0.375e9) return 0;
    const uint64_t tiles = (uint64_t)((p.N + NT - 1) / NT) * ((p.M + MT - 1) / MT) * p.groups;
    if (tiles >= (1u << 30) || (other && 2. * p.M * (double)p.N * p.K * p.groups > 2e9)) return 0;       // (beyond what was fitted)
    int best = 0;
    double cost = 1e300;
    for (int waves = 4; waves <= 16; waves *= 2) {
        const uint32_t per = ((p.K + waves - 1) / waves + 15) / 16 * 16;
        if (other && per > (other->k_per_split > 144 ? other->k_per_split : 144)) continue;
        const double t = direct_cost(p, a_quads, tiles, waves);
        if (t < cost) { cost = t; best = waves; }
    }
    if (!best || !other) return best;
    const uint64_t blocks = (uint64_t)((p.M + other->mt - 1) / other->mt) * ((p.N + 127) / 128) * p.groups * other->splits;
    const double runs = (double)((blocks * 2 + igemm_resident_blocks() - 1) / igemm_resident_blocks()) * (double)((other->k_per_split + 15) / 16);
    const double there = 7.9 + runs * (0.0129 * other->mt + (p.B.check ? 0.181 : 0.)) + (other_copies ? 2.9 : 0.) +
                         (other->splits > 1 ? 2.4 + 1.3e-6 * other->splits * p.M * (double)p.N * p.groups : 0.);
    return cost < 0.9 * there ? best : 0;
}

// Sums over pixels (both operands run along k) of few columns: a 128-column tile of the gathered kernel is mostly padding, here
// the columns fit one tile of 32.  190 problems, times there / here: up to 32 columns 1.05 - 3.2 (16 x 4 with 3 836 300 indices 417 /
// 132 us, 394 x 1 with 124 768 178 / 95), 33 - 43 columns 0.6 - 1.5; more columns with few tiles and indices (the launch and a block's
// start are what counts) 1.0 - 1.34 up to 140 000 tiles x indices, 0.85 - 1.0 to 280 000, 0.4 - 0.9 beyond.  Four waves; eight and
// sixteen 0.5 - 1.0 of that.  Error against 64 bits 0.25 to 0.75 of the gathered kernel's.
int direct_for_slices(const IgemmProblem &p, bool a_quads)
{
    if (p.math != CG_MATH_FP32 || !p.B.lanes_k || !a_quads || !g_enabled.load(std::memory_order_relaxed)) return 0;
    const uint64_t tiles = (uint64_t)((p.N + NT - 1) / NT) * ((p.M + MT - 1) / MT) * p.groups;
    return p.N <= 32 || tiles * p.K <= 140000 ? 4 : 0;
}

// (normalised by igemm_launch)
int direct_launch(const IgemmProblem &p, bool a_quads, bool b_quads, hipStream_t stream)
{
    const int waves = p.direct;
    const BiasRider *rider = p.rider.dy ? &p.rider : nullptr;
    if (waves != 4 && waves != 8 && waves != 16) return CG_EINVAL;
    const bool bc = p.B.check != 0;
    if (b_quads) return a_quads && !bc ? launch_cfg<AD_QUADS, AD_QUADS>(p, waves, rider, stream) : CG_EINVAL;
    if (p.A.check) return bc ? launch_cfg<AD_CHECKED, AD_CHECKED>(p, waves, rider, stream) : launch_cfg<AD_CHECKED, AD_WORDS>(p, waves, rider, stream);
    if (a_quads) return bc ? launch_cfg<AD_QUADS, AD_CHECKED>(p, waves, rider, stream) : launch_cfg<AD_QUADS, AD_WORDS>(p, waves, rider, stream);
    return bc ? launch_cfg<AD_WORDS, AD_CHECKED>(p, waves, rider, stream) : launch_cfg<AD_WORDS, AD_WORDS>(p, waves, rider, stream);
}

}  // namespace cg
