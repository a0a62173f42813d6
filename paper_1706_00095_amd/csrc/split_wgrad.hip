// Backward-weight of windows of five and more taps on the bf16 matrix instructions:
//   dw[m][c][tap] = sum over images and pixels of dy[n][m][pix] * x[n][c][window of pix at tap].
// split_gemm_kernel gathers x once per tap and column tile, and that gather (an address, a range check
// and a cut per element) is what it is bound by.  Here the reduction walks units (a few images, or a
// band of rows of one): for a unit a block keeps the zero-padded source rows of 16 input channels in
// LDS, cut into NP bf16 pieces once, as [piece][slot][16 channels], and multiplies all (at most nine)
// taps of its columns from there.  The matrix instruction wants eight PIXELS of a channel per lane where
// the patch has 16 CHANNELS of a pixel together: ds_read_b64_tr_b16 transposes 4 x 16 values on the way
// out of LDS, and since every lane names its own pixel's address, rows that wrap, strides and padding
// cost nothing.  dy goes from memory straight into registers, eight consecutive pixels of a row per
// lane; wave w owns 16*TM rows and all the columns, as in split_patch.hip (which also says why
// v_mfma_f32_16x16x32_bf16 and what the pieces do to the error).
// An image's pixels (a band's) are padded to a multiple of eight in the index space, so that a lane's
// eight never straddle two; the padding reads zeros of x.
#include <atomic>
#include <cstdio>
#include "cg_internal.h"
#include "igemm_device.h"
#include "split_device.h"

namespace cg {

namespace {

constexpr int TT = 9;                        // taps per block
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// Lanes 16g .. 16g+15 name four rows (pixels) of 16 values, lane i the 8-byte piece i % 4 of row i / 4 of its
// group; lane i receives value i of the four rows.
__device__ __forceinline__ v2u read_transposed(const char *lds_base, int32_t byte)
{
    return __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)(lds_base + byte)));
}

template <int NP, int NSL> struct BandLds {
    static constexpr int SLOTS = NSL * 64, PLANE = (SLOTS + 1) * 32;       // bytes; the last slot is zeros
    static constexpr size_t BYTES = (size_t)NP * PLANE;
};

}  // namespace

template <int NP, int TM, int NSL>
__global__ __launch_bounds__(256, 2) void split_wgrad_kernel(const IgemmProblem p)
{
    using L = BandLds<NP, NSL>;
    constexpr int MT = 64 * TM, NC = NSL / 2;               // chunks of 64 slots a wave brings
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const BandGeom &g = p.band;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, l16 = lane & 15;
    const uint32_t gr = __builtin_amdgcn_readfirstlane(blockIdx.z / p.splits), sp = blockIdx.z - gr * p.splits;
    const int cblk = __builtin_amdgcn_readfirstlane(blockIdx.x / g.tap_blocks), t0 = ((int)blockIdx.x - cblk * g.tap_blocks) * TT;
    const int c0 = cblk * 16, KK = g.KH * g.KW, P = g.OH * g.OW, HW = g.H * g.W;
    const uint32_t mw = blockIdx.y * MT + (uint32_t)(wave * TM * 16);
    const int u0 = (int)sp * g.units_per_split, u1 = min(g.units, u0 + g.units_per_split);

    const auto rX = buffer_of(g.x + (int64_t)gr * g.Cg * HW, (g.x_elems - (uint64_t)gr * g.Cg * HW) * 4);
    const auto rY = buffer_of(g.dy + (int64_t)gr * p.M * P, (g.dy_elems - (uint64_t)gr * p.M * P) * 4);

    // a unit: images n0 .. n0+ipu-1, output rows oy0 .. oy0+rows-1 of each
    struct Unit { int n0, oy0, npix; };
    auto unit_of = [&](int u) {
        const int grp = (int)fdiv((uint32_t)u, g.divNB), jb = u - grp * g.nb;
        return Unit{grp * g.ipu, jb * g.Rb, min(g.Rb, g.OH - jb * g.Rb) * g.OW};
    };

    // ---- patch: wave w brings channels 8 (w % 2) .. + 7, chunks (w / 2) + 2 e --------------------------
    int32_t sr[NC], sc[NC], simg[NC];        // row, column, image of this lane's slot in chunk e (row < 0: none)
#pragma unroll
    for (int e = 0; e < NC; ++e) {
        const uint32_t j = (uint32_t)(((wave >> 1) + 2 * e) * 64 + lane);
        const uint32_t seg = fdiv(j, g.divSS), in = j - seg * g.divSS.d, r = fdiv(in, g.divWp);
        simg[e] = (int32_t)seg;
        sr[e] = (int32_t)seg < g.ipu ? (int32_t)r : -(1 << 24);
        sc[e] = (int32_t)(in - r * g.divWp.d) - g.pad_w;
    }
    float pr[NC][8];
    auto load_chunk = [&](auto EC, int u) {
        constexpr int e = decltype(EC)::value;
        const Unit un = unit_of(u);
        const int32_t sy = un.oy0 * g.s - g.pad_h + sr[e], n = un.n0 + simg[e];
        const bool ok = (uint32_t)sy < (uint32_t)g.H && (uint32_t)sc[e] < (uint32_t)g.W && n < g.N && u < u1;
        const uint32_t voff = ok ? (uint32_t)((n * g.C) * HW + sy * g.W + sc[e]) * 4u : OOB_ROW;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int c = c0 + 8 * (wave & 1) + t;
            pr[e][t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rX, voff, c < g.Cg ? (uint32_t)(c * HW) * 4u : OOB_K, 0));
        }
    };
    auto store_chunk = [&](auto EC) {
        constexpr int e = decltype(EC)::value;
        v4u pc[NP];
        split8<NP>(pr[e], pc);
        char *at = smem + (((wave >> 1) + 2 * e) * 64 + lane) * 32 + (wave & 1) * 16;
#pragma unroll
        for (int k = 0; k < NP; ++k) *reinterpret_cast<v4u *>(at + k * L::PLANE) = pc[k];
    };

    // ---- dy: row 16 i + lane % 16, octet lane / 16 of a step's pixels -----------------------------------
    uint32_t yrow[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t m = mw + (uint32_t)(i * 16 + l16);
        yrow[i] = m < p.M ? m * (uint32_t)P * 4u : OOB_ROW;
    }
    float ar[TM][8];
    auto load_a = [&](int u, int s) {
        const Unit un = unit_of(u);
        const uint32_t oc = (uint32_t)(4 * s + q), seg = fdiv(oc, g.divP8), po = (oc - seg * g.divP8.d) * 8u;
        const int n = un.n0 + (int)seg;
        const bool live = u < u1 && (int)seg < g.ipu && n < g.N;
        const uint32_t off = (uint32_t)(n * g.M * P + un.oy0 * g.OW + (int)po) * 4u;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const uint32_t ko = live && (int)po + 4 * hf < un.npix ? off + 16u * hf : OOB_K;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(rY, yrow[i] + ko, 0, 0);
#pragma unroll
                for (int t = 0; t < 4; ++t) ar[i][4 * hf + t] = __uint_as_float((uint32_t)v[t]);
            }
        }
    };

    // slot displacement of the block's taps, in bytes
    int32_t toff[TT];
#pragma unroll
    for (int j = 0; j < TT; ++j) {
        const int t = min(t0 + j, KK - 1), ky = (int)fdiv((uint32_t)t, g.divKW);
        toff[j] = __builtin_amdgcn_readfirstlane((ky * g.Wp + (t - ky * g.KW)) * 32);
    }

    v4f acc[TM][TT];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    if (threadIdx.x < 8 * NP) *reinterpret_cast<uint32_t *>(smem + (threadIdx.x >> 3) * L::PLANE + L::SLOTS * 32 + (threadIdx.x & 7) * 4) = 0u;
    static_for<0, NC>([&](auto EC) { load_chunk(EC, u0); });
    load_a(u0, 0);
    static_for<0, NC>([&](auto EC) { store_chunk(EC); });
    block_sync_lds();

    for (int u = u0; u < u1; ++u) {
        const Unit un = unit_of(u);
        for (int s = 0; s < g.steps; ++s) {
            // this lane's octet of pixels: image of the unit, first pixel in the band
            const uint32_t oc = (uint32_t)(4 * s + q), seg = fdiv(oc, g.divP8);
            const int32_t po = (int32_t)(oc - seg * g.divP8.d) * 8;
            // A quad that reaches beyond the band's last pixel brings what follows in memory (the next row's
            // pixels, or the next channel's): it would meet zeros of x, but an infinity or a NaN times zero is NaN.
            if ((un.npix & 3) != 0 && __any(po < un.npix && po + 8 > un.npix))
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i) ar[i][t] = po + t < un.npix ? ar[i][t] : 0.f;
            v4u ap[TM][NP];
#pragma unroll
            for (int i = 0; i < TM; ++i) split8<NP>(ar[i], ap[i]);
            // a chunk of the next unit's patch, then the next step's rows
            static_for<0, NC>([&](auto EC) { if (s == decltype(EC)::value) load_chunk(EC, u + 1); });
            if (s + 1 < g.steps) load_a(u, s + 1);
            else load_a(u + 1, 0);
            // the two pixels this lane names in the transposed reads
            int32_t at[2], mask[2];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const int32_t px = po + 4 * hf + (l16 >> 2);
                const uint32_t row = fdiv((uint32_t)px, g.divOW);
                const int32_t col = px - (int32_t)(row * g.divOW.d);
                const bool ok = (int)seg < g.ipu && px < un.npix && un.n0 + (int)seg < g.N;
                mask[hf] = ok ? -1 : 0;
                at[hf] = (ok ? (int32_t)(seg * g.divSS.d) + (int32_t)row * g.s * g.Wp + col * g.s : L::SLOTS) * 32 + (l16 & 3) * 8;
            }
            using Step = MmaStep<NP, TM, TT, TM == 1 ? 3 : 1>;
            auto read_b = [&](int j, v4u (&pc)[NP]) {
                const int32_t a0 = at[0] + (toff[j] & mask[0]), a1 = at[1] + (toff[j] & mask[1]);
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const v2u lo = read_transposed(smem, a0 + k * L::PLANE), hi = read_transposed(smem, a1 + k * L::PLANE);
                    pc[k] = v4u{lo.x, lo.y, hi.x, hi.y};
                }
            };
            Step::run(ap, acc, read_b, typename Step::NoWork{});
        }
        if (u + 1 < u1) {
            static_for<0, NC>([&](auto EC) { if (g.steps <= decltype(EC)::value) load_chunk(EC, u + 1); });
            block_sync_lds();
            static_for<0, NC>([&](auto EC) { store_chunk(EC); });
            block_sync_lds();
        }
    }

    if constexpr (NP == 3) {
        if (not_finite(acc)) sums_in_fp32(acc, [&](int j, auto &&add) {
            const int t = min(t0 + j, KK - 1), ky = (int)fdiv((uint32_t)t, g.divKW), kx = t - ky * g.KW;
            for (int u = u0; u < u1; ++u) {
                const Unit un = unit_of(u);
                for (int n = un.n0; n < min(un.n0 + g.ipu, g.N); ++n)
                    for (int p0 = 0; p0 < un.npix; p0 += 16) {
                        // 16 pixels, four consecutive ones a lane, their loads in flight together
                        float a[4][TM], b[4];
                        const int32_t p4 = p0 + 4 * q;
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const auto f = __builtin_amdgcn_raw_buffer_load_b128(
                                rY, p4 < un.npix ? yrow[i] + (uint32_t)(n * g.M * P + un.oy0 * g.OW + p4) * 4u : OOB_K, 0, 0);
#pragma unroll
                            for (int v = 0; v < 4; ++v) a[v][i] = p4 + v < un.npix ? __uint_as_float((uint32_t)f[v]) : 0.f;
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int32_t px = p4 + v, row = (int32_t)fdiv((uint32_t)px, g.divOW), col = px - row * g.OW;
                            const int32_t sy = (un.oy0 + row) * g.s - g.pad_h + ky, sx = col * g.s - g.pad_w + kx;
                            const bool ok = px < un.npix && c0 + l16 < g.Cg && (uint32_t)sy < (uint32_t)g.H && (uint32_t)sx < (uint32_t)g.W;
                            b[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                rX, ok ? (uint32_t)((n * g.C + c0 + l16) * HW + sy * g.W + sx) * 4u : OOB_K, 0, 0));
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) add(a[v], b[v]);
                    }
            }
        });
    }
    // Lane (q, l) holds, for row l of a 16-row tile, the channels 4q .. 4q+3 of every tap: where the block has
    // all nine taps, 36 consecutive floats.
    float *c_base = p.c_ptr + (int64_t)gr * p.c_gstride + (int64_t)sp * p.c_split_stride;
    const int cq = c0 + 4 * q;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t m = mw + (uint32_t)(i * 16 + l16);
        if (m >= p.M) continue;
        float *row = c_base + (int64_t)m * p.c_row_stride;
        if (KK == TT && cq + 4 <= g.Cg) {
#pragma unroll
            for (int e = 0; e < TT; ++e) {
                f4u v;
#pragma unroll
                for (int f = 0; f < 4; ++f) v[f] = acc[i][(4 * e + f) % TT][(4 * e + f) / TT];
                *reinterpret_cast<f4u *>(row + cq * TT + 4 * e) = v;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < TT; ++j)
                    if (cq + r < g.Cg && t0 + j < KK) row[(cq + r) * KK + t0 + j] = acc[i][j][r];
        }
    }
}

namespace {

template <int NP, int TM, int NSL> int launch_cfg(const IgemmProblem &p, hipStream_t stream)
{
    constexpr int MT = 64 * TM;
    dim3 grid((unsigned)(((p.band.Cg + 15) / 16) * p.band.tap_blocks), (p.M + MT - 1) / MT, p.groups * p.splits);
    if (grid.y > 65535u || grid.z > 65535u) return CG_EUNSUPPORTED;
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, NP == 3 ? "igemm_kernel<%dx%d,band%d>" : NP == 1 ? "igemm_kernel<%dx%d,band%d,bf16>" : "igemm_kernel<%dx%d,band%d,bf16x3>", MT, 16 * TT, NSL);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    constexpr size_t lds = BandLds<NP, NSL>::BYTES;
    static_assert(2 * lds <= 160 * 1024, "two blocks of this tile do not fit the LDS of a compute unit");
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        CG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&split_wgrad_kernel<NP, TM, NSL>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((split_wgrad_kernel<NP, TM, NSL>), grid, dim3(256), lds, stream, p);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

}  // namespace

// This file is compiled once per number of pieces (CG_NP), in parallel.
#define CG_CAT_(a, b) a##b
#define CG_CAT(a, b) CG_CAT_(a, b)
int CG_CAT(split_wgrad_, CG_NP)(const IgemmProblem &p, hipStream_t stream)
{
    const int mt = p.band.mt;
    if (p.band.nsl == 4)
        return mt == 192 ? launch_cfg<CG_NP, 3, 4>(p, stream) : mt == 128 ? launch_cfg<CG_NP, 2, 4>(p, stream) : launch_cfg<CG_NP, 1, 4>(p, stream);
    return mt == 128 ? launch_cfg<CG_NP, 2, 8>(p, stream) : mt == 64 ? launch_cfg<CG_NP, 1, 8>(p, stream) : CG_EUNSUPPORTED;
}

#if CG_NP == 3
int split_wgrad_1(const IgemmProblem &p, hipStream_t stream);
int split_wgrad_2(const IgemmProblem &p, hipStream_t stream);

int split_wgrad_launch(const IgemmProblem &p, hipStream_t stream)
{
    const BandGeom &g = p.band;
    if (!p.c_ptr || !aligned16(p.c_ptr) || !g.x || !aligned16(g.x) || !g.dy || !aligned16(g.dy) || (g.nsl != 4 && g.nsl != 8) || p.M == 0 ||
        p.bias_mode || p.gate || p.accumulate || p.relu || p.c_scatter || (uint64_t)p.splits * g.units_per_split < (uint64_t)g.units)
        return CG_EINVAL;
    if (p.math == CG_MATH_BF16) return split_wgrad_1(p, stream);
    if (p.math == CG_MATH_BF16X3) return split_wgrad_2(p, stream);
    return p.math == CG_MATH_FP32 ? split_wgrad_3(p, stream) : CG_EINVAL;
}

// Expected times of this kernel and of the gathered one, us.  Fitted to 520 problems (9 to 384 channels a group, 33 to
// 448 rows, windows 2x3 to 7x7 and rows and columns of 5 to 11, strides 1 and 2, planes 7 to 60 wide, batches 2 to 256)
// in each arithmetic; one standard deviation of the relative error is 10 - 13 % and 5 - 11 %.  A block of this
// kernel multiplies whole 16 channels, nine taps, 32 pixels and mt rows, brings a patch a unit, and stores one by one
// unless the window has nine taps; the gathered kernel's blocks run one after another or in pairs on a compute unit and
// check every element where there is padding; both write their slices and read them again.
// Chosen by these the problems took 71.7 ms in fp32 (all here 83.0, all there 79.0, each at its best 71.5), 36.7 in
// bf16 (49.0, 37.9, 36.5), 45.8 in bf16x3 (59.2, 48.0, 45.7).
static double band_cost(const BandGeom &g, int chunks, double plane, uint64_t blocks, uint32_t splits, uint64_t resident, int math)
{
    struct Fit { double start, row, step, row_pair, step_pair, unit, unit8, byte, scattered; };
    static const Fit fit[3] = {{13.6, 0.543, 0.334, 0.502, 0., 1.66, 0., 2.59e-7, 7.82e-7},
                               {12.4, 0., 0.412, 0.291, 0.00465, 0.669, 0.328, 2.98e-7, 8.05e-7},
                               {13.3, 0.179, 0.398, 0.345, 0., 0.914, 0.315, 2.64e-7, 8.18e-7}};
    const Fit &f = fit[math];
    const bool pair = blocks * 2 > resident;
    const double rounds = (double)((blocks + resident - 1) / resident), units = rounds * g.units_per_split, steps = units * g.steps;
    return f.start + steps * (g.mt / 64 * (f.row + (pair ? f.row_pair : 0.)) + f.step + (pair ? f.step_pair : 0.)) +
           units * (f.unit + (chunks == 8 ? f.unit8 : 0.)) + splits * plane * ((splits > 1 ? f.byte * 2. : 0.) + (g.KH * g.KW != TT ? f.scattered : 0.));
}

static double gathered_cost(const SplitPlan &o, uint64_t blocks, double plane, bool padded, uint64_t resident, int math)
{
    struct Fit { double start, row, tile, check, byte, many; };
    static const Fit fit[3] = {{11.2, 0.00741, 0.118, 0.0939, 2.05e-7, 2.74},
                               {11.2, 0.00163, 0.184, 0.0398, 2.11e-7, 4.12},
                               {12.0, 0.00245, 0.246, 0.0664, 2.05e-7, 3.50}};
    const Fit &f = fit[math];
    const uint64_t units = resident > 1 ? resident / 2 : 1, n = (blocks + units - 1) / units;
    const double rounds = (n & 1) && n > 1 ? (double)(n - 1) + 1.2 : (double)n;
    return f.start + rounds * (double)((o.k_per_split + 15) / 16) * (f.row * o.mt + f.tile + (padded ? f.check : 0.)) +
           (o.splits > 1 ? f.byte * 2. * o.splits * plane : 0.) + (o.splits >= 16 ? f.many : 0.);
}

// Fills Wp, bands, dividers; chooses the unit, the row tile and the number of K slices.
bool band_plan(BandGeom &g, uint32_t M, uint32_t N, uint32_t groups, const SplitPlan &other, int math, uint32_t *splits)
{
    g.nsl = 0;
    const int KK = g.KH * g.KW;
    // (below nine channels more than half of a block's 16 would be padding; up to 32 rows more than half of its rows)
    if (math < 0 || math > 2 || KK < 5 || g.s <= 0 || g.Cg < 9 || g.N <= 0 || M < 33) return false;
    if (g.x_elems * 4 > kMaxBufferBytes || g.dy_elems * 4 > kMaxBufferBytes) return false;
    g.Wp = (g.OW - 1) * g.s + g.KW;
    // Row tile: the least padding, the taller one where equal.  Padded slots a unit may fill: 512 beside 128
    // rows, 256 beside the others (192 rows: the raw values of 512 slots in flight would spill, those of 256 spill 9; 64 rows: a block's
    // steps are short, and so should be the wait for its patch).  256 images of 13x13, us with 512 / 256:
    // 384 rows x 256 channels in tiles of 192 435 / 415, of 128 421 / 442; 192 rows in one tile 362 / 326.
    g.mt = M <= 64 ? 64 : (M + 191) / 192 * 192 <= (M + 127) / 128 * 128 ? 192 : 128;
    int ss = 0, p8 = 0;
    for (int slots = g.mt == 128 ? 512 : 256;; slots = 512) {
        if (slots == 512 && g.mt == 192) g.mt = 128;
        // as many output rows as the slots hold, evenly over the image; several images if they fit
        const int max_prow = slots / g.Wp, max_rows = (max_prow - g.KH) / g.s + 1;
        g.steps = 0;
        if (max_prow >= g.KH) {
            g.nb = (g.OH + max_rows - 1) / max_rows;
            g.Rb = (g.OH + g.nb - 1) / g.nb;
            g.nb = (g.OH + g.Rb - 1) / g.Rb;
            ss = ((g.Rb - 1) * g.s + g.KH) * g.Wp;
            g.ipu = g.nb > 1 ? 1 : slots / ss;
            if (g.ipu > g.N) g.ipu = g.N;
            p8 = (g.Rb * g.OW + 7) / 8;
            g.steps = (g.ipu * p8 + 3) / 4;
        }
        // a unit's patch has to be worth bringing: at least three steps
        if (g.steps >= 3) break;
        if (slots == 512) return false;
    }
    g.units = (g.N + g.ipu - 1) / g.ipu * g.nb;
    g.tap_blocks = (KK + TT - 1) / TT;
    // K slices: one round of two blocks a compute unit, whole units each (768 and 1024 blocks were slower)
    const uint64_t tiles = (uint64_t)((M + g.mt - 1) / g.mt) * ((g.Cg + 15) / 16) * g.tap_blocks * groups;
    const uint64_t resident = igemm_resident_blocks();
    uint64_t want = resident / tiles;
    if (want * 4 < (uint64_t)other.splits * 3) want = other.splits;      // no slice much longer than the gathered kernel's
    if (want > (uint64_t)g.units) want = (uint64_t)g.units;
    if (want < 1) want = 1;
    g.units_per_split = (int32_t)(((uint64_t)g.units + want - 1) / want);
    *splits = (uint32_t)(((uint64_t)g.units + g.units_per_split - 1) / g.units_per_split);
    // enough blocks to fill the chip, or the gathered kernel cuts K finer
    if (tiles * *splits * 2 < resident) return false;
    if ((uint64_t)*splits * groups * M * N >= (1ull << 31)) return false;
    const int chunks = g.ipu * ss <= 256 ? 4 : 8;
    const double plane = 4. * groups * M * N;
    const uint64_t other_blocks = (uint64_t)((M + other.mt - 1) / other.mt) * ((N + 127) / 128) * groups * other.splits;
    if (band_cost(g, chunks, plane, tiles * *splits, *splits, resident, math) >=
        0.97 * gathered_cost(other, other_blocks, plane, g.pad_h || g.pad_w, resident, math))
        return false;
    g.divSS = make_fastdiv((uint32_t)ss);
    g.divWp = make_fastdiv((uint32_t)g.Wp);
    g.divP8 = make_fastdiv((uint32_t)p8);
    g.divOW = make_fastdiv((uint32_t)g.OW);
    g.divKW = make_fastdiv((uint32_t)g.KW);
    g.divNB = make_fastdiv((uint32_t)g.nb);
    g.nsl = chunks;
    return true;
}
#endif  // CG_NP == 3

}  // namespace cg
