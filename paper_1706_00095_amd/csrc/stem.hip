// Forward convolutions of few input channels (a net's first layer) on the bf16 matrix instructions, fp32 operands in
// three pieces (split_device.h).
//
// What bounds it: the rows, the products and the stores of a block, one after the other, which two blocks a compute unit hide in
// part; the matrix pipe executes 47 % of the time a unit has work (256 images 3x227x227 -> 96, 11x11 stride 4, one run: 440 us,
// without 12 of the 13 steps of products 240, without the rows 369, without the stores 343, without products and rows 130).

//
// The gathered kernel loads every value of a window by an instruction of its own, 121 times a pixel and channel here, and
// the patch kernel wants 16 channels.  So a block keeps the source rows of a rectangle of at most 128 pixels in LDS, cut into
// pieces once, and a reduction index is a column of the window: four neighbouring columns of a window row (a quad; 11
// columns are three quads with one zero) are eight bytes of a row, so a lane's eight indices are two reads.  They have to start
// on eight bytes, hence a copy of the rows shifted by two columns for strides that are even, three more for odd ones.  The
// filters are cut by a small kernel beforehand (a net: with the other filter copies) into the order in which a wave's lanes
// load them, 1 KB at a time: read from the filter matrix itself, 16 rows apart, they took longer than the products.
// Waves share the rows of the block and its pixels, so that a fragment serves three row tiles or four pixel tiles.
// B = 32 3x224x224 -> 64, 7x7 stride 2: 115 -> 72 us; error against 64 bits 4.7e-8 where the fp32 instruction has 1.6e-7.
// Tried: eight waves a block (0.95 - 1.05), three blocks a compute unit (spills), 18 rows in flight (0.95); backward-weight the
// same way through transposed reads (7x7 stride 2 175 -> 117 us, 11x11 538 -> 860: 26 column tiles of accumulators spill).
#include <atomic>
#include <cstdio>
#include "cg_internal.h"
#include "igemm_device.h"
#include "split_device.h"

namespace cg {

namespace {

constexpr int PX = 128;                      // pixels of a tile, at most
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// a tile of pixels and its place
struct Tile { int n, ty0, tx0; };
__device__ __forceinline__ Tile tile_of(const StemGeom &g, uint32_t u)
{
    const uint32_t n = fdiv(u, g.divTpi), ti = u - n * g.divTpi.d, ry = fdiv(ti, g.divTx);
    return Tile{(int)n, (int)ry * g.Th, (int)(ti - ry * g.divTx.d) * g.Tw};
}

// Offset in a piece's plane, in values, of the window of pixel (py, px) of a tile: whole multiples of four values
// (8 bytes) from the start of the copy that is shifted by what is left.
__device__ __forceinline__ int window_at(const StemGeom &g, int py, int px)
{
    const int x = px * g.s, a = g.copies == 1 ? 0 : g.copies == 2 ? x & 2 : x & 3;
    return (g.copies == 2 ? a >> 1 : a) * g.copy_values + py * g.s * g.Wp + (x - a);
}

// Brings the source rows of a tile, cut into pieces, as [piece][copy][channel][row][column]: copy a holds the columns
// from a on.  A thread keeps its two columns and goes down the rows of a channel (and once more, one column on, where
// there are four copies), U of them in flight; what differs from one row to the next is uniform.
__device__ __forceinline__ void bring_rows(const StemGeom &g, __amdgpu_buffer_rsrc_t rX, const Tile &t, char *planes)
{
    const uint32_t half = g.divHalf.d, r0 = fdiv(threadIdx.x, g.divHalf), k = threadIdx.x - r0 * half;
    const int step = 256 / (int)half, y0 = t.ty0 * g.s - g.pad_h + (int)r0, row_bytes = g.W * 4;
    const int again = ((g.copies == 4 ? 2 : 1) * g.copy_values - 2) * 2;       // the copy shifted by two more holds a pair two values earlier
    const bool twice = g.copies > 1 && k > 0;
    constexpr int U = 3;
    if ((int)r0 >= step) return;
    for (int f = 0; f < (g.copies == 4 ? 2 : 1); ++f) {
        const int x = t.tx0 * g.s - g.pad_w + (int)(2 * k) + f;
        const bool in0 = (uint32_t)x < (uint32_t)g.W, in1 = (uint32_t)(x + 1) < (uint32_t)g.W;
        // (rows above the plane are below zero here, and nothing is loaded for them)
        const uint32_t lane0 = (uint32_t)(y0 * g.W + x) * 4u;
        for (int c = 0; c < g.Cg; ++c) {
            const uint32_t plane = (uint32_t)((t.n * g.C + c) * g.H * g.W) * 4u;
            char *const to0 = planes + (f * g.copy_values + (c * g.Rr + (int)r0) * g.Wp + (int)(2 * k)) * 2;
            for (int r = 0; r + (int)r0 < g.Rr; r += step * U) {
                float v[U][2];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int dr = r + u * step;
                    const bool ok = (uint32_t)(y0 + dr) < (uint32_t)g.H && (int)r0 + dr < g.Rr;
                    const uint32_t at = plane + lane0 + (uint32_t)(dr * row_bytes);
                    v[u][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rX, ok && in0 ? at : OOB_ROW, 0, 0));
                    v[u][1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rX, ok && in1 ? at + 4u : OOB_ROW, 0, 0));
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int dr = r + u * step;
                    if ((int)r0 + dr >= g.Rr) continue;
                    uint32_t pc[3];
                    split_pair<3>(v[u][0], v[u][1], pc);
                    char *const to = to0 + dr * g.Wp * 2;
#pragma unroll
                    for (int p = 0; p < 3; ++p) {
                        *reinterpret_cast<uint32_t *>(to + p * g.plane_values * 2) = pc[p];
                        if (twice) *reinterpret_cast<uint32_t *>(to + p * g.plane_values * 2 + again) = pc[p];
                    }
                }
            }
        }
    }
}

__device__ __forceinline__ float ldw(__amdgpu_buffer_rsrc_t r, uint32_t off) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0)); }

// Quads of four columns of the window: quad t is columns 4j .. 4j+3 of row t / quads of (channel, window row).  Byte offset of its
// first value from a pixel's window (0 behind the last quad, where the filters are zeros).
__device__ __forceinline__ uint32_t quad_at(const StemGeom &g, uint32_t t)
{
    const uint32_t row = fdiv(t, g.divQuads), j = t - row * g.divQuads.d, c = fdiv(row, g.divKH), ky = row - c * g.divKH.d;
    return t < (uint32_t)g.nquads ? (uint32_t)((((int)c * g.Rr + (int)ky) * g.Wp + 4 * (int)j) * 2) : 0u;
}

}  // namespace

struct StemArgs {
    IgemmProblem p;
    StemGeom g;
};

// Forward: a block is WM x (4 / WM) waves, 16 * TM * WM rows and one tile of pixels.
template <int TM, int WM>
__global__ __launch_bounds__(256, 2) void stem_fwd_kernel(const StemArgs args)
{
    constexpr int WN = 4 / WM, TN = PX / (16 * WN), MT = 16 * TM * WM;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const IgemmProblem &p = args.p;
    const StemGeom &g = args.g;
    const int lane = threadIdx.x & 63, q = lane >> 4, l16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const uint32_t m0 = blockIdx.y * MT, gr = blockIdx.z;
    const Tile t = tile_of(g, blockIdx.x);
    const int ns = (g.nquads + 7) / 8;

    const auto rA = buffer_of(p.A.ptr + (int64_t)gr * p.A.gstride, (p.A.elems - (uint64_t)gr * p.A.gstride) * 4);
    const auto rX = buffer_of(g.x + (int64_t)gr * g.Cg * g.H * g.W, (g.x_elems - (uint64_t)gr * g.Cg * g.H * g.W) * 4);
    const auto rF = buffer_of(g.copy + (uint64_t)gr * (g.copy_floats / p.groups), (g.copy_floats / p.groups) * 4);

    // the quads, eight a step, a lane's two of a step one 8-byte read
    uint32_t *const tab = reinterpret_cast<uint32_t *>(smem);
    for (uint32_t i = threadIdx.x; i < (uint32_t)ns * 8u; i += 256u) tab[i] = quad_at(g, i);
    char *const planes = smem + g.table_bytes;
    uint32_t arow[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t row = m0 + (uint32_t)((wm * TM + i) * 16 + l16);
        arow[i] = row < p.M ? row * p.K * 4u : OOB_ROW;
    }
    bring_rows(g, rX, t, planes);
    uint32_t win[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const uint32_t i = (uint32_t)((wn * TN + j) * 16 + l16), py = fdiv(i, g.divTw), px = i - py * g.divTw.d;
        win[j] = py < (uint32_t)g.Th ? (uint32_t)window_at(g, (int)py, (int)px) * 2u : 0u;
    }
    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    block_sync_lds();

    // rows of filters in pieces, as a lane multiplies with them (stem_filters_word), one step ahead
    v4u an[TM][3], ap[TM][3];
    v2u e{}, en{};
    auto load_a = [&](int s) {
        en = *reinterpret_cast<const v2u *>(tab + min(s, ns - 1) * 8 + 2 * q);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t tile = m0 / 16u + (uint32_t)(wm * TM + i), at = tile * 16u < p.M ? (tile * (uint32_t)ns + (uint32_t)min(s, ns - 1)) * 3072u + (uint32_t)lane * 16u : OOB_ROW;
#pragma unroll
            for (int k = 0; k < 3; ++k) an[i][k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rF, at + 1024u * k, 0, 0));
        }
    };
    load_a(0);
    using Step = MmaStep<3, TM, TN, TM >= 3 ? 1 : TN >= 4 && TM == 1 ? 4 : 2>;
    for (int s = 0; s < ns; ++s) {
        e = en;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) ap[i][k] = an[i][k];
        load_a(s + 1);
        const uint32_t b0 = e.x, b1 = e.y;
        auto read_b = [&](int j, v4u (&pc)[3]) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const v2u lo = *reinterpret_cast<const v2u *>(planes + win[j] + b0 + (uint32_t)(k * g.plane_values) * 2u);
                const v2u hi = *reinterpret_cast<const v2u *>(planes + win[j] + b1 + (uint32_t)(k * g.plane_values) * 2u);
                pc[k] = v4u{lo.x, lo.y, hi.x, hi.y};
            }
        };
        Step::run(ap, acc, read_b, typename Step::NoWork{});
    }
    struct Pixel { int oy, ox; bool ok; };
    auto pixel = [&](int i) {
        const uint32_t py = fdiv((uint32_t)i, g.divTw), px = (uint32_t)i - py * g.divTw.d;
        const int oy = t.ty0 + (int)py, ox = t.tx0 + (int)px;
        return Pixel{oy, ox, (int)py < g.Th && oy < g.OH && ox < g.OW};
    };
    if (not_finite(acc)) sums_in_fp32(acc, [&](int j, auto &&add) {
        const Pixel px = pixel((wn * TN + j) * 16 + l16);
        for (uint32_t k0 = 0; k0 < p.K; k0 += 16u) {
            float a[4][TM], b[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t k = k0 + (uint32_t)(4 * v + q), row = fdiv(k, g.divKW), kx = k - row * g.divKW.d, c = fdiv(row, g.divKH), ky = row - c * g.divKH.d;
                const int y = px.oy * g.s - g.pad_h + (int)ky, x = px.ox * g.s - g.pad_w + (int)kx;
                const bool ok = k < p.K && px.ok && (uint32_t)y < (uint32_t)g.H && (uint32_t)x < (uint32_t)g.W;
                b[v] = ldw(rX, ok ? (uint32_t)(((t.n * g.C + (int)c) * g.H + y) * g.W + x) * 4u : OOB_ROW);
#pragma unroll
                for (int i = 0; i < TM; ++i) a[v][i] = ldw(rA, arow[i] + (k < p.K ? k * 4u : OOB_K));
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) add(a[v], b[v]);
        }
    });
    store_columns_at<TM, TN, false>(p, acc, gr, 0u, m0 + (uint32_t)(wm * TM * 16), lane, [&](int c) {
        const Pixel px = pixel(wn * TN * 16 + c);
        return Columns{(uint32_t)((t.n * g.OH + px.oy) * g.OW + px.ox), px.ok ? (uint32_t)min(4, min(g.OW - px.ox, g.Tw - (px.ox - t.tx0))) : 0u};
    });
}

namespace {

template <class Kernel> int raise_lds(Kernel *k, std::atomic<bool> &done)
{
    if (done.load(std::memory_order_acquire)) return CG_OK;
    CG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kStemLds));
    done.store(true, std::memory_order_release);
    return CG_OK;
}

template <int TM, int WM> int launch_fwd(const StemArgs &a, hipStream_t stream)
{
    constexpr int MT = 16 * TM * WM;
    const IgemmProblem &p = a.p;
    dim3 grid((unsigned)a.g.units, (p.M + MT - 1) / MT, p.groups);
    if (grid.y > 65535u || grid.z > 65535u) return CG_EUNSUPPORTED;
    static std::atomic<bool> done{false};
    const int rc = raise_lds(&stem_fwd_kernel<TM, WM>, done);
    if (rc) return rc;
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, "igemm_stem_kernel<%d>", MT);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    hipLaunchKernelGGL((stem_fwd_kernel<TM, WM>), grid, dim3(256), (size_t)a.g.lds_bytes, stream, a);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

// the fewest tiles of at most 128 pixels whose rows fit
bool choose_tile(StemGeom &g)
{
    const int quads = (g.KW + 3) / 4;
    g.copies = g.s % 4 == 0 ? 1 : g.s % 2 == 0 ? 2 : 4;
    int64_t best = 0;
    for (int w = 4; w < g.OW + 4 && w <= PX; w += 4) {
        const int h = PX / w < g.OH ? PX / w : g.OH;
        const int Rr = (h - 1) * g.s + g.KH, Wp = ((w - 1) * g.s + 4 * quads + 3) / 4 * 4;
        const int64_t bytes = (int64_t)g.table_bytes + 6ll * g.copies * g.Cg * Rr * Wp;
        if (bytes > kStemLds || Wp > 512) continue;
        const int64_t tx = (g.OW + w - 1) / w, tiles = tx * ((g.OH + h - 1) / h), cost = tiles * (1000 + bytes / 256);     // fewer tiles, then smaller ones
        if (best && cost >= best) continue;
        best = cost;
        g.Tw = w; g.Th = h; g.Rr = Rr; g.Wp = Wp; g.lds_bytes = (int32_t)bytes;
        g.divTx = make_fastdiv((uint32_t)tx);
        g.divTpi = make_fastdiv((uint32_t)tiles);
        g.units = (int32_t)tiles;
    }
    if (!best || (int64_t)g.units * g.N >= (1 << 30)) return false;
    g.units *= g.N;
    g.copy_values = g.Cg * g.Rr * g.Wp;
    g.plane_values = g.copies * g.copy_values;
    g.divTw = make_fastdiv((uint32_t)g.Tw);
    g.divHalf = make_fastdiv((uint32_t)(g.Wp / 2));
    g.divKH = make_fastdiv((uint32_t)g.KH);
    g.divKW = make_fastdiv((uint32_t)g.KW);
    g.divQuads = make_fastdiv((uint32_t)quads);
    g.nquads = g.Cg * g.KH * quads;
    return true;
}

int fwd_rows(uint32_t M) { return M <= 16 ? 16 : M <= 32 ? 32 : M <= 48 ? 48 : M <= 64 ? 64 : M <= 96 ? 96 : (M + 127) / 128 * 128 <= (M + 95) / 96 * 96 ? 128 : 96; }

}  // namespace

// Expected times, us, from 200 problems (1 to 8 channels, windows 1x3 to 11x11, strides 1, 2 and 4, planes of 64 to 227
// pixels a side, up to 80 GFLOP): one standard deviation of the relative error is 22 % here and 28 % for the gathered
// kernel.  A block here sets up, brings its rows and multiplies whole steps of 32 indices (15 % more than there are in an
// 11x11 window of 3 channels) for mt rows.  Chosen by these (below 0.85 of the other) 52 of them became faster by
// 33 % in the mean, three slower than 0.97 (0.75 at worst).
bool stem_fwd_plan(StemGeom &g, uint32_t M, uint32_t N, uint32_t groups, const SplitPlan &other)
{
    const int quads = (g.KW + 3) / 4, taps = g.Cg * g.KH * g.KW, ns = (g.Cg * g.KH * quads + 7) / 8;
    if (g.Cg > 8 || g.KH * g.KW < 2 || g.x_elems * 4 > kMaxBufferBytes || taps >= (1 << 12)) return false;
    g.table_bytes = (ns * 32 + 15) / 16 * 16;
    if (!choose_tile(g)) return false;
    g.mt = fwd_rows(M);
    const double resident = igemm_resident_blocks(), row_blocks = (double)((M + g.mt - 1) / g.mt) * groups;
    const double rounds = g.units * row_blocks / resident, brought = 1e-3 * g.Cg * g.Rr * g.Wp * (g.copies == 4 ? 2 : 1);
    const double here = 10. + (rounds > 1. ? rounds : 1.) * (1.35 + 0.644 * brought + (1.64 * ns + 1.36) * g.mt / 96.);
    const double blocks = (double)((M + other.mt - 1) / other.mt) * ((N + 127) / 128) * groups * other.splits, turns = blocks * 2. / resident;
    const double there = 8.4 + (double)(uint64_t)(turns + 0.999) * ((other.k_per_split + 15) / 16) * (0.00942 * other.mt + 0.123 + (g.pad_h || g.pad_w ? 0.139 : 0.));
    if (here >= 0.85 * there) return false;
    g.copy_floats = stem_copy_floats((int)M, g.Cg, g.KH, g.KW) * groups;
    return g.copy_floats * 4 <= kMaxBufferBytes;
}

uint64_t stem_copy_floats(int Mg, int Cg, int KH, int KW)
{
    return (uint64_t)((Mg + 15) / 16) * (uint64_t)((Cg * KH * ((KW + 3) / 4) + 7) / 8) * 768u;
}

int stem_fwd_launch(const IgemmProblem &p, const StemGeom &g, hipStream_t stream)
{
    if (!p.c_ptr || !aligned16(p.c_ptr) || !p.A.ptr || !aligned16(p.A.ptr) || !g.x || !aligned16(g.x) || !g.copy || !aligned16(g.copy) || (p.bias_mode && !p.bias) || p.math != CG_MATH_FP32) return CG_EINVAL;
    const StemArgs a{p, g};
    switch (g.mt) {
    case 16: return launch_fwd<1, 1>(a, stream);
    case 32: return launch_fwd<1, 2>(a, stream);
    case 48: return launch_fwd<3, 1>(a, stream);
    case 64: return launch_fwd<2, 2>(a, stream);
    case 96: return launch_fwd<3, 2>(a, stream);
    default: return launch_fwd<2, 4>(a, stream);
    }
}

}  // namespace cg
