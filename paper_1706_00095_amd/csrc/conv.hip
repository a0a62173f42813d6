// Convolution and fully-connected passes expressed as implicit-GEMM problems.
//
// Forward:          Y[m][(n,oh,ow)]   = sum_{(c,kh,kw)} W[m][(c,kh,kw)] * X(n,c,oh*s-p+kh,ow*s-p+kw)
// Backward-data:    dX[c][(n,ih,iw)]  = sum_{(m,kh,kw)} Wt[c][(m,kh,kw)] * dY(n,m,(ih+p-kh)/s,(iw+p-kw)/s)
// Backward-weight:  dW[m][(c,kh,kw)]  = sum_{(n,oh,ow)} dY[m][(n,oh,ow)] * X(n,c,oh*s-p+kh,ow*s-p+kw)
// (section 2.1: forward propagation, backward propagation, gradient on the weights; the last
// one is the first step of every turn in Fig. 3).
#include <algorithm>
#include <mutex>
#include "cg_internal.h"
#include "split_device.h"

namespace cg {

namespace {

size_t round256(size_t v) { return (v + 255) / 256 * 256; }
__host__ __device__ inline int padded16(int c) { return (c + 15) / 16 * 16; }

// input pixel grid seen through the filter: index (n, oh, ow) -> window origin in x
IndexMap window_origin_map(const cg_conv_desc &d, int OH, int OW)
{
    IndexMap m{};
    m.count = (uint32_t)d.N * OH * OW;
    m.d1 = make_fastdiv((uint32_t)OH * OW);
    m.d2 = make_fastdiv((uint32_t)OW);
    m.s1 = d.C * d.H * d.W;
    m.s2 = d.stride_h * d.W;
    m.s3 = d.stride_w;
    m.o0 = -d.pad_h * d.W - d.pad_w;
    m.sa = d.stride_h; m.a0 = -d.pad_h;
    m.sb = d.stride_w; m.b0 = -d.pad_w;
    return m;
}

// filter tap index (c, kh, kw) -> displacement inside x
IndexMap tap_map(const cg_conv_desc &d, int Cg)
{
    IndexMap m{};
    m.count = (uint32_t)Cg * d.KH * d.KW;
    m.d1 = make_fastdiv((uint32_t)d.KH * d.KW);
    m.d2 = make_fastdiv((uint32_t)d.KW);
    m.s1 = d.H * d.W;
    m.s2 = d.W;
    m.s3 = 1;
    m.sa = 1; m.sb = 1;
    return m;
}

// wt[g][c][ml][kh][kw] = w[g*Mg + ml][c][kh][kw]: the filters as the row-major matrix that
// backward-data multiplies with (rows = input channels, reduction index = (ml, kh, kw))
__device__ __forceinline__ float transpose_filters_elem(const float *__restrict__ w, size_t i, int Mg, int Cg, int KK)
{
    const int kk = (int)(i % KK);
    size_t r = i / KK;
    const int ml = (int)(r % Mg); r /= Mg;
    const int c = (int)(r % Cg);
    const int g = (int)(r / Cg);
    return w[(((size_t)g * Mg + ml) * Cg + c) * KK + kk];
}

// Filters in three bf16 pieces, as a lane of stem_fwd_kernel multiplies with them: word i of
// dst[g][row / 16][step][piece][lane][4], two bf16 a word: lane (q, l) of a step holds row l's quads 8 * step + 2q and + 1, quad
// t being columns 4j .. 4j+3 of window row t / quads of (channel, ky); zeros where there is no column, quad or row.
__device__ __forceinline__ float stem_filters_word(const float *__restrict__ w, size_t i, int Mg, int Cg, int KH, int KW)
{
    const int Q = (KW + 3) / 4, nq = Cg * KH * Q, ns = (nq + 7) / 8, RT = (Mg + 15) / 16;
    const int word = (int)(i % 4), lane = (int)(i / 4 % 64), piece = (int)(i / 256 % 3);
    size_t u = i / 768;
    const int s = (int)(u % ns); u /= ns;
    const int rt = (int)(u % RT), g = (int)(u / RT), r = rt * 16 + lane % 16, t = 8 * s + 2 * (lane / 16) + word / 2, kx = 4 * (t % Q) + 2 * (word % 2);
    const float *row = w + (((size_t)g * Mg + r) * Cg * KH + t / Q) * KW + kx;
    const bool ok = r < Mg && t < nq;
    uint32_t pc[3];
    split_pair<3>(ok && kx < KW ? row[0] : 0.f, ok && kx + 1 < KW ? row[1] : 0.f, pc);
    return __uint_as_float(piece == 0 ? pc[0] : piece == 1 ? pc[1] : pc[2]);
}

__global__ __launch_bounds__(256) void stem_filters_kernel(const float *__restrict__ w, float *__restrict__ dst, size_t total, int Mg, int Cg, int KH, int KW)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256)
        dst[i] = stem_filters_word(w, i, Mg, Cg, KH, KW);
}

__global__ __launch_bounds__(256) void transpose_filters_kernel(const float *__restrict__ w, float *__restrict__ wt,
                                                                int G, int Mg, int Cg, int KK)
{
    const size_t total = (size_t)G * Mg * Cg * KK;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256)
        wt[i] = transpose_filters_elem(w, i, Mg, Cg, KK);
}

// The rearranged filters of several layers in one launch (a net prepares those of all its layers at
// the start of an iteration): block b belongs to the job whose [first_block, ...) range holds it and
// writes 256 * PER consecutive elements of that job's copy (pairs, where the copy holds pieces).  A thread's elements follow one
// another, index divisions and load and store, so that small copies, of a single layer mostly, take one a thread:
// two images of 77x62, 3 -> 215 channels 7x7 stride 2, backward-data with four 26.2 us, with one 24.0; 142x142, 3 -> 52
// channels 7x7 stride 4, bf16x3, 22.3 / 20.3.
constexpr int kPrepJobs = 8;
constexpr unsigned long long kPrepOneEach = 1u << 20;       // 4096 blocks, two rounds of the chip
struct PrepJob {
    const float *w;
    float *dst;
    int kind, Mg, Cg, KH, KW, sh, sw, Ah, Aw, pieces;
    unsigned first_block;
    unsigned long long total;          // what the threads write: elements of the copy, or pairs of values in pieces
};
struct PrepTable {
    PrepJob j[kPrepJobs];
    int n;
};

__device__ __forceinline__ uint32_t prep_rows(const PrepJob &f)
{
    return (uint32_t)(f.kind == CG_PREP_PERMUTE_FWD ? f.Mg : f.kind == CG_PREP_PERMUTE_BWD ? f.Cg : f.Cg * f.sh * f.sw);
}

// Filters as the patch kernel multiplies with them: dst[g][t][c / 16][r][c % 16], t a tap (units of 16 reduction indices, all
// rows of a unit contiguous: a wave's load is).  c runs over the next multiple of 16, zeros behind the last channel.
// Forward: r = output channel, c = input channel, t = kh*KW + kw: dst = w[g*Mg + r][c][t].
// Backward-data: r = input channel, c = output channel: dst = w[g*Mg + c][r][t].
// Strided backward-data (see bwd_data_strided_problem): r = (input channel, rh, rw), c = output channel, t = a*Aw + b, with filter
// tap kh = rh + sh*a, kw = rw + sw*b (zero where that tap does not exist).
__device__ __forceinline__ float tap_major_value(const PrepJob &f, uint32_t unit, uint32_t r, uint32_t k)
{
    const bool fwd = f.kind == CG_PREP_PERMUTE_FWD, strided = f.kind == CG_PREP_STRIDED_TAPS;
    const uint32_t Cr = (uint32_t)(fwd ? f.Cg : f.Mg), U = (Cr + 15) / 16, T = (uint32_t)(strided ? f.Ah * f.Aw : f.KH * f.KW);
    const uint32_t gt = unit / U, c = (unit - gt * U) * 16 + k, g = gt / T, t = gt - g * T;
    uint32_t ci = fwd ? c : r, tap = t;
    bool ok = c < Cr;
    if (strided) {
        const uint32_t q = r / (uint32_t)f.sw, a = t / (uint32_t)f.Aw, kh = q % (uint32_t)f.sh + (uint32_t)f.sh * a,
                       kw = r - q * (uint32_t)f.sw + (uint32_t)f.sw * (t - a * (uint32_t)f.Aw);
        ci = q / (uint32_t)f.sh;
        tap = kh * (uint32_t)f.KW + kw;
        ok = ok && kh < (uint32_t)f.KH && kw < (uint32_t)f.KW;
    }
    return ok ? f.w[(((size_t)g * f.Mg + (fwd ? r : c)) * f.Cg + ci) * (size_t)(f.KH * f.KW) + tap] : 0.f;
}

// The same as the pieces they are multiplied in: dst[g][t][c / 16][piece][r][c % 16], bf16.  Pair i of values, all its pieces.
template <int NP> __device__ __forceinline__ void cut_tap_major_pair(const PrepJob &f, uint32_t i)
{
    const uint32_t R = prep_rows(f), j = i % 8, q = i / 8, unit = q / R, r = q - unit * R;
    uint32_t pc[NP], *dst = reinterpret_cast<uint32_t *>(f.dst) + ((size_t)unit * NP * R + r) * 8 + j;
    split_pair<NP>(tap_major_value(f, unit, r, 2 * j), tap_major_value(f, unit, r, 2 * j + 1), pc);
#pragma unroll
    for (int k = 0; k < NP; ++k) dst[(size_t)k * R * 8] = pc[k];
}

// Filters as the gathered kernel's matrix of strided backward-data: dst[g][r][c][t], as above.
__device__ __forceinline__ float strided_rows_value(const PrepJob &f, uint32_t i)
{
    const uint32_t T = (uint32_t)(f.Ah * f.Aw), R = prep_rows(f);
    const uint32_t q = i / T, t = i - q * T, u = q / (uint32_t)f.Mg, m = q - u * (uint32_t)f.Mg, g = u / R, r = u - g * R;
    const uint32_t v = r / (uint32_t)f.sw, kh = v % (uint32_t)f.sh + (uint32_t)f.sh * (t / (uint32_t)f.Aw), kw = r % (uint32_t)f.sw + (uint32_t)f.sw * (t % (uint32_t)f.Aw);
    return kh < (uint32_t)f.KH && kw < (uint32_t)f.KW
               ? f.w[(((size_t)g * f.Mg + m) * f.Cg + v / (uint32_t)f.sh) * (size_t)(f.KH * f.KW) + kh * (uint32_t)f.KW + kw] : 0.f;
}

template <int PER> __global__ __launch_bounds__(256) void prepare_filters_kernel(const PrepTable t)
{
    int ji = 0;
#pragma unroll
    for (int k = 1; k < kPrepJobs; ++k)
        if (k < t.n && blockIdx.x >= t.j[k].first_block) ji = k;
    const PrepJob &jb = t.j[ji];
    const size_t base = (size_t)(blockIdx.x - jb.first_block) * (256 * PER) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const size_t i = base + (size_t)u * 256;
        if (i >= jb.total) break;
        if (jb.pieces == 3) { cut_tap_major_pair<3>(jb, (uint32_t)i); continue; }
        if (jb.pieces == 2) { cut_tap_major_pair<2>(jb, (uint32_t)i); continue; }
        if (jb.pieces == 1) { cut_tap_major_pair<1>(jb, (uint32_t)i); continue; }
        float v;
        if (jb.kind == CG_PREP_TRANSPOSE) v = transpose_filters_elem(jb.w, i, jb.Mg, jb.Cg, jb.KH * jb.KW);
        else if (jb.kind == CG_PREP_PIECES) v = stem_filters_word(jb.w, i, jb.Mg, jb.Cg, jb.KH, jb.KW);
        else if (jb.kind == CG_PREP_STRIDED_ROWS) v = strided_rows_value(jb, (uint32_t)i);
        else {
            const uint32_t R = prep_rows(jb), q = (uint32_t)i / 16, unit = q / R;
            v = tap_major_value(jb, unit, q - unit * R, (uint32_t)i % 16);
        }
        jb.dst[i] = v;
    }
}

// General-stride backward-data, gather form, one thread per dx element: the taps of the element's stride phase, four output
// channels at a time.  dy reads as zero outside its plane, as everywhere.
struct GatherArgs {
    cg_conv_desc d;
    int OH, OW;
    const float *dy, *w, *gate;
    float *dx;
    int accumulate;
    FastDiv divW, divH, divC, divCg, divSh, divSw;
};

__global__ __launch_bounds__(256) void bwd_data_strided_kernel(const GatherArgs a)
{
    const cg_conv_desc &d = a.d;
    const int Cg = d.C / d.groups, Mg = d.M / d.groups, KK = d.KH * d.KW, P = a.OH * a.OW;
    const uint32_t total = (uint32_t)d.N * d.C * d.H * d.W;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        const uint32_t q = fdiv(i, a.divW), r = fdiv(q, a.divH), n = fdiv(r, a.divC), c = r - n * d.C, g = fdiv(c, a.divCg);
        const uint32_t y = q - r * d.H + d.pad_h, x = i - q * d.W + d.pad_w;
        const int oh0 = (int)fdiv(y, a.divSh), ow0 = (int)fdiv(x, a.divSw), kh0 = (int)y - oh0 * d.stride_h, kw0 = (int)x - ow0 * d.stride_w;
        const float *yp = a.dy + (size_t)(n * d.M + g * Mg) * P, *wp = a.w + ((size_t)g * Mg * Cg + (c - g * Cg)) * KK;
        float s[4] = {};
        auto channels = [&](auto UC) {
            constexpr int U = decltype(UC)::value;
            for (int kh = kh0, oh = oh0; kh < d.KH; kh += d.stride_h, --oh)
                for (int kw = kw0, ow = ow0; kw < d.KW; kw += d.stride_w, --ow) {
                    const bool ok = (uint32_t)oh < (uint32_t)a.OH && (uint32_t)ow < (uint32_t)a.OW;
                    float v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = ok ? yp[u * P + oh * a.OW + ow] : 0.f;
#pragma unroll
                    for (int u = 0; u < U; ++u) s[u] = fmaf(v[u], wp[u * Cg * KK + kh * d.KW + kw], s[u]);
                }
            yp += U * P;
            wp += U * Cg * KK;
        };
        int m = 0;
        for (; m + 4 <= Mg; m += 4) channels(std::integral_constant<int, 4>{});
        for (; m < Mg; ++m) channels(std::integral_constant<int, 1>{});
        float out = (s[0] + s[1]) + (s[2] + s[3]);
        if (a.gate && !(a.gate[i] > 0.f)) out = 0.f;
        a.dx[i] = a.accumulate ? a.dx[i] + out : out;
    }
}

}  // namespace

int conv_check(const cg_conv_desc *d, int *OH, int *OW)
{
    if (!d) return CG_EINVAL;
    if (d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0 || d->M <= 0 || d->KH <= 0 || d->KW <= 0 ||
        d->stride_h <= 0 || d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0 || d->groups <= 0)
        return CG_EINVAL;
    if (d->C % d->groups || d->M % d->groups) return CG_EINVAL;
    const int eh = d->H + 2 * d->pad_h - d->KH, ew = d->W + 2 * d->pad_w - d->KW;
    if (eh < 0 || ew < 0) return CG_EINVAL;
    const int oh = eh / d->stride_h + 1, ow = ew / d->stride_w + 1;
    const uint64_t lim = (1ull << 31) / 4;   // elements per tensor
    if ((uint64_t)d->N * d->C * d->H * d->W >= lim || (uint64_t)d->N * d->M * oh * ow >= lim ||
        (uint64_t)d->M * (d->C / d->groups) * d->KH * d->KW >= lim)
        return CG_EUNSUPPORTED;
    if (d->KH > 4096 || d->KW > 4096 || d->H > (1 << 20) || d->W > (1 << 20)) return CG_EUNSUPPORTED;
    if (OH) *OH = oh;
    if (OW) *OW = ow;
    return CG_OK;
}

static IgemmProblem fwd_problem(const cg_conv_desc &d, int OH, int OW, const float *x, const float *w,
                                const float *bias, float *y, int64_t y_img_stride = 0)
{
    const int G = d.groups, Cg = d.C / G, Mg = d.M / G, Kg = Cg * d.KH * d.KW, P = OH * OW;
    IgemmProblem p{};
    p.A.ptr = w;
    p.A.row = linear_map(Mg, Kg);
    p.A.k = linear_map(Kg, 1);
    p.A.limA = p.A.limB = 1;
    p.A.gstride = (int64_t)Mg * Kg;
    p.A.elems = (uint64_t)d.M * Kg;
    p.A.lanes_k = 1;
    p.B.ptr = x;
    p.B.row = window_origin_map(d, OH, OW);
    p.B.k = tap_map(d, Cg);
    p.B.limA = d.H; p.B.limB = d.W;
    p.B.gstride = (int64_t)Cg * d.H * d.W;
    p.B.elems = (uint64_t)d.N * d.C * d.H * d.W;
    p.B.lanes_k = 0;
    p.B.check = (d.pad_h || d.pad_w) ? 1 : 0;
    p.c_ptr = y;
    p.c_row_stride = P;
    p.c_col = split_map((uint32_t)d.N * P, P, y_img_stride ? (int32_t)y_img_stride : d.M * P, 1);
    p.c_gstride = (int64_t)Mg * P;
    p.bias = bias; p.bias_mode = bias ? 1 : 0; p.bias_gstride = Mg;
    p.M = Mg; p.N = (uint32_t)d.N * P; p.K = Kg;
    p.groups = G; p.splits = 1; p.k_per_split = p.K;
    return p;
}

// Describes x as the patch operand of the forward pass; true if the patch kernel can run it.
static bool fwd_patch(const cg_conv_desc &d, int OH, int OW, const float *x, IgemmProblem &p)
{
    if (d.stride_h != d.stride_w) return false;
    const int G = d.groups, Cg = d.C / G;
    PatchGeom g{};
    g.src = x; g.src_elems = (uint64_t)d.N * d.C * d.H * d.W;
    g.gstride = (int64_t)Cg * d.H * d.W;
    g.Cred = (uint32_t)Cg; g.Hs = d.H; g.Ws = d.W; g.chan_stride = d.H * d.W; g.img_stride = d.C * d.H * d.W;
    g.OHo = OH; g.OWo = OW; g.s = d.stride_h; g.oy0 = -d.pad_h; g.ox0 = -d.pad_w; g.KH = d.KH; g.KW = d.KW; g.flip = 0;
    g.taps = g.tap_slots = 1;
    if (!patch_plan(g, (uint32_t)(d.M / G), (uint32_t)d.N * OH * OW, (uint32_t)G, p.math) || (g.Cred % 16 && igemm_in_pieces(p))) return false;
    p.patch = g; p.use_patch = 1;
    return true;
}

// Does the kernel for few input channels run the forward pass?  g: its geometry.
static bool fwd_stem(const cg_conv_desc &d, int OH, int OW, const float *x, const IgemmProblem &p, StemGeom &g)
{
    if (d.stride_h != d.stride_w || p.math != CG_MATH_FP32 || igemm_in_pieces(p)) return false;
    g = StemGeom{};
    g.x = x; g.x_elems = (uint64_t)d.N * d.C * d.H * d.W;
    g.N = d.N; g.C = d.C; g.Cg = d.C / d.groups; g.H = d.H; g.W = d.W; g.OH = OH; g.OW = OW; g.s = d.stride_h;
    g.pad_h = d.pad_h; g.pad_w = d.pad_w; g.KH = d.KH; g.KW = d.KW;
    return stem_fwd_plan(g, p.M, p.N, p.groups, gathered_plan(p.M, p.N, p.K, p.groups));
}

// Operand A of the patch kernel = the copy at m that `f` describes, made from w.
static void tap_major_filters(IgemmProblem &p, const FilterPrep &f, const float *m, const float *w)
{
    p.A = Operand{};
    p.A.ptr = m;
    p.A.gstride = (int64_t)(f.floats / p.groups);
    p.A.elems = f.floats;
    p.patch.filter_pieces = f.pieces;
    p.taps.w = w; p.taps.Mg = f.Mg; p.taps.Cg = f.Cg;
}

// Describes the copy of the filters that the patch kernel multiplies p with: `values` values.  In the reduced modes it always
// holds pieces: they take no more room than the values.  Three take half as much again, so a copy into a workspace holds
// them where the workspace has `room` bytes for them (a net's slots do), and where the kernel is the faster for it
// (patch_wants_pieces).
static void tap_major_copy(FilterPrep &f, uint64_t values, const IgemmProblem &p, size_t room)
{
    f.pieces = p.math == CG_MATH_BF16 ? 1 : p.math == CG_MATH_BF16X3 ? 2 : values * 6 <= kMaxBufferBytes && values * 6 <= room && patch_wants_pieces(p) ? 3 : 0;
    f.floats = f.pieces ? (size_t)values / 2 * f.pieces : (size_t)values;
}
constexpr size_t kSlotRoom = ~(size_t)0;

// bytes of the rearranged filters the patch kernel multiplies with
static size_t fwd_copy_bytes(const cg_conv_desc &d)
{
    return round256((size_t)d.M * padded16(d.C / d.groups) * d.KH * d.KW * sizeof(float));
}
static size_t bwd_copy_bytes(const cg_conv_desc &d)
{
    return round256((size_t)d.C * padded16(d.M / d.groups) * d.KH * d.KW * sizeof(float));
}

static FilterPrep fwd_patch_prep(const cg_conv_desc &d, const IgemmProblem &p, size_t room)
{
    FilterPrep f{};
    f.kind = CG_PREP_PERMUTE_FWD;
    f.Mg = d.M / d.groups; f.Cg = d.C / d.groups; f.KH = d.KH; f.KW = d.KW;
    tap_major_copy(f, (uint64_t)d.M * padded16(f.Cg) * d.KH * d.KW, p, room);
    return f;
}
static FilterPrep bwd_patch_prep(const cg_conv_desc &d, const IgemmProblem &p, size_t room)
{
    FilterPrep f{};
    f.kind = CG_PREP_PERMUTE_BWD;
    f.Mg = d.M / d.groups; f.Cg = d.C / d.groups; f.KH = d.KH; f.KW = d.KW;
    tap_major_copy(f, (uint64_t)d.C * padded16(f.Mg) * d.KH * d.KW, p, room);
    return f;
}

static bool math_ok(int math) { return math == CG_MATH_FP32 || math == CG_MATH_BF16 || math == CG_MATH_BF16X3; }

int conv_fwd_impl(const cg_conv_desc &d, const float *x, const float *w, const float *bias, float *y, void *ws,
                  size_t ws_bytes, int relu, hipStream_t stream, int64_t y_img_stride, int math, const float *prepared)
{
    if (!math_ok(math)) return CG_EINVAL;
    ProfTag tag("conv_fwd", -1);
    int OH, OW;
    const int rc = conv_check(&d, &OH, &OW);
    if (rc) return rc;
    // y_img_stride: elements between the images of y when y is a channel slice of a wider tensor
    // (0 = dense, M*OH*OW); the whole wider tensor must stay below 2^31 elements
    if (y_img_stride < 0 || (y_img_stride && (y_img_stride < (int64_t)d.M * OH * OW ||
                                              y_img_stride * (int64_t)d.N >= (1ll << 31)))) return CG_EINVAL;
    IgemmProblem p = fwd_problem(d, OH, OW, x, w, bias, y, y_img_stride);
    p.relu = relu;
    p.math = math;
    const size_t wt_bytes = fwd_copy_bytes(d);
    // (a copy with padded channels is dropped where the workspace has no room for it)
    const bool room = d.C / d.groups % 16 == 0 || (ws && ws_bytes >= wt_bytes), patch = room && fwd_patch(d, OH, OW, x, p);
    if (patch) {
        if (!ws || ws_bytes < wt_bytes) return CG_ENOSPC;
        if (!aligned16(ws)) return CG_EINVAL;
        const FilterPrep f = fwd_patch_prep(d, p, prepared ? kSlotRoom : ws_bytes);
        float *copy = static_cast<float *>(ws);
        if (!prepared) {
            const int rc2 = filter_prep_launch(1, &f, &w, &copy, stream);
            if (rc2) return rc2;
        }
        tap_major_filters(p, f, prepared ? prepared : copy, w);
        return igemm_run(p, nullptr, 0, stream);
    }
    StemGeom sg;
    if (fwd_stem(d, OH, OW, x, p, sg) && ws && ws_bytes >= sg.copy_floats * sizeof(float) && aligned16(ws)) {
        const int rs = igemm_scratch_check(p, ws, ws_bytes);
        if (rs) return rs;
        sg.copy = prepared ? prepared : static_cast<const float *>(ws);
        if (!prepared) {
            const unsigned blocks = (unsigned)((sg.copy_floats + 255) / 256 < 4096 ? (sg.copy_floats + 255) / 256 : 4096);
            hipLaunchKernelGGL(stem_filters_kernel, dim3(blocks), dim3(256), 0, stream, w, static_cast<float *>(ws), (size_t)sg.copy_floats, d.M / d.groups,
                               d.C / d.groups, d.KH, d.KW);
            CG_HIP_TRY(hipGetLastError());
        }
        return stem_fwd_launch(p, sg, stream);
    }
    return igemm_run(p, ws, ws_bytes, stream);
}

// A 1x1 window without padding at stride 1: backward-data is the plain product of the transposed
// filter matrix with dy, and the transposed matrix can be read from w with the loader that runs the
// row index along the lanes (as the fully-connected layers do), so no transposed copy is made.
static bool bwd_data_reads_filters_in_place(const cg_conv_desc &d)
{
    return d.KH == 1 && d.KW == 1 && d.pad_h == 0 && d.pad_w == 0 && d.stride_h == 1 && d.stride_w == 1;
}

static IgemmProblem bwd_data_problem(const cg_conv_desc &d, int OH, int OW, const float *dy, const float *wt,
                                     float *dx, int accumulate)
{
    const int G = d.groups, Cg = d.C / G, Mg = d.M / G, KK = d.KH * d.KW, P = OH * OW;
    const int Kp = Mg * KK;
    IgemmProblem p{};
    p.A.ptr = wt;
    p.A.row = linear_map(Cg, Kp);
    p.A.k = linear_map(Kp, 1);
    p.A.limA = p.A.limB = 1;
    p.A.gstride = (int64_t)Cg * Kp;
    p.A.elems = (uint64_t)d.M * Cg * KK;
    p.A.lanes_k = 1;
    if (bwd_data_reads_filters_in_place(d)) {
        // one tap: A(c, m) is w[m][c] itself, rows (input channels) along the lanes -- `wt` is then w
        p.A.row = linear_map(Cg, 1);
        p.A.k = linear_map(Mg, Cg);
        p.A.lanes_k = 0;
    }
    // dy seen from an input pixel (n, ih, iw): origin (ih + p, iw + p), taps subtract (kh, kw)
    p.B.ptr = dy;
    IndexMap pix{};
    pix.count = (uint32_t)d.N * d.H * d.W;
    pix.d1 = make_fastdiv((uint32_t)d.H * d.W);
    pix.d2 = make_fastdiv((uint32_t)d.W);
    pix.s1 = d.M * P; pix.s2 = OW; pix.s3 = 1; pix.o0 = d.pad_h * OW + d.pad_w;
    pix.sa = 1; pix.a0 = d.pad_h; pix.sb = 1; pix.b0 = d.pad_w;
    IndexMap tap{};
    tap.count = (uint32_t)Kp;
    tap.d1 = make_fastdiv((uint32_t)KK);
    tap.d2 = make_fastdiv((uint32_t)d.KW);
    tap.s1 = P; tap.s2 = -OW; tap.s3 = -1;
    tap.sa = -1; tap.sb = -1;
    p.B.row = pix; p.B.k = tap;
    p.B.limA = OH; p.B.limB = OW;
    p.B.gstride = (int64_t)Mg * P;
    p.B.elems = (uint64_t)d.N * d.M * P;
    p.B.lanes_k = 0;
    p.B.check = (KK > 1 || d.pad_h || d.pad_w) ? 1 : 0;
    const int HW = d.H * d.W;
    p.c_ptr = dx;
    p.c_row_stride = HW;
    p.c_col = split_map((uint32_t)d.N * HW, HW, d.C * HW, 1);
    p.c_gstride = (int64_t)Cg * HW;
    p.M = Cg; p.N = (uint32_t)d.N * HW; p.K = Kp;
    p.groups = G; p.splits = 1; p.k_per_split = p.K;
    p.accumulate = accumulate;
    return p;
}

// The same for direct_kernel, which reads the filters where they are: A(c, (m, kh, kw)) = w[m][c][kh][kw].
static IgemmProblem bwd_data_direct_problem(const cg_conv_desc &d, int OH, int OW, const float *dy, const float *w, float *dx, int accumulate)
{
    const int Cg = d.C / d.groups, Mg = d.M / d.groups, KK = d.KH * d.KW;
    IgemmProblem p = bwd_data_problem(d, OH, OW, dy, w, dx, accumulate);
    p.A.row = linear_map((uint32_t)Cg, KK);
    p.A.k = split_map((uint32_t)Mg * KK, KK, Cg * KK, 1);
    p.A.lanes_k = 0;
    return p;
}

// Up to 16 rows, channels that are no multiple of 16 and 800 indices or more: where the small-tile kernel would run the problem
// if the patch kernel did not, it is the faster one (patch kernel's time over its own 1.03 - 1.5, seven problems of 350 to 660
// tiles; with fewer indices 0.85 - 1.4, twelve problems, median 0.98).
static bool direct_before_patch(IgemmProblem &pd, const IgemmProblem &p, const PatchGeom &g)
{
    return p.M <= 16 && g.Cred % 16 && p.K >= 800 && !patch_forced() && igemm_take_direct(pd, &p);
}

// dy as the patch operand of backward-data at stride 1 (pixels = input positions, mirrored taps)
static bool bwd_data_patch(const cg_conv_desc &d, int OH, int OW, const float *dy, IgemmProblem &p)
{
    const int G = d.groups, Mg = d.M / G;
    PatchGeom g{};
    g.src = dy; g.src_elems = (uint64_t)d.N * d.M * OH * OW;
    g.gstride = (int64_t)Mg * OH * OW;
    g.Cred = (uint32_t)Mg; g.Hs = OH; g.Ws = OW; g.chan_stride = OH * OW; g.img_stride = d.M * OH * OW;
    g.OHo = d.H; g.OWo = d.W; g.s = 1; g.oy0 = d.pad_h - (d.KH - 1); g.ox0 = d.pad_w - (d.KW - 1);
    g.KH = d.KH; g.KW = d.KW; g.flip = 1;
    g.taps = g.tap_slots = 1;
    if (!patch_plan(g, (uint32_t)(d.C / G), (uint32_t)d.N * d.H * d.W, (uint32_t)G, p.math) || (g.Cred % 16 && igemm_in_pieces(p))) return false;
    IgemmProblem pd = bwd_data_direct_problem(d, OH, OW, dy, nullptr, nullptr, 0);
    pd.math = p.math;
    if (direct_before_patch(pd, p, g)) return false;
    p.patch = g; p.use_patch = 1;
    return true;
}

// Backward-data of a convolution with stride (sh, sw) > 1 as ONE stride-1 problem on the matrix
// cores.  Write an input row as ih + ph = sh*i + rh (cell i, phase rh < sh).  Only the taps
// kh = rh + sh*a reach it, from output row oh = i - a, so
//   dx[n, c, sh*i + rh - ph, sw*j + rw - pw] = sum_{m, a, b} dy[n, m, i - a, j - b] * w[m, c, rh + sh*a, rw + sw*b]:
// a correlation of dy with Ah x Aw = ceil(KH/sh) x ceil(KW/sw) taps whose "output channels" are the
// Cg * sh * sw pairs (channel, phase), the filters rearranged accordingly (zeros for taps beyond
// the window), and whose result is scattered cell by cell into dx (depth to space; phases outside
// the image are dropped).  Every dx element is the row/column pair of exactly one cell and phase,
// so dx is overwritten completely.  The first layer of the benchmark net (3 channels, 11x11,
// stride 4) becomes 48 rows x 864 reduction indices, of which 121/144 multiply a real tap.
struct StridedGeom { int sh, sw, Ah, Aw, Ch, Cw, R, Kp; uint32_t Np; };

static bool strided_geom(const cg_conv_desc &d, StridedGeom &s, int min_rows = 8)
{
    s.sh = d.stride_h; s.sw = d.stride_w;
    s.Ah = (d.KH + s.sh - 1) / s.sh; s.Aw = (d.KW + s.sw - 1) / s.sw;
    s.Ch = (d.H - 1 + d.pad_h) / s.sh + 1; s.Cw = (d.W - 1 + d.pad_w) / s.sw + 1;
    const int64_t R = (int64_t)(d.C / d.groups) * s.sh * s.sw, Kp = (int64_t)(d.M / d.groups) * s.Ah * s.Aw;
    const int64_t Np = (int64_t)d.N * s.Ch * s.Cw;
    if (R < min_rows || R >= (1 << 20) || Kp >= (1 << 28) || Np >= (1ll << 30) || R * Kp * d.groups >= (1ll << 29)) return false;
    s.R = (int)R; s.Kp = (int)Kp; s.Np = (uint32_t)Np;
    return true;
}

static StridedTaps strided_taps(const cg_conv_desc &d, int OH, int OW, const float *dy, const float *w, int math)
{
    return StridedTaps{dy, w, OH, OW, d.M, d.M / d.groups, d.C / d.groups, d.KH, d.KW, d.stride_h, d.stride_w, math == CG_MATH_BF16};
}

static IgemmProblem bwd_data_strided_problem(const cg_conv_desc &d, const StridedGeom &sg, int OH, int OW, const float *dy,
                                             const float *wt, float *dx, int accumulate)
{
    const int G = d.groups, Cg = d.C / G, Mg = d.M / G, P = OH * OW, T = sg.Ah * sg.Aw;
    IgemmProblem p{};
    p.A.ptr = wt;
    p.A.row = linear_map((uint32_t)sg.R, sg.Kp);
    p.A.k = linear_map((uint32_t)sg.Kp, 1);
    p.A.limA = p.A.limB = 1;
    p.A.gstride = (int64_t)sg.R * sg.Kp;
    p.A.elems = (uint64_t)G * sg.R * sg.Kp;
    p.A.lanes_k = 1;
    // dy seen from a cell (n, i, j): origin (i, j), tap (m, a, b) subtracts (a, b)
    p.B.ptr = dy;
    IndexMap cell{};
    cell.count = sg.Np;
    cell.d1 = make_fastdiv((uint32_t)sg.Ch * sg.Cw);
    cell.d2 = make_fastdiv((uint32_t)sg.Cw);
    cell.s1 = d.M * P; cell.s2 = OW; cell.s3 = 1;
    cell.sa = 1; cell.sb = 1;
    IndexMap tap{};
    tap.count = (uint32_t)sg.Kp;
    tap.d1 = make_fastdiv((uint32_t)T);
    tap.d2 = make_fastdiv((uint32_t)sg.Aw);
    tap.s1 = P; tap.s2 = -OW; tap.s3 = -1;
    tap.sa = -1; tap.sb = -1;
    p.B.row = cell; p.B.k = tap;
    p.B.limA = OH; p.B.limB = OW;
    p.B.gstride = (int64_t)Mg * P;
    p.B.elems = (uint64_t)d.N * d.M * P;
    p.B.lanes_k = 0;
    p.B.check = 1;
    // C: row (c, rh, rw) and cell (n, i, j) -> dx[n, c, sh*i + rh - ph, sw*j + rw - pw]
    const int HW = d.H * d.W;
    p.c_ptr = dx;
    p.c_scatter = 1;
    p.c_row = IndexMap{};
    p.c_row.count = (uint32_t)sg.R;
    p.c_row.d1 = make_fastdiv((uint32_t)sg.sh * sg.sw);
    p.c_row.d2 = make_fastdiv((uint32_t)sg.sw);
    p.c_row.s1 = HW; p.c_row.s2 = d.W; p.c_row.s3 = 1; p.c_row.o0 = -d.pad_h * d.W - d.pad_w;
    p.c_row.sa = 1; p.c_row.a0 = -d.pad_h; p.c_row.sb = 1; p.c_row.b0 = -d.pad_w;
    p.c_col = IndexMap{};
    p.c_col.count = sg.Np;
    p.c_col.d1 = make_fastdiv((uint32_t)sg.Ch * sg.Cw);
    p.c_col.d2 = make_fastdiv((uint32_t)sg.Cw);
    p.c_col.s1 = d.C * HW; p.c_col.s2 = sg.sh * d.W; p.c_col.s3 = sg.sw;
    p.c_col.sa = sg.sh; p.c_col.sb = sg.sw;
    p.c_limA = d.H; p.c_limB = d.W;
    p.c_gstride = (int64_t)Cg * HW;
    p.M = (uint32_t)sg.R; p.N = sg.Np; p.K = (uint32_t)sg.Kp;
    p.flops = 2.0 * Mg * Cg * d.KH * d.KW * ((double)d.N * P) * G;
    p.groups = G; p.splits = 1; p.k_per_split = p.K;
    p.accumulate = accumulate;
    return p;
}

// The same for direct_kernel: A((c, rh, rw), (m, a, b)) = w[m][c][rh + sh*a][rw + sw*b], nothing beyond the window.
static IgemmProblem bwd_data_strided_direct_problem(const cg_conv_desc &d, const StridedGeom &sg, int OH, int OW, const float *dy,
                                                    const float *w, float *dx, int accumulate)
{
    const int Cg = d.C / d.groups, Mg = d.M / d.groups, KK = d.KH * d.KW;
    IgemmProblem p = bwd_data_strided_problem(d, sg, OH, OW, dy, w, dx, accumulate);
    p.A.row = IndexMap{};
    p.A.row.count = (uint32_t)sg.R;
    p.A.row.d1 = make_fastdiv((uint32_t)sg.sh * sg.sw);
    p.A.row.d2 = make_fastdiv((uint32_t)sg.sw);
    p.A.row.s1 = KK; p.A.row.s2 = d.KW; p.A.row.s3 = 1;
    p.A.row.sa = 1; p.A.row.sb = 1;
    p.A.k = IndexMap{};
    p.A.k.count = (uint32_t)sg.Kp;
    p.A.k.d1 = make_fastdiv((uint32_t)sg.Ah * sg.Aw);
    p.A.k.d2 = make_fastdiv((uint32_t)sg.Aw);
    p.A.k.s1 = Cg * KK; p.A.k.s2 = sg.sh * d.KW; p.A.k.s3 = sg.sw;
    p.A.k.sa = sg.sh; p.A.k.sb = sg.sw;
    p.A.limA = d.KH; p.A.limB = d.KW;
    p.A.check = 1;
    p.A.gstride = (int64_t)Mg * Cg * KK;
    p.A.elems = (uint64_t)d.M * Cg * KK;
    p.A.lanes_k = 0;
    return p;
}

// dy as the patch operand of that problem: cells are the pixels, the taps are mirrored
static bool bwd_data_strided_patch(const cg_conv_desc &d, const StridedGeom &sg, int OH, int OW, const float *dy,
                                   IgemmProblem &p)
{
    const int G = d.groups, Mg = d.M / G;
    PatchGeom g{};
    g.src = dy; g.src_elems = (uint64_t)d.N * d.M * OH * OW;
    g.gstride = (int64_t)Mg * OH * OW;
    g.Cred = (uint32_t)Mg; g.Hs = OH; g.Ws = OW; g.chan_stride = OH * OW; g.img_stride = d.M * OH * OW;
    g.OHo = sg.Ch; g.OWo = sg.Cw; g.s = 1; g.oy0 = -(sg.Ah - 1); g.ox0 = -(sg.Aw - 1);
    g.KH = sg.Ah; g.KW = sg.Aw; g.flip = 1;
    g.taps = (uint32_t)(d.KH * d.KW); g.tap_slots = (uint32_t)(sg.Ah * sg.sh * sg.Aw * sg.sw);
    if (!patch_plan(g, (uint32_t)sg.R, sg.Np, (uint32_t)G, p.math) || (g.Cred % 16 && igemm_in_pieces(p))) return false;
    IgemmProblem pd = bwd_data_strided_direct_problem(d, sg, OH, OW, dy, nullptr, nullptr, 0);
    pd.math = p.math;
    if (direct_before_patch(pd, p, g)) return false;
    p.patch = g; p.use_patch = 1;
    return true;
}

static uint64_t copy_elems(const cg_conv_desc &d, const StridedGeom &sg)
{
    return (uint64_t)d.groups * sg.R * padded16(d.M / d.groups) * sg.Ah * sg.Aw;
}
static size_t strided_copy_bytes(const cg_conv_desc &d, const StridedGeom &sg) { return round256((size_t)copy_elems(d, sg) * sizeof(float)); }

// patch: in the patch kernel's order, else the gathered kernel's
static FilterPrep strided_prep(const cg_conv_desc &d, const StridedGeom &sg, bool patch, const IgemmProblem &p, size_t room)
{
    FilterPrep f{};
    f.kind = patch ? CG_PREP_STRIDED_TAPS : CG_PREP_STRIDED_ROWS;
    f.Mg = d.M / d.groups; f.Cg = d.C / d.groups; f.KH = d.KH; f.KW = d.KW;
    f.sh = sg.sh; f.sw = sg.sw; f.Ah = sg.Ah; f.Aw = sg.Aw;
    f.floats = (size_t)d.groups * sg.R * sg.Kp;
    if (patch) tap_major_copy(f, copy_elems(d, sg), p, room);
    return f;
}

int conv_bwd_data_impl(const cg_conv_desc &d, const float *dy, const float *w, float *dx, const float *gate, void *ws,
                       size_t ws_bytes, int accumulate, hipStream_t stream, int math, const float *prepared,
                       bool beside_other_stream)
{
    if (!math_ok(math)) return CG_EINVAL;
    ProfTag tag("conv_bwd_data", -1);
    int OH, OW;
    const int rc = conv_check(&d, &OH, &OW);
    if (rc) return rc;
    StridedGeom sg;
    if ((d.stride_h != 1 || d.stride_w != 1) && strided_geom(d, sg)) {
        const size_t wt_bytes = round256((size_t)d.groups * sg.R * sg.Kp * sizeof(float));
        if (!ws || ws_bytes < wt_bytes) return CG_ENOSPC;
        if (!aligned16(ws)) return CG_EINVAL;
        float *wt = static_cast<float *>(ws);
        IgemmProblem p = bwd_data_strided_problem(d, sg, OH, OW, dy, prepared ? prepared : wt, dx, accumulate);
        p.gate = gate;
        p.math = math;
        p.taps = strided_taps(d, OH, OW, dy, w, math);
        const size_t copy = strided_copy_bytes(d, sg);
        const bool patch = ws_bytes >= copy && bwd_data_strided_patch(d, sg, OH, OW, dy, p);
        const FilterPrep f = strided_prep(d, sg, patch, p, prepared ? kSlotRoom : ws_bytes);
        if (patch) tap_major_filters(p, f, p.A.ptr, w);
        if (!patch) {
            IgemmProblem pd = bwd_data_strided_direct_problem(d, sg, OH, OW, dy, w, dx, accumulate);
            pd.gate = gate;
            pd.math = math;
            pd.taps = p.taps;
            if (igemm_take_direct(pd, &p)) {
                const int rs = igemm_scratch_check(p, static_cast<char *>(ws) + wt_bytes, ws_bytes - wt_bytes);
                return rs ? rs : igemm_launch(pd, stream);
            }
        }
        if (!prepared) {
            const int rc2 = filter_prep_launch(1, &f, &w, &wt, stream);
            if (rc2) return rc2;
        }
        if (patch) return igemm_run(p, nullptr, 0, stream);
        return igemm_run(p, static_cast<char *>(ws) + wt_bytes, ws_bytes - wt_bytes, stream);
    }
    if ((d.stride_h != 1 || d.stride_w != 1) && math != CG_MATH_FP32) return CG_EUNSUPPORTED;   // fewer than eight rows: fp32 only
    if (d.stride_h != 1 || d.stride_w != 1) {
        // Fewer than eight (channel, phase) rows of a group fill less than half of a matrix tile.  What a matrix tile takes hardly
        // depends on them, what a thread per element takes goes with rows times indices, and up to 288 of these the
        // latter is faster: 700 problems, direct_kernel's time over this one's at 2 - 7 rows 1.15 - 6.6, median 2.2 (64 images of 28x28,
        // 256 channels in as many groups, 3x3 stride 2: 326 / 32 us; by stride phase, as it once was, 234); beyond, 0.4 - 1.1 with
        // 5 to 7 rows, 0.6 - 1.5 with fewer, and down to 0.1 from a thousand indices on (16 images of 86x95, 504 -> 1 channels,
        // 3x3 stride 2: 51 us; by stride phase 290).  Dimensions that direct_kernel's index maps do not cover end here too.
        if (strided_geom(d, sg, 1) && (int64_t)sg.R * sg.Kp > 288) {
            IgemmProblem pd = bwd_data_strided_direct_problem(d, sg, OH, OW, dy, w, dx, accumulate);
            pd.gate = gate;
            pd.taps = strided_taps(d, OH, OW, dy, w, math);
            if ((pd.direct = direct_choice(pd, false, nullptr, false)) != 0) {
                const int rc2 = igemm_launch(pd, stream);
                if (rc2 != CG_EUNSUPPORTED) return rc2;
            }
        }
        const GatherArgs a{d, OH, OW, dy, w, gate, dx, accumulate, make_fastdiv((uint32_t)d.W), make_fastdiv((uint32_t)d.H), make_fastdiv((uint32_t)d.C),
                           make_fastdiv((uint32_t)(d.C / d.groups)), make_fastdiv((uint32_t)d.stride_h), make_fastdiv((uint32_t)d.stride_w)};
        const size_t total = (size_t)d.N * d.C * d.H * d.W;
        const unsigned blocks = (unsigned)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
        hipLaunchKernelGGL(bwd_data_strided_kernel, dim3(blocks), dim3(256), 0, stream, a);
        CG_HIP_TRY(hipGetLastError());
        return CG_OK;
    }
    const int G = d.groups, Cg = d.C / G, Mg = d.M / G, KK = d.KH * d.KW;
    const size_t wt_bytes = round256((size_t)d.M * Cg * KK * sizeof(float));
    if (!ws || ws_bytes < wt_bytes) return CG_ENOSPC;
    if (!aligned16(ws)) return CG_EINVAL;
    float *wt = static_cast<float *>(ws);
    const float *wuse = prepared ? prepared : wt;
    {
        IgemmProblem pp = bwd_data_problem(d, OH, OW, dy, wuse, dx, accumulate);
        pp.gate = gate;
        pp.math = math;
        pp.beside_other_stream = beside_other_stream ? 1 : 0;
        const size_t copy = bwd_copy_bytes(d);
        if (bwd_data_patch(d, OH, OW, dy, pp) && ws_bytes >= copy) {
            const FilterPrep f = bwd_patch_prep(d, pp, prepared ? kSlotRoom : ws_bytes);
            if (!prepared) {
                const int rc2 = filter_prep_launch(1, &f, &w, &wt, stream);
                if (rc2) return rc2;
            }
            tap_major_filters(pp, f, wuse, w);
            return igemm_run(pp, nullptr, 0, stream);
        }
    }
    const bool in_place = bwd_data_reads_filters_in_place(d);
    IgemmProblem p = bwd_data_problem(d, OH, OW, dy, in_place ? w : wuse, dx, accumulate);
    p.gate = gate;
    p.math = math;
    if (!in_place) {
        IgemmProblem pd = bwd_data_direct_problem(d, OH, OW, dy, w, dx, accumulate);
        pd.gate = gate;
        pd.math = math;
        if (igemm_take_direct(pd, &p)) {
            const int rs = igemm_scratch_check(p, static_cast<char *>(ws) + wt_bytes, ws_bytes - wt_bytes);
            return rs ? rs : igemm_launch(pd, stream);
        }
    }
    if (!in_place && !prepared) {
        const size_t total = (size_t)d.M * Cg * KK;
        const unsigned blocks = (unsigned)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
        hipLaunchKernelGGL(transpose_filters_kernel, dim3(blocks), dim3(256), 0, stream, w, wt, G, Mg, Cg, KK);
        CG_HIP_TRY(hipGetLastError());
    }
    return igemm_run(p, static_cast<char *>(ws) + wt_bytes, ws_bytes - wt_bytes, stream);
}

FilterPrep conv_fwd_filter_prep(const cg_conv_desc &d, int math)
{
    FilterPrep f{};
    int OH, OW;
    if (conv_check(&d, &OH, &OW)) return f;
    IgemmProblem p = fwd_problem(d, OH, OW, nullptr, nullptr, nullptr, nullptr);
    p.math = math;
    StemGeom sg;
    if (!fwd_patch(d, OH, OW, nullptr, p)) {
        if (!fwd_stem(d, OH, OW, nullptr, p, sg)) return f;
        f.kind = CG_PREP_PIECES;
        f.Mg = d.M / d.groups; f.Cg = d.C / d.groups; f.KH = d.KH; f.KW = d.KW;
        f.floats = (size_t)sg.copy_floats;
        return f;
    }
    return fwd_patch_prep(d, p, kSlotRoom);
}

FilterPrep conv_bwd_data_filter_prep(const cg_conv_desc &d, int math)
{
    FilterPrep f{};
    int OH, OW;
    if (conv_check(&d, &OH, &OW)) return f;
    f.Mg = d.M / d.groups; f.Cg = d.C / d.groups; f.KH = d.KH; f.KW = d.KW;
    StridedGeom sg;
    if ((d.stride_h != 1 || d.stride_w != 1) && strided_geom(d, sg)) {
        IgemmProblem p = bwd_data_strided_problem(d, sg, OH, OW, nullptr, nullptr, nullptr, 0);
        p.math = math;
        const bool patch = bwd_data_strided_patch(d, sg, OH, OW, nullptr, p);
        IgemmProblem pd = bwd_data_strided_direct_problem(d, sg, OH, OW, nullptr, nullptr, nullptr, 0);
        pd.math = math;
        if (!patch && igemm_take_direct(pd, &p)) return f;
        return strided_prep(d, sg, patch, p, kSlotRoom);
    }
    if (d.stride_h != 1 || d.stride_w != 1) return f;            // fewer than eight (channel, phase) rows: w itself is read
    IgemmProblem pp = bwd_data_problem(d, OH, OW, nullptr, nullptr, nullptr, 0);
    pp.math = math;
    f.floats = (size_t)d.M * f.Cg * d.KH * d.KW;
    if (bwd_data_patch(d, OH, OW, nullptr, pp)) return bwd_patch_prep(d, pp, kSlotRoom);
    if (!bwd_data_reads_filters_in_place(d)) {
        IgemmProblem pd = bwd_data_direct_problem(d, OH, OW, nullptr, nullptr, nullptr, 0);
        pd.math = math;
        if (igemm_take_direct(pd, &pp)) return f;
        f.kind = CG_PREP_TRANSPOSE;
    }
    return f;
}

size_t conv_filter_prep_max_floats(const cg_conv_desc &d)
{
    const size_t fwd = (size_t)d.M * padded16(d.C / d.groups), bwd = (size_t)d.C * padded16(d.M / d.groups);
    size_t m = (fwd > bwd ? fwd : bwd) * d.KH * d.KW / 2 * 3;          // (three pieces of each value)
    int OH, OW;
    StemGeom st;
    if (conv_check(&d, &OH, &OW) == CG_OK && fwd_stem(d, OH, OW, nullptr, fwd_problem(d, OH, OW, nullptr, nullptr, nullptr, nullptr), st) && st.copy_floats > m)
        m = (size_t)st.copy_floats;
    StridedGeom sg;
    if ((d.stride_h != 1 || d.stride_w != 1) && strided_geom(d, sg)) {
        const size_t s2 = (size_t)copy_elems(d, sg) / 2 * 3;
        if (s2 > m) m = s2;
    }
    return m;
}

int filter_prep_launch(int n, const FilterPrep *jobs, const float *const *w, float *const *dst, hipStream_t stream)
{
    auto items_of = [](const FilterPrep &f) -> unsigned long long { return f.kind == CG_PREP_NONE ? 0 : f.pieces ? f.floats / f.pieces : f.floats; };
    unsigned long long all = 0;
    for (int k = 0; k < n; ++k) all += items_of(jobs[k]);
    const int per = all <= kPrepOneEach ? 1 : 4;
    int i = 0;
    while (i < n) {
        PrepTable t{};
        unsigned long long blocks = 0;
        while (i < n && t.n < kPrepJobs) {
            const FilterPrep &f = jobs[i];
            if (f.kind == CG_PREP_NONE || f.floats == 0) { ++i; continue; }
            if (!w[i] || !dst[i] || !aligned16(dst[i])) return CG_EINVAL;
            const unsigned long long items = items_of(f), need = (items + 256 * per - 1) / (256 * per);
            if (blocks + need >= (1ull << 31)) break;
            PrepJob &j = t.j[t.n++];
            j.w = w[i]; j.dst = dst[i]; j.kind = f.kind; j.Mg = f.Mg; j.Cg = f.Cg; j.KH = f.KH; j.KW = f.KW;
            j.sh = f.sh; j.sw = f.sw; j.Ah = f.Ah; j.Aw = f.Aw;
            j.pieces = f.pieces; j.first_block = (unsigned)blocks; j.total = items;
            blocks += need;
            ++i;
        }
        if (t.n == 0) {
            if (i < n) return CG_EUNSUPPORTED;
            break;
        }
        hipLaunchKernelGGL(per == 1 ? prepare_filters_kernel<1> : prepare_filters_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, stream, t);
        CG_HIP_TRY(hipGetLastError());
    }
    return CG_OK;
}

// The reduction runs over pixels (n, oh, ow).  Its index space pads every image's OH*OW pixels to
// a multiple of four (padding indices read as zero in B), so that dy, contiguous along the pixels
// of one image, can be fetched in aligned groups of four that never straddle two images.
static IgemmProblem bwd_weight_problem(const cg_conv_desc &d, int OH, int OW, const float *x, const float *dy,
                                       float *dw, int math)
{
    const int G = d.groups, Cg = d.C / G, Mg = d.M / G, Kg = Cg * d.KH * d.KW, P = OH * OW;
    const int Pp = (P + 3) / 4 * 4;
    IgemmProblem p{};
    p.A.ptr = dy;
    p.A.row = linear_map(Mg, P);
    p.A.k = split_map((uint32_t)d.N * Pp, Pp, d.M * P, 1);
    p.A.limA = p.A.limB = 1;
    p.A.gstride = (int64_t)Mg * P;
    p.A.elems = (uint64_t)d.N * d.M * P;
    p.A.lanes_k = 1;
    p.B.ptr = x;
    p.B.row = tap_map(d, Cg);
    p.B.k = window_origin_map(d, OH, OW);
    p.B.k.count = (uint32_t)d.N * Pp;
    p.B.k.d1 = make_fastdiv((uint32_t)Pp);
    p.B.k.r1_lim = (uint32_t)P;
    if (bwd_data_reads_filters_in_place(d)) {           // a 1x1 window at stride 1: x lies along the pixels as dy does
        p.B.k = split_map((uint32_t)d.N * Pp, Pp, d.C * P, 1);
        p.B.k.r1_lim = (uint32_t)P;
    }
    p.B.limA = d.H; p.B.limB = d.W;
    p.B.gstride = (int64_t)Cg * d.H * d.W;
    p.B.elems = (uint64_t)d.N * d.C * d.H * d.W;
    p.B.lanes_k = 1;
    p.B.check = (d.pad_h || d.pad_w) ? 1 : 0;
    p.c_ptr = dw;
    p.c_row_stride = Kg;
    p.c_col = linear_map(Kg, 1);
    p.c_gstride = (int64_t)Mg * Kg;
    p.M = Mg; p.N = Kg; p.K = (uint32_t)d.N * Pp;
    p.flops = 2.0 * Mg * (double)Kg * ((double)d.N * P) * G;
    p.groups = G; p.splits = 1; p.k_per_split = p.K;
    // the band kernel, where it applies: x as padded rows in LDS, dy in tiles of 16 pixels
    if (d.stride_h == d.stride_w) {
        WgradGeom wgm{};
        wgm.x = x; wgm.x_elems = (uint64_t)d.N * d.C * d.H * d.W;
        wgm.C = d.C; wgm.Cg = Cg; wgm.H = d.H; wgm.W = d.W; wgm.OH = OH; wgm.OW = OW; wgm.s = d.stride_h;
        wgm.pad_h = d.pad_h; wgm.pad_w = d.pad_w; wgm.KH = d.KH; wgm.KW = d.KW; wgm.M = d.M;
        uint32_t splits = 1;
        if (wgrad_plan(wgm, (uint32_t)Mg, (uint32_t)Kg, (uint32_t)G, (uint32_t)d.N, &splits)) {
            p.use_wgrad = 1;
            p.wgrad = wgm;
            p.splits = splits;
        }
        BandGeom bg{};
        bg.x = x; bg.x_elems = wgm.x_elems; bg.dy = dy; bg.dy_elems = p.A.elems;
        bg.N = d.N; bg.C = d.C; bg.Cg = Cg; bg.H = d.H; bg.W = d.W; bg.OH = OH; bg.OW = OW; bg.s = d.stride_h;
        bg.pad_h = d.pad_h; bg.pad_w = d.pad_w; bg.KH = d.KH; bg.KW = d.KW; bg.M = d.M;
        if (!p.use_wgrad && band_plan(bg, p.M, p.N, p.groups, gathered_plan(p.M, p.N, p.K, p.groups), math, &splits)) {
            p.use_band = 1;
            p.band = bg;
            p.splits = splits;
        }
    }
    return p;
}

int conv_bwd_weight_impl(const cg_conv_desc &d, const float *x, const float *dy, float *dw, float *db,
                         void *ws, size_t ws_bytes, hipStream_t stream, int math, hipStream_t bias_stream,
                         void *bias_ws, size_t bias_ws_bytes)
{
    if (!math_ok(math)) return CG_EINVAL;
    ProfTag tag("conv_bwd_weight", -1);
    int OH, OW;
    const int rc = conv_check(&d, &OH, &OW);
    if (rc) return rc;
    IgemmProblem p = bwd_weight_problem(d, OH, OW, x, dy, dw, math);
    p.math = math;
    if (math != CG_MATH_FP32 && p.use_wgrad) { p.use_wgrad = 0; p.splits = 1; }    // the fp32 band kernel
    const size_t bias_bytes = db ? bias_grad_ws_bytes(d.N, d.M) : 0;
    size_t split_bytes = round256(igemm_ws_bytes(p));
    if (p.use_band && ws_bytes < split_bytes + bias_bytes) {      // what the gathered kernel needs is always enough
        p.use_band = 0;
        p.splits = 1;
        split_bytes = round256(igemm_ws_bytes(p));
    }
    if (split_bytes + bias_bytes > 0) {
        if (!ws || ws_bytes < split_bytes + bias_bytes) return CG_ENOSPC;
        if (!aligned16(ws)) return CG_EINVAL;
    }
    // The bias sums go first: they need only dy and stream through HBM while another stream's matrix
    // kernel still runs; behind the weight gradient of a net's first layer they would sit, alone on
    // the GPU, between that kernel and the update the next iteration waits for.
    // (bias_stream: a stream of the caller's that has nothing else to do meanwhile -- a net's first
    // layer has no backward-data -- so that the sums run beside the matrix kernel, not in front of it.
    // Their partial sums then live in bias_ws, scratch memory that is free in THAT stream's order: `ws`
    // is only ordered by `stream`, on which earlier launches may still be reading it.)
    // A small layer's sums (one block per channel, one launch) ride in the launch that adds the K slices.
    const bool ride = db && !bias_stream && bias_grad_single_launch(d.N, OH * OW);
    if (db && !ride) {
        int rb;
        if (bias_stream) {
            if (!bias_ws || bias_ws_bytes < bias_bytes) return CG_ENOSPC;
            rb = bias_grad_launch(dy, d.N, d.M, OH * OW, db, bias_ws, bias_bytes, bias_stream);
        } else
            rb = bias_grad_launch(dy, d.N, d.M, OH * OW, db, static_cast<char *>(ws) + split_bytes, bias_bytes, stream);
        if (rb) return rb;
    }
    const BiasRider rider{dy, d.N, d.M, OH * OW, db};
    bool taken = false;
    const int rr = igemm_run(p, ws, split_bytes, stream, ride ? &rider : nullptr, &taken);
    if (rr || !ride || taken) return rr;
    return bias_grad_launch(dy, d.N, d.M, OH * OW, db, static_cast<char *>(ws) + split_bytes, bias_bytes, stream);
}

// K slices of the gathered kernel (and, where a test has switched it on, of the fp32 band kernel): the least any mode needs
static size_t gathered_bwd_weight_bytes(const cg_conv_desc &d, int OH, int OW)
{
    IgemmProblem p = bwd_weight_problem(d, OH, OW, nullptr, nullptr, nullptr, CG_MATH_FP32);
    if (p.use_band) { p.use_band = 0; p.splits = 1; }
    return igemm_ws_bytes(p);
}

size_t conv_ws_bytes(const cg_conv_desc &d, int pass)
{
    int OH, OW;
    if (conv_check(&d, &OH, &OW)) return 0;
    if (pass == CG_PASS_FWD) {
        IgemmProblem p = fwd_problem(d, OH, OW, nullptr, nullptr, nullptr, nullptr);
        const size_t gathered = igemm_ws_bytes(p);
        StemGeom sg;
        const size_t stem = fwd_stem(d, OH, OW, nullptr, p, sg) ? (size_t)sg.copy_floats * sizeof(float) : 0;
        IgemmProblem fp32 = p;
        p.math = CG_MATH_BF16;                   // (the mode in which most problems take the patch kernel)
        if (!fwd_patch(d, OH, OW, nullptr, p)) return stem > gathered ? stem : gathered;
        const size_t copy = fwd_copy_bytes(d);
        if (d.C / d.groups % 16 == 0 && fwd_patch(d, OH, OW, nullptr, fp32)) return copy;
        return std::max({copy, gathered, stem});
    }
    if (pass == CG_PASS_BWD_DATA) {
        StridedGeom sg;
        if ((d.stride_h != 1 || d.stride_w != 1) && strided_geom(d, sg)) {
            IgemmProblem p = bwd_data_strided_problem(d, sg, OH, OW, nullptr, nullptr, nullptr, 0);
            const size_t gathered = round256((size_t)d.groups * sg.R * sg.Kp * sizeof(float)) + igemm_ws_bytes(p);
            IgemmProblem fp32 = p;
            p.math = CG_MATH_BF16;
            if (!bwd_data_strided_patch(d, sg, OH, OW, nullptr, p)) return gathered;
            const size_t copy = strided_copy_bytes(d, sg);
            if (d.M / d.groups % 16 == 0 && bwd_data_strided_patch(d, sg, OH, OW, nullptr, fp32)) return copy;
            return copy > gathered ? copy : gathered;
        }
        if (d.stride_h != 1 || d.stride_w != 1) return 0;
        IgemmProblem p = bwd_data_problem(d, OH, OW, nullptr, nullptr, nullptr, 0);
        const size_t gathered = round256((size_t)d.M * (d.C / d.groups) * d.KH * d.KW * sizeof(float)) + igemm_ws_bytes(p);
        p.math = CG_MATH_BF16;
        const size_t copy = bwd_data_patch(d, OH, OW, nullptr, p) ? bwd_copy_bytes(d) : 0;
        return copy > gathered ? copy : gathered;
    }
    if (pass == CG_PASS_BWD_WEIGHT) {
        size_t most = gathered_bwd_weight_bytes(d, OH, OW);
        for (int math : {CG_MATH_FP32, CG_MATH_BF16, CG_MATH_BF16X3}) {
            const size_t b = igemm_ws_bytes(bwd_weight_problem(d, OH, OW, nullptr, nullptr, nullptr, math));
            if (b > most) most = b;
        }
        return round256(most) + bias_grad_ws_bytes(d.N, d.M);
    }
    return 0;
}

// ---- fully connected: y[b][o] = bias[o] + sum_i x[b][i] W[o][i] ------------------------------

static IgemmProblem fc_fwd_problem(int B, int IN, int OUT, const float *x, const float *W, const float *bias,
                                   float *y)
{
    IgemmProblem p{};
    p.A.ptr = x; p.A.row = linear_map(B, IN); p.A.k = linear_map(IN, 1); p.A.limA = p.A.limB = 1;
    p.A.elems = (uint64_t)B * IN; p.A.lanes_k = 1;
    p.B.ptr = W; p.B.row = linear_map(OUT, IN); p.B.k = linear_map(IN, 1); p.B.limA = p.B.limB = 1;
    p.B.elems = (uint64_t)OUT * IN; p.B.lanes_k = 1;
    p.c_ptr = y; p.c_row_stride = OUT; p.c_col = linear_map(OUT, 1);
    p.bias = bias; p.bias_mode = bias ? 2 : 0;
    p.M = B; p.N = OUT; p.K = IN;
    p.groups = 1; p.splits = 1; p.k_per_split = p.K;
    return p;
}

// dx[b][i] = sum_o dy[b][o] W[o][i]
static IgemmProblem fc_bwd_data_problem(int B, int IN, int OUT, const float *dy, const float *W, float *dx,
                                        int accumulate)
{
    IgemmProblem p{};
    p.A.ptr = dy; p.A.row = linear_map(B, OUT); p.A.k = linear_map(OUT, 1); p.A.limA = p.A.limB = 1;
    p.A.elems = (uint64_t)B * OUT; p.A.lanes_k = 1;
    p.B.ptr = W; p.B.row = linear_map(IN, 1); p.B.k = linear_map(OUT, IN); p.B.limA = p.B.limB = 1;
    p.B.elems = (uint64_t)OUT * IN; p.B.lanes_k = 0;
    p.c_ptr = dx; p.c_row_stride = IN; p.c_col = linear_map(IN, 1);
    p.M = B; p.N = IN; p.K = OUT;
    p.groups = 1; p.splits = 1; p.k_per_split = p.K;
    p.accumulate = accumulate;
    return p;
}

// dW[o][i] = sum_b dy[b][o] x[b][i];  db[o] = sum_b dy[b][o]
static IgemmProblem fc_bwd_weight_problem(int B, int IN, int OUT, const float *x, const float *dy, float *dW)
{
    IgemmProblem p{};
    p.A.ptr = dy; p.A.row = linear_map(OUT, 1); p.A.k = linear_map(B, OUT); p.A.limA = p.A.limB = 1;
    p.A.elems = (uint64_t)B * OUT; p.A.lanes_k = 0;
    p.B.ptr = x; p.B.row = linear_map(IN, 1); p.B.k = linear_map(B, IN); p.B.limA = p.B.limB = 1;
    p.B.elems = (uint64_t)B * IN; p.B.lanes_k = 0;
    p.c_ptr = dW; p.c_row_stride = IN; p.c_col = linear_map(IN, 1);
    p.M = OUT; p.N = IN; p.K = B;
    p.groups = 1; p.splits = 1; p.k_per_split = p.K;
    return p;
}

int fc_fwd_impl(int B, int IN, int OUT, const float *x, const float *W, const float *bias, float *y, void *ws,
                size_t ws_bytes, int relu, hipStream_t stream, int math)
{
    ProfTag tag("fc_fwd", -1);
    if (B <= 0 || IN <= 0 || OUT <= 0 || !math_ok(math)) return CG_EINVAL;
    IgemmProblem p = fc_fwd_problem(B, IN, OUT, x, W, bias, y);
    p.relu = relu;
    p.math = math;
    return igemm_run(p, ws, ws_bytes, stream);
}

int fc_bwd_data_impl(int B, int IN, int OUT, const float *dy, const float *W, float *dx, const float *gate,
                     int accumulate, void *ws, size_t ws_bytes, hipStream_t stream, int math)
{
    ProfTag tag("fc_bwd_data", -1);
    if (B <= 0 || IN <= 0 || OUT <= 0 || !math_ok(math)) return CG_EINVAL;
    IgemmProblem p = fc_bwd_data_problem(B, IN, OUT, dy, W, dx, accumulate);
    p.gate = gate;
    p.math = math;
    return igemm_run(p, ws, ws_bytes, stream);
}

int fc_bwd_weight_impl(int B, int IN, int OUT, const float *x, const float *dy, float *dW, float *db, void *ws,
                       size_t ws_bytes, hipStream_t stream, int math)
{
    ProfTag tag("fc_bwd_weight", -1);
    if (B <= 0 || IN <= 0 || OUT <= 0 || !math_ok(math)) return CG_EINVAL;
    IgemmProblem pw = fc_bwd_weight_problem(B, IN, OUT, x, dy, dW);
    pw.math = math;
    const int r = igemm_run(pw, ws, ws_bytes, stream);
    if (r) return r;
    if (db) return fc_bias_grad_launch(dy, B, OUT, db, stream);
    return CG_OK;
}

size_t fc_ws_bytes(int B, int IN, int OUT, int pass)
{
    if (B <= 0 || IN <= 0 || OUT <= 0) return 0;
    if (pass == CG_PASS_FWD) return igemm_ws_bytes(fc_fwd_problem(B, IN, OUT, nullptr, nullptr, nullptr, nullptr));
    if (pass == CG_PASS_BWD_DATA) return igemm_ws_bytes(fc_bwd_data_problem(B, IN, OUT, nullptr, nullptr, nullptr, 0));
    return igemm_ws_bytes(fc_bwd_weight_problem(B, IN, OUT, nullptr, nullptr, nullptr));
}

}  // namespace cg

// ---- C ABI --------------------------------------------------------------------------------

using namespace cg;

extern "C" int cg_debug_conv_operand(const cg_conv_desc *d, int pass, int operand, unsigned row, unsigned k,
                                     unsigned group, long long *elem_offset, int *valid)
{
    int OH, OW;
    const int rc = conv_check(d, &OH, &OW);
    if (rc) return rc;
    if (!elem_offset || !valid || (operand != 0 && operand != 1) || group >= (unsigned)d->groups) return CG_EINVAL;
    IgemmProblem p;
    if (pass == CG_PASS_FWD) p = fwd_problem(*d, OH, OW, nullptr, nullptr, nullptr, nullptr);
    else if (pass == CG_PASS_BWD_DATA) {
        if (d->stride_h != 1 || d->stride_w != 1) return CG_EUNSUPPORTED;
        p = bwd_data_problem(*d, OH, OW, nullptr, nullptr, nullptr, 0);
    } else if (pass == CG_PASS_BWD_WEIGHT)
        p = bwd_weight_problem(*d, OH, OW, nullptr, nullptr, nullptr, CG_MATH_FP32);
    else return CG_EINVAL;
    const Operand &op = operand == 0 ? p.A : p.B;
    if (row >= op.row.count || k >= p.K) return CG_EINVAL;
    int64_t off;
    igemm_host_element(op, row, k, &off, valid);
    *elem_offset = off + (int64_t)group * op.gstride;
    return CG_OK;
}

extern "C" int cg_debug_band_kernel(int on)
{
    wgrad_set_enabled(on);
    return CG_OK;
}

extern "C" int cg_debug_direct_kernel(int on)
{
    direct_set_enabled(on);
    return CG_OK;
}

extern "C" int cg_debug_patch_min_tiles(int tiles)
{
    if (tiles < 1) return CG_EINVAL;
    patch_set_min_tiles((uint32_t)tiles);
    return CG_OK;
}

extern "C" int cg_debug_resident_blocks(int blocks)
{
    if (blocks < 1) return CG_EINVAL;
    patch_set_resident_blocks((uint32_t)blocks);
    return CG_OK;
}

extern "C" int cg_conv_out_shape(const cg_conv_desc *d, int *OH, int *OW)
{
    return conv_check(d, OH, OW);
}

extern "C" size_t cg_conv_workspace_bytes(const cg_conv_desc *d, int pass)
{
    return d ? conv_ws_bytes(*d, pass) : 0;
}

extern "C" int cg_conv_fwd(const cg_conv_desc *d, const float *x, const float *w, const float *bias, float *y,
                           void *ws, size_t ws_bytes, void *stream)
{
    if (!d || !x || !w || !y) return CG_EINVAL;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y)) return CG_EINVAL;
    return conv_fwd_impl(*d, x, w, bias, y, ws, ws_bytes, 0, static_cast<hipStream_t>(stream));
}

extern "C" int cg_conv_bwd_data(const cg_conv_desc *d, const float *dy, const float *w, float *dx, void *ws,
                                size_t ws_bytes, void *stream)
{
    if (!d || !dy || !w || !dx) return CG_EINVAL;
    if (!aligned16(dy) || !aligned16(w) || !aligned16(dx)) return CG_EINVAL;
    return conv_bwd_data_impl(*d, dy, w, dx, nullptr, ws, ws_bytes, 0, static_cast<hipStream_t>(stream));
}

extern "C" int cg_conv_bwd_weight(const cg_conv_desc *d, const float *x, const float *dy, float *dw, float *dbias,
                                  void *ws, size_t ws_bytes, void *stream)
{
    if (!d || !x || !dy || !dw) return CG_EINVAL;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dw)) return CG_EINVAL;
    return conv_bwd_weight_impl(*d, x, dy, dw, dbias, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

// ---- the three passes with the arithmetic of the matrix instructions chosen by the caller -----------

extern "C" int cg_conv_fwd_math(const cg_conv_desc *d, const float *x, const float *w, const float *bias, float *y,
                                void *ws, size_t ws_bytes, int math, void *stream)
{
    if (!d || !x || !w || !y) return CG_EINVAL;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y)) return CG_EINVAL;
    return conv_fwd_impl(*d, x, w, bias, y, ws, ws_bytes, 0, static_cast<hipStream_t>(stream), 0, math);
}

extern "C" int cg_conv_bwd_data_math(const cg_conv_desc *d, const float *dy, const float *w, float *dx, void *ws,
                                     size_t ws_bytes, int math, void *stream)
{
    if (!d || !dy || !w || !dx) return CG_EINVAL;
    if (!aligned16(dy) || !aligned16(w) || !aligned16(dx)) return CG_EINVAL;
    return conv_bwd_data_impl(*d, dy, w, dx, nullptr, ws, ws_bytes, 0, static_cast<hipStream_t>(stream), math);
}

extern "C" int cg_conv_bwd_weight_math(const cg_conv_desc *d, const float *x, const float *dy, float *dw, float *dbias,
                                       void *ws, size_t ws_bytes, int math, void *stream)
{
    if (!d || !x || !dy || !dw) return CG_EINVAL;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dw)) return CG_EINVAL;
    return conv_bwd_weight_impl(*d, x, dy, dw, dbias, ws, ws_bytes, static_cast<hipStream_t>(stream), math);
}

// ---- backward-weight without a caller's workspace ------------------------------------------------
//
// The partial sums of the K slices and of the bias gradient live in a device array that is part of
// the library's code object: every GPU the library runs on holds its own copy, at its own address,
// from the moment the module is loaded until the process ends.  In host code the array's name is
// only a handle for hipGetSymbolAddress; the address that call returns for the current device is
// what the kernels are given.  Nothing has to start at zero: the matrix kernel writes every partial
// sum the finishing kernels read.  All calls on one GPU share the array, so two calls that overlap
// on that GPU (different streams, or threads) race.
static __device__ __align__(256) unsigned char scratch[CG_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];       // per device, filled on the first call with that device current

int scratch_for_current_device(void **out)
{
    int dev = -1;
    CG_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return CG_EUNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        CG_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || !aligned16(ptr)) return CG_EHIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return CG_OK;
}
}  // namespace

extern "C" int cg_conv_bwd_weight_noalloc(const cg_conv_desc *d, const float *x, const float *dy, float *dw,
                                          float *dbias, void *stream)
{
    if (!d || !x || !dy || !dw) return CG_EINVAL;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dw)) return CG_EINVAL;
    int OH, OW;
    const int rc = conv_check(d, &OH, &OW);
    if (rc) return rc;
    if (round256(gathered_bwd_weight_bytes(*d, OH, OW)) + bias_grad_ws_bytes(d->N, d->M) > (size_t)CG_NOALLOC_SCRATCH_BYTES) return CG_ENOSPC;
    void *ptr = nullptr;
    const int rs = scratch_for_current_device(&ptr);
    if (rs) return rs;
    return conv_bwd_weight_impl(*d, x, dy, dw, dbias, ptr, (size_t)CG_NOALLOC_SCRATCH_BYTES,
                                static_cast<hipStream_t>(stream));
}
