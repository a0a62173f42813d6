// Planning of the dense contractions: which kernel, which tile, how many K slices; and the kernels that
// add the slices and the bias gradient.
#include <algorithm>
#include <atomic>
#include <cstdio>
#include "cg_internal.h"
#include "igemm_device.h"

namespace cg {


namespace {

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

constexpr int KT = 16;                       // reduction indices per K-tile of the gathered kernel

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

// Row tile of split_gemm_kernel for the problems that run faster there than on the gathered kernel, 0 for
// all others.  Its blocks have one step of 32 indices in flight, the gathered kernel three or four K-tiles of 16: short
// and small problems, and backward-weight, whose long reduction is cut into slices, belong there (1x1 layers
// of 32 images of 28x28 forward 17.8 us there, 21.7 here; 375 x 336 with 5772 indices 46.5, 66.7).
// The lines, from 620 problems a mode; times there / here:
// - at most 16 rows (a 32-row tile wastes half): from 180 indices and 600 blocks 0.98 - 1.29, median 1.1 (one and two
//   pieces 1.1 - 1.5); fewer blocks only where the reduction is very long (4096 indices and more 1.04 - 1.1).
// - 1x1 backward-data, whose filters are read across (a load per element on both sides there): few padded rows, a
//   short reduction, 150 blocks and more: fp32 1.1 - 1.6; at 256 indices one and two pieces 0.83 - 0.9, so they end
//   before.  192 rows (a quarter padding) 0.8 - 0.9, two rounds of 256 rows 0.97.
// - images with few padded rows in fp32, enough blocks times indices: 0.98 - 1.46, median 1.1; whole multiples of 128 rows
//   suit both (0.93 - 1.14), more padding suits the 192- and 96-row tiles there (0.7 - 1.0); one and two pieces 0.7 - 1.24.
// - fully-connected forward and backward-data in fp32 from 108 images: 1.0 - 1.3 (256 images, 9216 -> 4096 159.6 / 151.0 us,
//   4096 -> 4096 backward-data 79.5 / 69.1); 64 images 0.8 - 1.0.  Not where columns lie apart in memory (1x1 layers
//   of planes of one pixel: 0.82).
// - their backward-weight in fp32 (rows across on both sides, the batch the reduction), whole steps of one layer, us: blocks times
//   images from 30 000 on 0 to 122 faster (256 images 9216 -> 4096 472 / 410, 4096 -> 4096 255 / 235, 4096 -> 1000 136 / 127), 16 000 to
//   26 000 -4.5 to 1.8, below or with fewer than 64 blocks -13 to 0.  Error against 64 bits 0.2 to 0.8 of what it was.
int pieces_mt(const IgemmProblem &p)
{
    if (p.A.check || p.B.k.r1_lim) return 0;
    const bool fp32 = p.math == CG_MATH_FP32, aq = quad_ok(p.A, p.K), image = p.B.row.d1.d > 1;
    if (!aq && p.A.lanes_k) return 0;
    const uint64_t rows = (uint64_t)(p.M + 127) / 128 * 128, blocks = rows / 128 * ((p.N + 127) / 128) * p.groups;
    if (rows / 128 > 65535) return 0;            // more row tiles than a launch takes along y: the gathered kernel has taller ones
    if (p.B.lanes_k || !image) {
        const bool bq = quad_ok(p.B, p.K) && p.K % 4 == 0, rows_in_line = !p.B.lanes_k && p.B.row.d2.d == 1 && p.B.row.s1 == 1;
        if (fp32 && !aq && rows_in_line && p.B.k.d1.d == 1 && p.B.k.d2.d == 1)
            return blocks >= 64 && blocks * p.K >= 30000 && p.M * 100ull >= rows * 84 ? 128 : 0;
        return fp32 && aq && (bq || rows_in_line) && p.N >= 1000 && p.K >= 512 && p.M * 100ull >= rows * 84 ? 128 : 0;
    }
    if (p.M <= 16) return (p.K >= 180 && blocks >= 600) || (p.K >= 4096 && p.N >= 16384) ? 16 : 0;
    if (!aq)
        return p.K >= 24 && p.K <= (fp32 ? 320u : 255u) && p.M * 100ull >= rows * 82 && blocks >= 150 && (blocks <= 256 || p.M > 256) ? 128 : 0;
    return fp32 && p.M > 64 && p.M % 128 != 0 && p.M * 100ull >= rows * 84 && p.N >= 4096 && p.K >= 128 && blocks * (p.K / 128) >= 400 ? 128 : 0;
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

void patch_set_resident_blocks(uint32_t b) { g_resident_override.store(b, std::memory_order_relaxed); }
uint32_t igemm_resident_blocks() { return resident_blocks(); }

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
    if (p.A.check && !p.direct) return CG_EUNSUPPORTED;
    if (p.c_scatter && (!p.taps.dy || !p.taps.w || (p.direct ? !p.A.check : !p.B.check || p.B.lanes_k))) return CG_EINVAL;
    p.A.shift = p.B.shift = 0;
    int rc = normalise_operand(p.A, p.groups);
    if (rc) return rc;
    if (p.A.row.count != p.M || p.B.row.count != p.N || p.A.k.count != p.K || p.B.k.count != p.K) return CG_EINVAL;
    rc = normalise_operand(p.B, p.groups);
    if (rc) return rc;
    if (!p.A.check) { p.A.limA = p.A.limB = 1; }
    if (!p.B.check) { p.B.limA = p.B.limB = 1; }

    if (p.direct) return direct_launch(p, quad_ok(p.A, p.K), quad_ok(p.A, p.K) && quad_ok(p.B, p.K), stream);
    const int mt = p.mt ? p.mt : pick_mt(p.M, p.N, p.groups, p.K);
    // how an operand's elements are fetched: 0 rows along the lanes, 1 k along the lanes, 2 aligned quads of k
    const int am = quad_ok(p.A, p.K) ? 2 : p.A.lanes_k ? 1 : 0;
    int bm = quad_ok(p.B, p.K) ? 2 : p.B.lanes_k ? 1 : 0;
    // A quad that reaches beyond K, or into the padding of a run of reduction indices, delivers the
    // floats that follow in memory (the next row's first elements): harmless only if the other
    // operand delivers exact zeros there, which the loaders that check every element do and the quad
    // loader does not.  Quads on both sides need a reduction range without any such position.
    if (am == 2 && bm == 2 && (p.K % 4 != 0 || p.A.k.r1_lim != 0 || p.B.k.r1_lim != 0)) bm = 1;
    if (!p.pieces) {
        if (p.math == CG_MATH_BF16) return gather_launch_1(p, mt, am, bm, stream);
        if (p.math == CG_MATH_BF16X3) return gather_launch_2(p, mt, am, bm, stream);
        return gather_launch_0(p, mt, am, bm, stream);
    }
    if (am == 1 || bm == 1) return CG_EUNSUPPORTED;
    if (p.math == CG_MATH_BF16) return split_gemm_1(p, mt, am == 2, bm == 2, stream);
    if (p.math == CG_MATH_BF16X3) return split_gemm_2(p, mt, am == 2, bm == 2, stream);
    return split_gemm_3(p, mt, am == 2, bm == 2, stream);
}

// ---- split-K: more blocks for problems whose C has few tiles ---------------------------------

namespace {

struct FinishArgs {
    float *part;
    int64_t plane;            // floats between consecutive K slices: groups * M * N
    int splits;
    float *c_ptr;
    int32_t c_row_stride;
    IndexMap c_col;
    IndexMap c_row;           // SCATTER only
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
    StridedTaps taps;
};

// C = (sum over the K slices) + bias, written through the problem's output map.  With few slices a
// thread adds them in slice order.  With many (ROWS = 8) a block owns 32 consecutive elements, its
// 8 thread rows add interleaved slices (row r: slices r, r+8, ...), and the 8 row sums are added
// in row order.  Either way the association is fixed by the number of slices alone, so the result
// does not depend on scheduling.
// (Written out here and in direct.hip: through one shared template the compiler orders this kernel's index arithmetic
// otherwise, and the pass after the backward weights of 64 images, 13 x 13, 384 -> 384 channels, 3 x 3, two groups, takes
// 23.7 us, not 21.9.)
template <bool SCATTER> __device__ __forceinline__ void finish_store(const FinishArgs &a, uint32_t i, float s)
{
    const uint32_t g = fdiv(i, a.divMN), rem = i - g * a.divMN.d;
    const uint32_t m = fdiv(rem, a.divN), n = rem - m * a.divN.d;
    if (a.bias_mode == 1) s += a.bias[(int64_t)g * a.bias_gstride + m];
    else if (a.bias_mode == 2) s += a.bias[(int64_t)g * a.bias_gstride + n];
    if (a.relu) s = fmaxf(s, 0.f);
    const Info ci = map_info(a.c_col, n);
    int32_t in_group = (int32_t)m * a.c_row_stride + ci.off;
    if constexpr (SCATTER) {
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

// Strided backward-data: a sum that is not finite is kept in place of its first slice (which nobody else reads) until the thread's
// other sums are stored, and done again from its taps then.  At its place in the loop this made the pass after 199 -> 12
// channels 5x5 stride 4, 52 images of 67x67, 20.3 us, not 18.3.
template <bool SCATTER> __device__ __forceinline__ bool finish_or_keep(const FinishArgs &a, uint32_t i, float s)
{
    if (SCATTER && __builtin_expect(!__builtin_isfinite(s), 0)) {
        a.part[i] = s;
        return true;
    }
    finish_store<SCATTER>(a, i, s);
    return false;
}
__device__ __forceinline__ void finish_kept(uint32_t i)
{
    const FinishArgs &a = first_argument<FinishArgs>();
    if (__builtin_isfinite(a.part[i])) return;
    const uint32_t g = fdiv(i, a.divMN), rem = i - g * a.divMN.d;
    const uint32_t m = fdiv(rem, a.divN), n = rem - m * a.divN.d;
    finish_store<true>(a, i, sum_of_taps(a.taps, a.c_row, a.c_col, g, m, n));
}

// AHEAD: a thread's next eight loads are in flight together (under a condition each, where fewer are left).  It pays
// where a thread has many; whole passes, us, plain / ahead: one thread per element, 2 slices 33.8 / 39.8, 3 slices
// 26.9 / 28.4, 7 slices 16.1 / 15.0, 13 slices 16.1 / 14.4; eight rows of threads, 32 slices 44.8 / 49.4, 49 slices 15.3 / 14.0,
// 64 slices 113.8 / 109.2, 512 slices 55.6 / 44.9.
template <int ROWS, bool AHEAD, bool SCATTER> __global__ __launch_bounds__(256) void splitk_finish_kernel(const FinishArgs a)
{
    if (a.r_dy && blockIdx.x >= a.finish_blocks) {       // a rider block: one channel of the bias gradient
        const int m = (int)(blockIdx.x - a.finish_blocks);
        __shared__ float red[256];
        const float s = bias_channel_sum(a.r_dy, a.rM, a.rP, m, 0, a.rN, a.r_divQP, 256u, red);
        if (threadIdx.x == 0) a.r_db[m] = s;
        return;
    }
    const uint32_t nblk = a.r_dy ? a.finish_blocks : gridDim.x;
    bool kept = false;
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
            kept |= finish_or_keep<SCATTER>(a, i, s);
        }
        if (SCATTER && kept)
            for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < a.total; i += nblk * 256) finish_kept(i);
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
            kept |= finish_or_keep<SCATTER>(a, i, s);
        }
        __syncthreads();
    }
    if (SCATTER && kept)
        for (uint32_t i0 = blockIdx.x * 32; i0 < a.total; i0 += nblk * 32)
            if (i0 + el < a.total) finish_kept(i0 + el);
}

// The same, four consecutive columns a thread (they are four consecutive elements of C): one look at the maps and one 16-byte
// load a slice for the four.  An element's sums are added in the same order.  Bound by launch and HBM: 384 x 1728 in two groups,
// 25 slices (66 MB), 21.2 -> 14.3 us alone.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void finish_store4(const FinishArgs &a, uint32_t i, f4 s)
{
    const uint32_t g = fdiv(i, a.divMN), rem = i - g * a.divMN.d;
    const uint32_t m = fdiv(rem, a.divN), n = rem - m * a.divN.d;
    if (a.bias_mode == 1) s += a.bias[(int64_t)g * a.bias_gstride + m];
    else if (a.bias_mode == 2) s += *reinterpret_cast<const f4u *>(a.bias + (int64_t)g * a.bias_gstride + n);
    if (a.relu)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = fmaxf(s[e], 0.f);
    const int64_t idx = (int64_t)g * a.c_gstride + ((int32_t)m * a.c_row_stride + map_info(a.c_col, n).off);
    if (a.gate) {
        const f4u gt = *reinterpret_cast<const f4u *>(a.gate + idx);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = gt[e] > 0.f ? s[e] : 0.f;
    }
    f4u *dst = reinterpret_cast<f4u *>(a.c_ptr + idx);
    if (a.accumulate) s += *dst;
    *dst = s;
}
template <int ROWS, bool AHEAD> __global__ __launch_bounds__(256) void splitk_finish4_kernel(const FinishArgs a)
{
    if (a.r_dy && blockIdx.x >= a.finish_blocks) {
        const int m = (int)(blockIdx.x - a.finish_blocks);
        __shared__ float red[256];
        const float s = bias_channel_sum(a.r_dy, a.rM, a.rP, m, 0, a.rN, a.r_divQP, 256u, red);
        if (threadIdx.x == 0) a.r_db[m] = s;
        return;
    }
    const uint32_t nblk = a.r_dy ? a.finish_blocks : gridDim.x, quads = a.total / 4;
    const int64_t plane = a.plane / 4;
    const f4 *part = reinterpret_cast<const f4 *>(a.part);
    // slices r, r + ROWS, ...
    auto sum = [&](uint32_t i, int r) {
        f4 s = {0.f, 0.f, 0.f, 0.f};
        if (ROWS == 1) { s = part[i]; r = 1; }           // (a chain of one starts with its first slice, of eight with zero)
        if constexpr (!AHEAD)
            for (int k = r; k < a.splits; k += ROWS) s += part[(int64_t)k * plane + i];
        else for (int k0 = r; k0 < a.splits; k0 += 8 * ROWS) {
            f4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = k0 + ROWS * u < a.splits ? part[(int64_t)(k0 + ROWS * u) * plane + i] : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + ROWS * u < a.splits) s += v[u];
        }
        return s;
    };
    if (ROWS == 1) {
        for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < quads; i += nblk * 256) finish_store4(a, 4 * i, sum(i, 0));
        return;
    }
    __shared__ f4 rows[8][32];
    const int el = threadIdx.x & 31, r = threadIdx.x >> 5;
    for (uint32_t i0 = blockIdx.x * 32; i0 < quads; i0 += nblk * 32) {
        const uint32_t i = i0 + el;
        rows[r][el] = i < quads ? sum(i, r) : f4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
        if (r == 0 && i < quads) {
            f4 s = rows[0][el];
#pragma unroll
            for (int k = 1; k < 8; ++k) s += rows[k][el];
            finish_store4(a, 4 * i, s);
        }
        __syncthreads();
    }
}

// Are the sums of K slices added four columns a thread?  Where aligned groups of four columns lie one behind the other in C, from
// 32 768 elements on.  Fewer leave a quarter of the blocks for as long a chain of loads a thread: 2 to 512 slices, us, one column /
// four: 512 to 12 288 elements 3.4 / 3.5 up to 48 slices, 4.2 / 4.7 with 200, 5.5 / 6.4 with 512; 32 768 and 36 864 within 0.3 of each other,
// 8.2 / 8.0 with 256; 147 456 4.6 / 3.2 with 16 and 53 / 46 with 512; 331 776 14.8 / 10.2 with 39.  (Both add an element's
// sums in the same order.)
bool columns_in_quads(const IgemmProblem &p)
{
    const IndexMap &c = p.c_col;
    return (uint64_t)p.groups * p.M * p.N >= 32768 && !p.c_scatter && p.N % 4 == 0 && c.d2.d == 1 && (c.d1.d == 1 ? c.s1 == 1 : c.d1.d % 4 == 0 && c.s2 == 1);
}

}  // namespace

// K slices for row tiles of mt rows: as many as make one round of resident blocks, at least 128
// reduction indices each.
static SplitPlan slices(uint32_t M, uint32_t N, uint32_t K, uint32_t groups, int mt)
{
    SplitPlan pl{1, K, 0, mt, 0};
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
    if (pl.splits < 2) return SplitPlan{1, K, 0, mt, 0};
    pl.ws_bytes = (size_t)pl.splits * groups * M * N * sizeof(float);
    return pl;
}

// A slice's sums are as long as its share of K, and their rounding error with them: split_gemm_kernel cuts K at least
// three quarters as often as the gathered kernel (in two or more rounds of blocks if need be), and never
// more often, so that the scratch memory a caller is told to bring is the gathered kernel's.
static SplitPlan plan_split(const IgemmProblem &p)
{
    const SplitPlan old = gathered_plan(p.M, p.N, p.K, p.groups);
    const int mt = pieces_mt(p);
    if (!mt) return old;
    SplitPlan pl = slices(p.M, p.N, p.K, p.groups, mt);
    pl.pieces = 1;
    const uint64_t tiles = (uint64_t)((p.M + mt - 1) / mt) * ((p.N + 127) / 128) * p.groups;
    uint64_t want = pl.splits;
    if (old.splits >= 2 && pl.splits * 4 < old.splits * 3)
        for (uint64_t rounds = 1; want * 4 < (uint64_t)old.splits * 3; ++rounds) want = rounds * kSplitBlocks / tiles;
    if (want > old.splits) want = old.splits;
    if (want == pl.splits) return pl;
    const uint64_t per = ((p.K + want - 1) / want + KT - 1) / KT * KT;
    pl.k_per_split = (uint32_t)per;
    pl.splits = (uint32_t)((p.K + per - 1) / per);
    pl.ws_bytes = pl.splits > 1 ? (size_t)pl.splits * p.groups * p.M * p.N * sizeof(float) : 0;
    return pl;
}

SplitPlan gathered_plan(uint32_t M, uint32_t N, uint32_t K, uint32_t groups)
{
    return slices(M, N, K, groups, pick_mt(M, N, groups, K));
}

// Scratch memory of the gathered kernel's K slices; split_gemm_kernel never takes more.
size_t igemm_ws_bytes(const IgemmProblem &p)
{
    if (p.use_patch) return 0;
    if (p.use_wgrad || p.use_band) return p.splits > 1 ? (size_t)p.splits * p.groups * p.M * p.N * sizeof(float) : 0;
    return gathered_plan(p.M, p.N, p.K, p.groups).ws_bytes;
}

bool igemm_in_pieces(const IgemmProblem &p) { return pieces_mt(p) == 128; }

bool igemm_take_direct(IgemmProblem &p, const IgemmProblem *other)
{
    const IgemmProblem &o = other ? *other : p;
    p.direct = 0;
    // (what split_gemm_kernel runs is added up from short sums of exact products: closer to 64 bits than the fp32 instruction)
    if (p.math != CG_MATH_FP32 || pieces_mt(o)) return false;
    const SplitPlan pl = plan_split(o);
    p.direct = direct_choice(p, quad_ok(p.A, p.K), &pl, o.A.lanes_k && !p.A.lanes_k);
    return p.direct != 0;
}

int igemm_scratch_check(const IgemmProblem &p, const void *ws, size_t ws_bytes)
{
    const SplitPlan pl = plan_split(p);
    if (pl.splits <= 1) return CG_OK;
    if (!ws || ws_bytes < pl.ws_bytes) return CG_ENOSPC;
    return aligned16(ws) ? CG_OK : CG_EINVAL;
}

int igemm_run(const IgemmProblem &p0, void *ws, size_t ws_bytes, hipStream_t stream, const BiasRider *rider, bool *rider_taken)
{
    if (rider_taken) *rider_taken = false;
    const bool ride = rider && rider->dy && rider->db && rider->M > 0 && rider->M <= 65536 &&
                      (uint64_t)rider->N * (uint64_t)((rider->P + 3) / 4) < (1ull << 31);
    if (!p0.use_patch && !p0.use_wgrad && !p0.use_band) {
        IgemmProblem p = p0;
        if (igemm_take_direct(p)) {
            const int rc = igemm_scratch_check(p0, ws, ws_bytes);        // a call is refused for the same reasons whichever kernel runs it
            if (rc) return rc;
            p.splits = 1; p.k_per_split = p.K;
            if (ride) p.rider = *rider;
            if (rider_taken) *rider_taken = ride;
            return igemm_launch(p, stream);
        }
    }
    const SplitPlan pl = p0.use_patch   ? SplitPlan{1, p0.K, 0, 0, 0}
                         : p0.use_wgrad || p0.use_band ? SplitPlan{p0.splits, p0.K, (size_t)(p0.splits > 1 ? p0.splits : 0) * p0.groups * p0.M * p0.N * sizeof(float), 0, 0}
                                        : plan_split(p0);
    if (pl.splits <= 1) {
        IgemmProblem p = p0;
        p.splits = 1; p.k_per_split = p.K; p.mt = pl.mt; p.pieces = pl.pieces;
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
    p.splits = pl.splits; p.k_per_split = pl.k_per_split; p.mt = pl.mt; p.pieces = pl.pieces;
    if (!p0.use_wgrad && !p0.use_band && !pl.pieces) p.direct = direct_for_slices(p0, quad_ok(p0.A, p0.K));
    const int rc = igemm_launch(p, stream);
    if (rc) return rc;
    FinishArgs a{};
    a.part = static_cast<float *>(ws);
    a.plane = p.c_split_stride;
    a.splits = (int)pl.splits;
    a.c_ptr = p0.c_ptr; a.c_row_stride = p0.c_row_stride; a.c_col = p0.c_col; a.c_gstride = p0.c_gstride;
    a.c_row = p0.c_row; a.c_limA = p0.c_limA; a.c_limB = p0.c_limB;
    a.taps = p0.taps;
    a.bias = p0.bias; a.bias_mode = p0.bias_mode; a.bias_gstride = p0.bias_gstride;
    a.M = p0.M; a.N = p0.N;
    a.divN = make_fastdiv(p0.N);
    a.divMN = make_fastdiv(p0.M * p0.N);
    a.accumulate = p0.accumulate; a.relu = p0.relu; a.gate = p0.gate;
    a.total = p0.groups * p0.M * p0.N;
    unsigned riders = 0;
    if (ride) {
        a.r_dy = rider->dy; a.rN = rider->N; a.rM = rider->M; a.rP = rider->P; a.r_db = rider->db;
        a.r_divQP = make_fastdiv((uint32_t)(rider->P + 3) / 4);
        riders = (unsigned)rider->M;
        if (rider_taken) *rider_taken = true;
    }
    const bool rows = pl.splits >= 16;
    const bool quads = columns_in_quads(p0);
    const uint32_t items = quads ? a.total / 4 : a.total;
    const unsigned blocks = rows ? std::min((items + 31) / 32, 65536u) : std::min((items + 255) / 256, 16384u);
    a.finish_blocks = blocks;
    auto launch = [&](auto *kernel) { hipLaunchKernelGGL(kernel, dim3(blocks + riders), dim3(256), 0, stream, a); };
    auto pick = [&](auto SC) {
        constexpr bool scatter = decltype(SC)::value;
        if (rows) pl.splits >= 40 ? launch(&splitk_finish_kernel<8, true, scatter>) : launch(&splitk_finish_kernel<8, false, scatter>);
        else pl.splits >= 6 ? launch(&splitk_finish_kernel<1, true, scatter>) : launch(&splitk_finish_kernel<1, false, scatter>);
    };
    if (quads) {
        if (rows) pl.splits >= 40 ? launch(&splitk_finish4_kernel<8, true>) : launch(&splitk_finish4_kernel<8, false>);
        else pl.splits >= 6 ? launch(&splitk_finish4_kernel<1, true>) : launch(&splitk_finish4_kernel<1, false>);
    } else if (p0.c_scatter) pick(std::true_type{});
    else pick(std::false_type{});
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

// ---- bias gradient of a convolution: db[m] = sum over n and pixels of dy[n][m][pix] ------------

namespace {

// block (m, s) sums the samples of slice s; the slices are added afterwards in slice order.
// The (image, group of four pixels) pairs of the slice are spread over the threads, each moving
// 16 bytes (4-byte aligned: planes of an odd pixel count start anywhere).
__global__ __launch_bounds__(256) void bias_grad_partial_kernel(const float *__restrict__ dy, int N, int M, int P,
                                                                int n_per, FastDiv divQP, float *__restrict__ part)
{
    const int m = blockIdx.x, sl = blockIdx.y;
    const int n_beg = sl * n_per, n_end = min(N, n_beg + n_per);
    __shared__ float red[256];
    const float s = bias_channel_sum(dy, M, P, m, n_beg, n_end, divQP, 256u, red);
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
