// Implicit GEMM on the bf16 matrix instructions: C[m][n] = sum_k A(m,k) * B(n,k).  The second kernel for
// gathered problems; igemm.hip says which of them it gets and what both take.  Operand elements are addressed
// through index maps (cg_internal.h), so the im2col matrix is never materialised; zero padding is
// folded into the load address (an offset outside the buffer reads 0).
//
// fp32 operands are cut into NP bf16 pieces on their way into the matrix cores (split_device.h,
// split_patch.hip say what that does to the error and why v_mfma_f32_16x16x32_bf16).
//
// What bounds it: the matrix pipe where the reduction is long, the address arithmetic of the gather
// (one load per element) where B is an image seen through a window.
//
// Split of the work.  A block is MT rows and 128 columns, 32 reduction indices a step.
// 128 rows: a wave owns 16*TM rows and all 128 columns; its part of A is shared by nobody, goes from
// memory straight into registers in the layout of the matrix instruction (eight consecutive k of a
// row per lane) and is cut there.  B is shared by all waves: 16 (eight waves: 8) elements per thread and step are
// loaded one step ahead, cut once, and written to LDS as [piece][octet of k][column], from where an
// operand is one 16-byte read per piece.  Two LDS buffers, one barrier a step.
// 16 rows: every one of four waves takes all the rows and 32 columns.
#include <atomic>
#include <cstdio>
#include "cg_internal.h"
#include "igemm_device.h"
#include "split_device.h"

namespace cg {

namespace {

constexpr int KS = 32;                       // reduction indices per step
constexpr int OS = 128 + 2;                  // 16-byte units between octets in LDS (+2: octets on different banks)

using Rsrc = __amdgpu_buffer_rsrc_t;

__device__ __forceinline__ float ldf(Rsrc r, uint32_t voff, uint32_t soff = 0u)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ void ldq(Rsrc r, uint32_t voff, float *f)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) f[t] = __uint_as_float((uint32_t)v[t]);
}

// byte offset of reduction index k (< kend, else out of range) of a map that is a plain stride
__device__ __forceinline__ uint32_t k_offset(const IndexMap &m, uint32_t k, uint32_t kend)
{
    return k < kend ? (k * (uint32_t)m.s1 + (uint32_t)m.o0) * 4u : OOB_K;
}

// ---- A: eight consecutive k of row (16 i + lane % 16), octet lane / 16 -------------------------------
// A_QUAD: k is unit-stride and an aligned group of four one 16-byte load (4-byte aligned); what a group holds
// beyond K meets zeros of B.  A_ROWS: one load per element, neighbouring lanes on neighbouring rows, k a plain stride.
enum { A_ROWS = 0, A_QUAD = 1 };
template <int TM, int KIND> struct LoadA {
    uint32_t roff[TM];
    __device__ __forceinline__ void init(const Operand &op, uint32_t row0, uint32_t nrows, int lane)
    {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t row = row0 + (uint32_t)(i * 16 + (lane & 15));
            roff[i] = row < nrows ? (uint32_t)map_info(op.row, row).off * 4u : OOB_ROW;
        }
    }
    __device__ __forceinline__ void load(Rsrc r, const Operand &op, uint32_t k0, uint32_t kend, int lane, float (&f)[TM][8])
    {
        const uint32_t k = k0 + 8u * (uint32_t)(lane >> 4);
        if constexpr (KIND == A_QUAD) {
            const uint32_t ka = k_offset(op.k, k, kend), kb = k_offset(op.k, k + 4u, kend);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                ldq(r, roff[i] + ka, &f[i][0]);
                ldq(r, roff[i] + kb, &f[i][4]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint32_t ko = k_offset(op.k, k + (uint32_t)t, kend);
#pragma unroll
                for (int i = 0; i < TM; ++i) f[i][t] = ldf(r, roff[i] + ko);
            }
        }
    }
};

// ---- B: 128 columns x 32 k, NU tasks of eight k per thread (2 with four waves, 1 with eight) ------------------------------------------
// Columns along the lanes (an image seen through a window, a row-major matrix read across): wave w
// takes octet w % 4, lane the columns lane and lane + 64 (with eight waves one of them); k is uniform, its
// map runs on the scalar unit.
template <int NU, bool CHECK, bool LIN = false> struct LoadBRows {       // LIN: k is a plain stride
    uint32_t roff[NU];
    int32_t ra[NU], rb[NU];
    __device__ __forceinline__ static int column(int u, int wave, int lane) { return (NU == 2 ? u : wave >> 2) * 64 + lane; }
    __device__ __forceinline__ void init(const Operand &op, uint32_t row0, uint32_t nrows, int wave, int lane)
    {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const uint32_t row = row0 + (uint32_t)column(u, wave, lane);
            const Info q = map_info(op.row, row);
            roff[u] = row < nrows ? (uint32_t)q.off * 4u : OOB_ROW;
            ra[u] = q.a; rb[u] = q.b;
        }
    }
    // part P of four: k = 2P, 2P + 1 of the octet
    template <int P>
    __device__ __forceinline__ void load(Rsrc r, const Operand &op, uint32_t k0, uint32_t kend, int wave, int, float (&f)[NU][8])
    {
#pragma unroll
        for (int t = 2 * P; t < 2 * P + 2; ++t) {
            const uint32_t k = k0 + (uint32_t)(8 * (wave & 3) + t);
            const Info kq = LIN ? Info{} : map_info(op.k, k);
            const uint32_t ko = LIN ? k_offset(op.k, k, kend) : k < kend ? (uint32_t)kq.off * 4u : OOB_K;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                uint32_t voff = roff[u];
                if (CHECK) {
                    const bool ok = (uint32_t)(ra[u] + kq.a) < op.limA && (uint32_t)(rb[u] + kq.b) < op.limB;
                    voff = ok ? voff : OOB_ROW;
                }
                f[u][t] = ldf(r, voff, ko);
            }
        }
    }
    __device__ __forceinline__ static int unit(int u, int wave, int lane) { return (wave & 3) * OS + column(u, wave, lane); }
};

// k along the lanes, a plain unit stride: thread takes octet thread % 4 of columns thread / 4 and thread / 4 + 64
// as aligned quads.
template <int NU> struct LoadBK {
    uint32_t roff[NU];
    __device__ __forceinline__ void init(const Operand &op, uint32_t row0, uint32_t nrows, int wave, int lane)
    {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const uint32_t row = row0 + (uint32_t)(u * 64 + wave * 16 + (lane >> 2));
            roff[u] = row < nrows ? (uint32_t)map_info(op.row, row).off * 4u : OOB_ROW;
        }
    }
    template <int P>
    __device__ __forceinline__ void load(Rsrc r, const Operand &op, uint32_t k0, uint32_t kend, int, int lane, float (&f)[NU][8])
    {
        if constexpr (P % 2 == 0) {
            const uint32_t ka = k_offset(op.k, k0 + 8u * (uint32_t)(lane & 3) + 2u * P, kend);
#pragma unroll
            for (int u = 0; u < NU; ++u) ldq(r, roff[u] + ka, &f[u][2 * P]);
        }
    }
    __device__ __forceinline__ static int unit(int u, int wave, int lane) { return (lane & 3) * OS + u * 64 + wave * 16 + (lane >> 2); }
};

__device__ __forceinline__ Rsrc rsrc_of(const Operand &op, uint32_t g)
{
    const int64_t first = (int64_t)g * op.gstride + op.shift;
    return buffer_of(op.ptr + first, (uint64_t)((int64_t)op.elems - first) * 4u);
}

}  // namespace

template <int NP, int TM, int WM, class LA, class LB, bool SCATTER>
__global__ __launch_bounds__(WM == 8 ? 512 : 256, 2) void split_gemm_kernel(const IgemmProblem p)
{
    constexpr int WAVES = WM == 8 ? 8 : 4, WN = WAVES / WM, TN = 128 / (16 * WN), MT = WM * TM * 16, NT = 128, NU = 8 / WAVES;
    static_assert(WM * WN == WAVES && TN % 2 == 0, "four or eight waves");
    constexpr int PLANE = 4 * OS, BUF = NP * PLANE;
    extern __shared__ __attribute__((aligned(16))) v4u lds[];        // [2][NP][4][OS]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int q = lane >> 4, l16 = lane & 15;
    const uint32_t m0 = blockIdx.y * MT, n0 = blockIdx.x * NT;
    const uint32_t g = __builtin_amdgcn_readfirstlane(blockIdx.z / p.splits), sp = blockIdx.z - g * p.splits;
    const uint32_t kbeg = sp * p.k_per_split, kend = min(p.K, kbeg + p.k_per_split);
    const int ns = (int)((kend - kbeg + KS - 1) / KS);

    const Rsrc rA = rsrc_of(p.A, g), rB = rsrc_of(p.B, g);
    LA la;
    LB lb;
    la.init(p.A, m0 + (uint32_t)(wm * TM * 16), p.M, lane);
    lb.init(p.B, n0, p.N, wave, lane);

    // raw operands one step ahead of their cutting, pieces one step ahead of their use
    // (32 rows a wave and three pieces: the rows are cut in front of the products of their own step instead,
    // 24 registers less; two column tiles at a time then fit, without which the sums wait for each other)
    constexpr bool LATE = NP == 3 && TM == 2 && WM == 4;
    float ar[TM][8], br[NU][8];
    v4u ap[LATE ? 1 : 2][TM][NP], bc[NP];
    auto store_b = [&](int u, int buf) {
        const int at = buf * BUF + LB::unit(u, wave, lane);
#pragma unroll
        for (int k = 0; k < NP; ++k) lds[at + k * PLANE] = bc[k];
    };
    auto load_columns = [&](uint32_t k0) {
        static_for<0, 4>([&](auto PC) { lb.template load<decltype(PC)::value>(rB, p.B, k0, kend, wave, lane, br); });
    };

    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    load_columns(kbeg);
    la.load(rA, p.A, kbeg, kend, lane, ar);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        split8<NP>(br[u], bc);
        store_b(u, 0);
    }
    load_columns(kbeg + KS);
    if constexpr (!LATE) {
#pragma unroll
        for (int i = 0; i < TM; ++i) split8<NP>(ar[i], ap[0][i]);
        la.load(rA, p.A, kbeg + KS, kend, lane, ar);
    }

    using Step = MmaStep<NP, TM, TN, WM == 8 ? 2 : ColumnGroup<TM, TN>::G>;
    auto step = [&](auto PC, int s) {
        constexpr int par = LATE ? 0 : decltype(PC)::value, nxt = LATE ? 0 : par ^ 1;
        block_sync_lds();           // this step's columns are in LDS, and everyone is done with the other buffer
        const int rd = (s & 1) * BUF + q * OS + wn * TN * 16 + l16;
        const uint32_t k2 = kbeg + (uint32_t)(s + 2) * KS;
        if constexpr (LATE) {
#pragma unroll
            for (int i = 0; i < TM; ++i) split8<NP>(ar[i], ap[0][i]);
            la.load(rA, p.A, kbeg + (uint32_t)(s + 1) * KS, kend, lane, ar);
        }
        auto read_b = [&](int j, v4u (&pc)[NP]) {
#pragma unroll
            for (int k = 0; k < NP; ++k) pc[k] = lds[rd + j * 16 + k * PLANE];
        };
        // The next step's rows are cut (4*TM items, then one to fetch the rows after),
        // then its columns (4*NU), then the columns after are fetched (4).
        auto item = [&](auto OC) {
            constexpr int o = decltype(OC)::value, A1 = LATE ? -1 : 4 * TM, B0 = A1 + 1, B1 = B0 + 4 * NU;
            if constexpr (o < A1) split8_pair<NP>(ar[o / 4], o % 4, ap[nxt][o / 4]);
            else if constexpr (o == A1) la.load(rA, p.A, k2, kend, lane, ar);
            else if constexpr (o < B1) {
                constexpr int u = (o - B0) / 4, t = (o - B0) % 4;
                split8_pair<NP>(br[u], t, bc);
                if constexpr (t == 3) store_b(u, (s + 1) & 1);
            } else lb.template load<o - B1>(rB, p.B, k2, kend, wave, lane, br);
        };
        Step::run(ap[par], acc, read_b, Step::template spread<(LATE ? 0 : 4 * TM + 1) + 4 * NU + 4>(item));
    };
    for (int s = 0; s < ns; s += 2) {
        step(std::integral_constant<int, 0>{}, s);
        if (s + 1 < ns) step(std::integral_constant<int, 1>{}, s + 1);
    }
    if constexpr (NP == 3 && !SCATTER) {          // (scattered sums are looked at when they are stored)
        if (not_finite(acc)) sums_in_fp32(acc, [&](int j, auto &&add) {
            const uint32_t col = n0 + (uint32_t)((wn * TN + j) * 16 + l16);
            const Info r = map_info(p.B.row, col);
            const uint32_t boff = col < p.N ? (uint32_t)r.off * 4u : OOB_ROW;
            uint32_t aoff[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const uint32_t row = m0 + (uint32_t)((wm * TM + i) * 16 + l16);
                aoff[i] = row < p.M ? (uint32_t)map_info(p.A.row, row).off * 4u : OOB_ROW;
            }
            for (uint32_t k0 = kbeg; k0 < kend; k0 += 16u) {
                float a[4][TM], b[4];                   // 16 indices, their loads in flight together
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const uint32_t k = k0 + (uint32_t)(4 * v + q);
                    const Info kq = map_info(p.B.k, k);
                    const bool ok = k < kend && (!p.B.check || ((uint32_t)(r.a + kq.a) < p.B.limA && (uint32_t)(r.b + kq.b) < p.B.limB));
                    b[v] = ldf(rB, ok ? boff + (uint32_t)kq.off * 4u : OOB_ROW);
#pragma unroll
                    for (int i = 0; i < TM; ++i) a[v][i] = ldf(rA, aoff[i] + k_offset(p.A.k, k, kend));
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) add(a[v], b[v]);
            }
        });
    }
    store_columns<TM, TN, SCATTER>(p, acc, g, sp, m0 + (uint32_t)(wm * TM * 16), n0 + (uint32_t)(wn * TN * 16), p.N, lane);
}

namespace {

template <int NP, int TM, int WM, class LA, class LB, bool SCATTER>
int launch_cfg(const IgemmProblem &p, const char *modes, hipStream_t stream)
{
    constexpr int MT = WM * TM * 16;
    dim3 grid((p.N + 127) / 128, (p.M + MT - 1) / MT, p.groups * p.splits);
    if (grid.y > 65535u || grid.z > 65535u) return CG_EUNSUPPORTED;
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, NP == 3 ? "igemm_kernel<%dx128,%s,pieces>" : NP == 1 ? "igemm_kernel<%dx128,%s,pieces,bf16>" : "igemm_kernel<%dx128,%s,pieces,bf16x3>", MT, modes);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    constexpr size_t lds = (size_t)2 * NP * 4 * OS * 16;
    static_assert(2 * lds <= 160 * 1024, "two blocks of this tile do not fit the LDS of a compute unit");
    static std::atomic<bool> attr_set{false};      // raising the dynamic-LDS limit: once per kernel (repeating it is harmless)
    if (!attr_set.load(std::memory_order_acquire)) {
        CG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&split_gemm_kernel<NP, TM, WM, LA, LB, SCATTER>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((split_gemm_kernel<NP, TM, WM, LA, LB, SCATTER>), grid, dim3(WM == 8 ? 512 : 256), lds, stream, p);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

// At most one block a compute unit: eight waves of 16 rows instead of four of 32, so that two share a
// SIMD (a lone wave issues a step's instructions one after the other: 2.3 us a step).
template <int AK, template <int> class LB, bool ROWS16, bool WAVES8, bool SCATTER = false>
int launch_rows(const IgemmProblem &p, int mt, const char *modes, hipStream_t stream)
{
    if constexpr (ROWS16) {
        if (mt == 16) return launch_cfg<CG_NP, 1, 1, LoadA<1, AK>, LB<2>, SCATTER>(p, modes, stream);
    }
    if (mt != 128) return CG_EUNSUPPORTED;
    if constexpr (WAVES8) if ((uint64_t)((p.N + 127) / 128) * ((p.M + 127) / 128) * p.groups * p.splits <= 256)
        return launch_cfg<CG_NP, 1, 8, LoadA<1, AK>, LB<1>, SCATTER>(p, modes, stream);
    return launch_cfg<CG_NP, 2, 4, LoadA<2, AK>, LB<2>, SCATTER>(p, modes, stream);
}
template <int NU> using BRowsCheck = LoadBRows<NU, true>;
template <int NU> using BRowsPlain = LoadBRows<NU, false>;
template <int NU> using BRowsLin = LoadBRows<NU, false, true>;

}  // namespace

// This file is compiled once per number of pieces (CG_NP), in parallel.  16 or 128 rows; b_quads: B as aligned quads
// of k, else rows along the lanes.
#define CG_CAT_(a, b) a##b
#define CG_CAT(a, b) CG_CAT_(a, b)
int CG_CAT(split_gemm_, CG_NP)(const IgemmProblem &p, int mt, bool a_quads, bool b_quads, hipStream_t stream)
{
    const bool bc = p.B.check != 0;
    const bool a_lin = p.A.k.d1.d == 1 && p.A.k.d2.d == 1, b_lin = p.B.k.d1.d == 1 && p.B.k.d2.d == 1;
    const char modes[4] = {a_quads ? '4' : 'r', b_quads ? '4' : 'r', bc ? 'c' : '-', 0};
    if (!a_lin || p.B.k.r1_lim) return CG_EUNSUPPORTED;
    // (padding means an image, and images get 128 rows only where there are blocks for more than one a compute unit)
    if (b_quads) return a_quads && b_lin && !bc ? launch_rows<A_QUAD, LoadBK, false, true>(p, mt, modes, stream) : CG_EUNSUPPORTED;
    // (scattered rows: strided backward-data, whose columns are an image's cells under a window)
    if (p.c_scatter) return a_quads && bc ? launch_rows<A_QUAD, BRowsCheck, true, false, true>(p, mt, modes, stream) : CG_EUNSUPPORTED;
    if (a_quads)
        return bc ? launch_rows<A_QUAD, BRowsCheck, true, false>(p, mt, modes, stream)
                  : launch_rows<A_QUAD, BRowsPlain, true, true>(p, mt, modes, stream);
    return bc || !b_lin ? CG_EUNSUPPORTED : launch_rows<A_ROWS, BRowsLin, true, true>(p, mt, modes, stream);
}

}  // namespace cg
