// Device code shared by the matrix kernels: buffer descriptors, unrolled loops, the epilogue.
#pragma once
#include <type_traits>
#include <utility>
#include "cg_internal.h"

namespace cg {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) float lds_float;
typedef uint32_t BufferRsrc __attribute__((ext_vector_type(4)));   // the four descriptor words of a raw buffer

namespace {

// Offsets that no buffer descriptor of this library covers (descriptors span < 0x7fffff00 bytes).
// Their sum does not wrap, and either one added to a valid offset (< 2^31) stays out of range.
constexpr uint32_t OOB_ROW = 0x80000000u, OOB_K = 0x7fffff00u;
constexpr uint64_t kMaxBufferBytes = 0x7fffff00ull;

template <int B, class F, int... Is>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, B + Is>{}), ...);
}
template <int B, int E, class F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl<B>(f, std::make_integer_sequence<int, (E > B ? E - B : 0)>{});
}

// Buffer descriptor over the part of an operand's tensor that starts at group g (+ the shift that
// keeps per-index offsets non-negative).  igemm_launch has checked that the span fits the format.
// Words: base address (48 bits, stride 0), number of bytes, format word of a raw dword buffer.
__device__ __forceinline__ BufferRsrc operand_rsrc(const Operand &op, uint32_t g)
{
    const int64_t first = (int64_t)g * op.gstride + op.shift;
    const uint64_t base = (uint64_t)reinterpret_cast<uintptr_t>(op.ptr) + (uint64_t)(first * 4);
    const uint32_t bytes = (uint32_t)(((int64_t)op.elems - first) * 4);
    BufferRsrc r;       // wave-uniform by construction; readfirstlane pins the words to scalar registers
    r.x = __builtin_amdgcn_readfirstlane((uint32_t)base);
    r.y = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
    r.z = __builtin_amdgcn_readfirstlane(bytes);
    r.w = 0x00020000u;
    return r;
}

// Epilogue of the matrix kernels: a wave's TM x TN accumulator tiles, whose first row / column
// are (mw, nw), go to C (columns below n_end) with bias, rectifier, gate and accumulation applied.
// Accumulator register r of lane (h, li) holds C row 8*(r/4) + 4*h + r%4, column li of its 32x32
// sub-tile: stored from there, every store instruction would write 4 bytes per lane in runs of
// 128 bytes.  Instead each 32-row slab of the wave's tile is turned around in LDS (`wlds`, private
// to the wave, EpiLds<TN>::FLOATS floats, free once the block has left the K loop) so that a lane
// owns four consecutive columns of a row and a store instruction writes whole runs of 32*TN
// columns, 16 bytes per lane (4-byte aligned).  Columns whose C offsets are not consecutive
// (a pixel tile that crosses into the next image) or that reach beyond n_end go one by one.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

template <int TN> struct EpiLds {
    static constexpr int W = TN * 32, LS = W + 8, FLOATS = 32 * LS;
};

// Sum (m, n) of a strided backward-data problem by one thread, over the taps that row m's phase has; dy reads as zero outside
// its plane, as everywhere.
__device__ __forceinline__ float sum_of_taps(const StridedTaps &t, const IndexMap &rows, const IndexMap &cols, uint32_t g, uint32_t m, uint32_t n)
{
    const uint32_t c = fdiv(m, rows.d1), ph = m - c * rows.d1.d, rh = fdiv(ph, rows.d2), rw = ph - rh * rows.d2.d;
    const uint32_t img = fdiv(n, cols.d1), cell = n - img * cols.d1.d, i = fdiv(cell, cols.d2), j = cell - i * cols.d2.d;
    float s = 0.f;
    for (int k = 0; k < t.Mg; ++k) {
        const size_t ch = (size_t)g * t.Mg + k;
        const float *y = t.dy + ((size_t)img * t.M + ch) * t.OH * t.OW, *w = t.w + (ch * t.Cg + c) * t.KH * t.KW;
        for (int kh = (int)rh, oh = (int)i; kh < t.KH; kh += t.sh, --oh)
            for (int kw = (int)rw, ow = (int)j; kw < t.KW; kw += t.sw, --ow) {
                float a = (uint32_t)oh < (uint32_t)t.OH && (uint32_t)ow < (uint32_t)t.OW ? y[oh * t.OW + ow] : 0.f, b = w[kh * t.KW + kw];
                if (t.bf16) { a = (float)(__bf16)a; b = (float)(__bf16)b; }
                s = fmaf(a, b, s);
            }
    }
    return s;
}

// The kernel's first argument, read where it lies: in code that hardly ever runs, so that the compiler does not keep its
// fields in scalar registers from the start of the kernel on, and spill others for them.
template <class Args> __device__ __forceinline__ const Args &first_argument()
{
    auto at = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const Args *)at;
}

// Element (m, n) of a strided backward-data problem (the kernel's first argument), whose sum came out as s.
__device__ __forceinline__ void store_scattered(uint32_t g, uint32_t m, uint32_t n, float s)
{
    const IgemmProblem &p = first_argument<IgemmProblem>();
    if (m >= p.M || n >= p.N) return;
    const Info ri = map_info(p.c_row, m), ci = map_info(p.c_col, n);
    if (!((uint32_t)(ri.a + ci.a) < p.c_limA && (uint32_t)(ri.b + ci.b) < p.c_limB)) return;
    const int64_t at = (int64_t)g * p.c_gstride + ri.off + ci.off;
    if (p.gate && !(p.gate[at] > 0.f)) s = 0.f;
    else if (!__builtin_isfinite(s)) s = sum_of_taps(p.taps, p.c_row, p.c_col, g, m, n);
    p.c_ptr[at] = p.accumulate ? p.c_ptr[at] + s : s;
}

// A slab is SR rows, the tile NS slabs of W columns; turn(i) writes slab i of the accumulators to wlds
// as rows of W + 8 floats.  PB: row groups (one store instruction each) per batch.
template <int SR, int NS, int W, int PB, bool PLAIN, class Turn>
__device__ __forceinline__ void store_slabs(const IgemmProblem &p, Turn &&turn, uint32_t g, uint32_t sp, uint32_t mw,
                                            uint32_t nw, uint32_t n_end, int lane, float *wlds)
{
    constexpr int LS = W + 8, QR = W / 4, RPI = 64 / QR;      // quads per row, rows per instruction
    constexpr int NRG = SR / RPI;                   // row groups of a slab
    static_assert(64 % QR == 0 && SR % RPI == 0 && NRG % PB == 0, "whole row groups and batches");
    constexpr int NBS = NRG / PB, NBT = NS * NBS;   // batches per slab and of the whole tile
    const int qd = lane % QR, rr = lane / QR;
    float *c_base = p.c_ptr + (int64_t)g * p.c_gstride + (int64_t)sp * p.c_split_stride;
    const float *bias = p.bias_mode ? p.bias + (int64_t)g * p.bias_gstride : nullptr;
    const float *gate = (!PLAIN && p.gate) ? p.gate + (int64_t)g * p.c_gstride : nullptr;
    const bool accumulate = !PLAIN && p.accumulate, scatter = !PLAIN && p.c_scatter;
    const uint32_t n = nw + 4u * (uint32_t)qd;
    int32_t off[4], ca[4], cb[4];
    float bcol[4];
    uint32_t okbits = 0u;       // bit e: column n + e exists (kept in a vector register: lane masks are scalar-register pairs)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool ok = n + (uint32_t)e < n_end;
        const Info ci = map_info(p.c_col, ok ? n + (uint32_t)e : 0u);
        off[e] = ok ? ci.off : 0;
        ca[e] = ci.a; cb[e] = ci.b;
        bcol[e] = (p.bias_mode == 2 && ok) ? bias[n + (uint32_t)e] : 0.f;
        okbits |= ok ? 1u << e : 0u;
    }
    const bool quad = !scatter && (okbits & 8u) && off[1] == off[0] + 1 && off[2] == off[0] + 2 && off[3] == off[0] + 3;
    // Loads and stores leave the vector-memory counter in the order they were issued, so a load
    // issued behind stores is waited for together with them, a whole write latency.  Hence what a
    // batch of row groups reads from global memory (per-row bias, gate, C when accumulating) is
    // requested one batch ahead, before the stores of the batch in front of it: the wait for it
    // then leaves those stores outstanding.
    struct Batch {
        f4u gt[PB], old[PB];
        float brow[PB];
        int32_t roff[PB];
        uint32_t okm;           // bit 4u+e: element e of row group u is inside C (a vector register, not 16 lane masks)
    };
    Batch bt[2];
    auto prepare = [&](auto BC, Batch &t) {
        constexpr int b = decltype(BC)::value, i = b / NBS, p0 = (b % NBS) * PB;
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int row = (p0 + u) * RPI + rr;
            const uint32_t m = mw + (uint32_t)(i * SR + row);
            t.gt[u] = f4u{1.f, 1.f, 1.f, 1.f};
            t.old[u] = f4u{0.f, 0.f, 0.f, 0.f};
            t.roff[u] = (int32_t)m * p.c_row_stride;
            t.brow[u] = (p.bias_mode == 1 && m < p.M) ? bias[m] : 0.f;
            uint32_t bits = m < p.M ? okbits : 0u;
            if (scatter && m < p.M) {
                const Info ri = map_info(p.c_row, m);
                t.roff[u] = ri.off;
                bits = 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    bits |= ((okbits >> e & 1u) && (uint32_t)(ri.a + ca[e]) < p.c_limA && (uint32_t)(ri.b + cb[e]) < p.c_limB) ? 1u << e : 0u;
            }
            if (u == 0) t.okm = 0u;
            t.okm |= bits << (4 * u);
            if (m < p.M && (gate || accumulate)) {
                const int32_t row_off = t.roff[u];
                if (quad) {
                    if (gate) t.gt[u] = *reinterpret_cast<const f4u *>(gate + row_off + off[0]);
                    if (accumulate) t.old[u] = *reinterpret_cast<const f4u *>(c_base + row_off + off[0]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (gate && (bits >> e & 1u)) t.gt[u][e] = gate[row_off + off[e]];
                        if (accumulate && (bits >> e & 1u)) t.old[u][e] = c_base[row_off + off[e]];
                    }
                }
            }
        }
    };
    prepare(std::integral_constant<int, 0>{}, bt[0]);
    static_for<0, NBT>([&](auto BC) {
        constexpr int b = decltype(BC)::value, i = b / NBS, p0 = (b % NBS) * PB;
        if constexpr (b % NBS == 0) {
            turn(std::integral_constant<int, i>{});
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the slab is in LDS (one wave: no barrier)
        }
        float4 q[PB];
#pragma unroll
        for (int u = 0; u < PB; ++u) q[u] = *reinterpret_cast<const float4 *>(wlds + ((p0 + u) * RPI + rr) * LS + 4 * qd);
        if constexpr (b + 1 < NBT) prepare(std::integral_constant<int, b + 1>{}, bt[(b + 1) & 1]);
        const Batch &t = bt[b & 1];
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int row = (p0 + u) * RPI + rr;
            const uint32_t m = mw + (uint32_t)(i * SR + row);
            if (m >= p.M || !(okbits & 1u)) continue;
            float val[4] = {q[u].x + bcol[0], q[u].y + bcol[1], q[u].z + bcol[2], q[u].w + bcol[3]};
            const float br = t.brow[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                val[e] += br;
                if (p.relu) val[e] = fmaxf(val[e], 0.f);
            }
            const int32_t row_off = t.roff[u];
            if constexpr (!PLAIN) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!(t.gt[u][e] > 0.f)) val[e] = 0.f;
            }
            f4u out = {val[0], val[1], val[2], val[3]};
            if (accumulate) out += t.old[u];
            if (quad) {
                *reinterpret_cast<f4u *>(c_base + row_off + off[0]) = out;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (t.okm >> (4 * u + e) & 1u) c_base[row_off + off[e]] = out[e];
            }
        }
        if constexpr (b % NBS == NBS - 1)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // slab read before the next one overwrites it
    });
}

// Does any lane of the wave hold a sum that is an infinity or a NaN?
template <class Tile, int TM, int TN> __device__ __forceinline__ bool not_finite(const Tile (&acc)[TM][TN])
{
    float z[4] = {};            // (a chain of its own for every fourth element: an addition waits for the one before it)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < (int)(sizeof(Tile) / 4); ++e) z[e % 4] = fmaf(acc[i][j][e], 0.f, z[e % 4]);
    return __builtin_expect(__any(!((z[0] + z[1]) + (z[2] + z[3]) == 0.f)), 0);
}

// wave tiles of 32x32 accumulators.  SCATTER: the kernel instance runs problems with c_scatter.  (Only the second look at their
// sums is left out of the others: with all of it left out, the patch kernel took 135.7 us, not 134.5, for backward-data of 256
// images of 13x13, 384 -> 256 channels, 3x3, two groups, in two pieces.)
template <int TM, int TN, bool SCATTER>
__device__ __forceinline__ void store_tile(const IgemmProblem &p, const v16f (&acc)[TM][TN], uint32_t g, uint32_t sp,
                                           uint32_t mw, uint32_t nw, uint32_t n_end, int lane, float *wlds)
{
    constexpr int LS = EpiLds<TN>::LS, NRG = 32 / (64 / (TN * 8));
    constexpr int PB = TM >= 4 ? 2 : NRG < 4 ? NRG : 4;      // fewer beside 128 accumulator registers
    const int h = lane >> 5, li = lane & 31;
    auto turn = [&](auto IC) {
        constexpr int i = decltype(IC)::value;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) wlds[((r >> 2) * 8 + h * 4 + (r & 3)) * LS + j * 32 + li] = acc[i][j][r];
    };
    if (SCATTER && p.c_scatter && not_finite(acc)) {
        // element by element: an infinity may have met the zero of a tap that does not exist
        static_for<0, TM>([&](auto IC) {
            turn(IC);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            for (int at = lane; at < 32 * TN * 32; at += 64) {
                const uint32_t r = (uint32_t)at / (TN * 32), c = (uint32_t)at % (TN * 32);
                store_scattered(g, mw + (uint32_t)(decltype(IC)::value * 32) + r, nw + c, wlds[r * LS + c]);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        });
        return;
    }
    if (!p.gate && !p.accumulate && !p.c_scatter) store_slabs<32, TM, TN * 32, PB, true>(p, turn, g, sp, mw, nw, n_end, lane, wlds);
    else store_slabs<32, TM, TN * 32, PB, false>(p, turn, g, sp, mw, nw, n_end, lane, wlds);
}

// Epilogue of the kernels whose wave tiles are 16x16 accumulators with the columns on the registers:
// lane (q = lane / 16, l = lane % 16) holds row l and the columns 4q .. 4q+3 of a sub-tile and stores
// them as one 16-byte access (4-byte aligned), 16 rows x 64 bytes an instruction, without a turn through LDS.
// What is read (gate, C when accumulating) is requested for JB column tiles at once, in front of their stores.
// Columns whose offsets are not consecutive (a pixel tile that crosses into the next image), that reach beyond n_end
// or are scattered go one by one.
typedef float v4f __attribute__((ext_vector_type(4)));
// at(c): the four columns that start at column c of the wave's tile, as the first one's index in C and how many of them
// exist; they follow one another in C.
struct Columns { uint32_t n, cnt; };
template <int TM, int TN, bool PLAIN, class At>
__device__ __forceinline__ void store_columns_impl(const IgemmProblem &p, const v4f (&acc)[TM][TN], uint32_t g, uint32_t sp,
                                                   uint32_t mw, int lane, At &&at)
{
    constexpr int JB = PLAIN ? 1 : TN < 4 ? TN : TM >= 3 ? 2 : 4;
    const int q = lane >> 4, l16 = lane & 15;
    float *c_base = p.c_ptr + (int64_t)g * p.c_gstride + (int64_t)sp * p.c_split_stride;
    const float *bias = p.bias_mode ? p.bias + (int64_t)g * p.bias_gstride : nullptr;
    const float *gate = (!PLAIN && p.gate) ? p.gate + (int64_t)g * p.c_gstride : nullptr;
    const bool accumulate = !PLAIN && p.accumulate, scatter = !PLAIN && p.c_scatter, linear = p.c_col.d1.d == 1;
    int32_t roff[TM], ra[TM], rb[TM];
    float brow[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t m = mw + (uint32_t)(i * 16 + l16);
        roff[i] = m < p.M ? (int32_t)m * p.c_row_stride : -1;
        ra[i] = rb[i] = 0;
        brow[i] = (p.bias_mode == 1 && m < p.M) ? bias[m] : 0.f;
        if (scatter && m < p.M) {
            const Info ri = map_info(p.c_row, m);
            roff[i] = ri.off; ra[i] = ri.a; rb[i] = ri.b;
        }
    }
    static_for<0, TN / JB>([&](auto BC) {
        constexpr int j0 = decltype(BC)::value * JB;
        int32_t off[JB];
        uint32_t first[JB], cnt[JB];    // this lane's four columns, how many of them exist
        bool quad[JB];
        v4f bcol[JB], gt[JB][TM], old[JB][TM];
#pragma unroll
        for (int u = 0; u < JB; ++u) {
            const Columns four = at((j0 + u) * 16 + 4 * q);
            const uint32_t n = first[u] = four.n;
            cnt[u] = four.cnt;
            off[u] = 0;
            quad[u] = false;
            bcol[u] = v4f{0.f, 0.f, 0.f, 0.f};
            if (cnt[u]) {
                off[u] = linear ? (int32_t)n * p.c_col.s1 + p.c_col.o0 : map_info(p.c_col, n).off;
                if (cnt[u] == 4u && !scatter) {
                    const int32_t o3 = linear ? off[u] + 3 * p.c_col.s1 : map_info(p.c_col, n + 3u).off;
                    quad[u] = o3 == off[u] + 3;
                }
                if (p.bias_mode == 2)
#pragma unroll
                    for (int e = 0; e < 4; ++e) bcol[u][e] = (uint32_t)e < cnt[u] ? bias[n + (uint32_t)e] : 0.f;
            }
            if constexpr (!PLAIN) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    gt[u][i] = v4f{1.f, 1.f, 1.f, 1.f};
                    old[u][i] = v4f{0.f, 0.f, 0.f, 0.f};
                    if (quad[u] && mw + (uint32_t)(i * 16 + l16) < p.M) {
                        if (gate) gt[u][i] = *reinterpret_cast<const f4u *>(gate + roff[i] + off[u]);
                        if (accumulate) old[u][i] = *reinterpret_cast<const f4u *>(c_base + roff[i] + off[u]);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < JB; ++u) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const bool row_ok = mw + (uint32_t)(i * 16 + l16) < p.M;
                v4f v = acc[i][j0 + u] + bcol[u] + v4f{brow[i], brow[i], brow[i], brow[i]};
                if (p.relu)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
                if (quad[u]) {
                    if constexpr (!PLAIN) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = gt[u][i][e] > 0.f ? v[e] : 0.f;
                        if (accumulate) v += old[u][i];
                    }
                    if (row_ok) *reinterpret_cast<f4u *>(c_base + roff[i] + off[u]) = v;
                } else if (row_ok && cnt[u]) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if ((uint32_t)e >= cnt[u]) continue;
                        const Info ci = map_info(p.c_col, first[u] + (uint32_t)e);
                        if (scatter && !((uint32_t)(ra[i] + ci.a) < p.c_limA && (uint32_t)(rb[i] + ci.b) < p.c_limB)) continue;
                        const int32_t to = roff[i] + ci.off;
                        float x = v[e];
                        if (gate && !(gate[to] > 0.f)) x = 0.f;
                        if (accumulate) x += c_base[to];
                        c_base[to] = x;
                    }
                }
            }
        }
    });
}

template <int TM, int TN, bool SCATTER, class At>
__device__ __forceinline__ void store_columns_at(const IgemmProblem &p, const v4f (&acc)[TM][TN], uint32_t g, uint32_t sp, uint32_t mw, int lane, At &&at)
{
    if (SCATTER && p.c_scatter && not_finite(acc)) {
        // element by element: an infinity may have met the zero of a tap that does not exist
        const int q = lane >> 4, l16 = lane & 15;
#pragma unroll 1
        for (int k = 0; k < TM * TN * 4; ++k) {
            float s = 0.f;                       // (the accumulators stay in registers: no index into them)
            static_for<0, TM * TN * 4>([&](auto KC) {
                constexpr int c = decltype(KC)::value;
                s = k == c ? acc[c / 4 % TM][c / 4 / TM][c % 4] : s;
            });
            const Columns four = at(k / 4 / TM * 16 + 4 * q);
            if ((uint32_t)(k % 4) < four.cnt) store_scattered(g, mw + (uint32_t)(k / 4 % TM * 16 + l16), four.n + (uint32_t)(k % 4), s);
        }
        return;
    }
    if (!p.gate && !p.accumulate && !p.c_scatter) store_columns_impl<TM, TN, true>(p, acc, g, sp, mw, lane, at);
    else store_columns_impl<TM, TN, false>(p, acc, g, sp, mw, lane, at);
}
// columns nw, nw + 1, ... below n_end
template <int TM, int TN, bool SCATTER>
__device__ __forceinline__ void store_columns(const IgemmProblem &p, const v4f (&acc)[TM][TN], uint32_t g, uint32_t sp,
                                              uint32_t mw, uint32_t nw, uint32_t n_end, int lane)
{
    store_columns_at<TM, TN, SCATTER>(p, acc, g, sp, mw, lane, [&](int c) {
        const uint32_t n = nw + (uint32_t)c;
        return Columns{n, n < n_end ? min(4u, n_end - n) : 0u};
    });
}

// Sum of dy[n][m][0..P) over the images n_beg..n_end-1, by one block (T threads, a power of two; `red` a float each);
// thread 0 returns it.
// The (image, group of four pixels) pairs are spread over the threads, each moving 16 bytes
// (4-byte aligned: planes of an odd pixel count start anywhere) with eight loads in flight: a block that rides beside the K-slice sums
// of a small layer is what its launch waits for, a turn of loads after the other (32 images of 28x28, 192 -> 96 channels 1x1, whole pass
// 31.4 us with four, 30.4 with eight).
__device__ __forceinline__ float bias_channel_sum(const float *__restrict__ dy, int M, int P, int m, int n_beg, int n_end,
                                                  FastDiv divQP, uint32_t T, float *red)
{
    const uint32_t QP = divQP.d, total = (uint32_t)(n_end - n_beg) * QP;
    float s = 0.f;
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += T * 8) {
        f4u v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = i0 + u * T;
            v[u] = f4u{0.f, 0.f, 0.f, 0.f};
            if (i < total) {
                const uint32_t n = fdiv(i, divQP), qd = i - n * QP;
                const float *src = dy + ((size_t)(n_beg + (int)n) * M + m) * P + 4 * qd;
                const int rem = P - 4 * (int)qd;
                if (rem >= 4) v[u] = __builtin_nontemporal_load(reinterpret_cast<const f4u *>(src));
                else {
                    v[u].x = src[0];
                    if (rem > 1) v[u].y = src[1];
                    if (rem > 2) v[u].z = src[2];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (v[u].x + v[u].y) + (v[u].z + v[u].w);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = (int)T / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

}  // namespace
}  // namespace cg
