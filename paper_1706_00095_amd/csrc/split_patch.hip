// Convolutions from raw image rows on the bf16 matrix instructions: forward, stride-1 backward-data
// and strided backward-data (as a stride-1 problem over dy).  See PatchGeom in cg_internal.h for the
// geometry.  One kernel serves the three arithmetics of cg.h by the number of bf16 pieces an fp32
// operand is cut into on its way into the matrix cores:
//   NP = 3 (CG_MATH_FP32):   x = h + m + l, h = bf16(x), m = bf16(x - h), l = bf16(x - h - m): exact, 24 bits
//                            (of x times 2^24: split_device.h).  Six products l*h + h*l + m*m + m*h + h*m + h*h,
//                            small ones first; what is dropped (m*l, l*m, l*l) is 2^-29 of a product at the median, at
//                            most 2^-24.  A step's products are added up from zero and then to the accumulator
//                            (MmaStep, OWN): the error against 64 bits is 4.2e-8 where the fp32 instruction has
//                            1.7e-7 (256 images, 256 channels of 13x13, 384 rows, 3x3), in 355 us instead of 591.
//                            Sums that end as an infinity or a NaN are computed anew in fp32 (sums_in_fp32): 523 us for
//                            the same pass with one infinity in its input, 1.8 ms where every sum is one.
//   NP = 2 (CG_MATH_BF16X3): x = h + l, three products.
//   NP = 1 (CG_MATH_BF16):   x = h.
//
// What bounds it: the matrix pipe.  v_mfma_f32_16x16x32_bf16 rather than 32x32x16: on random operands
// the former holds 1970 TFLOP/s, the latter 1700 (power; both 2450 on zeros), with the same LDS traffic
// for the same wave tile.  Power bounds the rest too: the clock stands at 2.0 GHz of 2.4 with the pipe 53 % busy, and what a
// variant leaves out comes off the time whether or not it overlapped (256 images of 13x13, 256 -> 384 channels 3x3, fp32 filters, 375 us: cutting
// them 55, bringing and cutting the patch 26, reading fragments 35, own sums 20).  So the filters come cut.
//
// Split of the work.  A block is four waves and 128 pixels; wave w owns 16*TM rows of its own and
// ALL 128 pixels.  So the filters are shared by nobody and need no LDS: a lane fetches its eight
// consecutive reduction indices of a row straight from L2 (the filter copy is laid out so that a wave's load is
// contiguous), a 16-byte load per piece, cut once by the kernel that makes the copy: every pixel tile cut the same values
// again before (375 -> 346 us there; 5x5 of 48 rows 670 -> 568).  Where a workspace has no room for three pieces
// (half as much again as the values), or fp32 is the faster form (patch_wants_pieces), the copy is fp32, two loads, and a lane
// cuts its values in registers.  The
// image patch is cut once per block, on its way into LDS, 32 channels at a time, as
// [piece][octet of channels][slot][8 channels]: a lane's operand is then one 16-byte read per piece
// whose address runs over consecutive slots, and one patch serves every tap.  There is no barrier
// inside the taps of a channel group: waves of a block drift, and those of two blocks share a SIMD, so
// one cuts filters while the other multiplies.
// A step multiplies two units of 16 reduction indices (a unit = one tap of 16 channels): both channel
// halves of a tap, or, for a last group of only 16 channels, two taps of it.
#include <atomic>
#include <cstdio>
#include "cg_internal.h"
#include "igemm_device.h"
#include "split_device.h"

namespace cg {

namespace {

typedef uint32_t v2u __attribute__((ext_vector_type(2)));      // four bf16

template <int NP, int TM, int WK, int NSL, bool CUT> struct PatchLds {
    // In 16-byte units; behind the octets of every piece lies one unit of zeros.  Four octets of channels are a group's; where
    // registers allow no third block and two more octets find room beside another block, the octets of the groups go round: a
    // group's first two are stored while the group before is multiplied, and a wave holds 16 values on their way, not 32, which is
    // what lets 192-row tiles take filters in pieces (256 images of 13x13, 3x3, two groups, 384 -> 384 channels, backward-data 331 -> 285 us
    // with it; fp32 filters 310).  Beside fp32 filters it is no gain (310 / 321).
    static constexpr bool RING = CUT && NSL == 4 && TM >= 2 && WK == 1;
    static constexpr int OCTETS = RING ? 6 : 4, SLOTS = NSL * 64, ZERO = OCTETS * SLOTS, PLANE = ZERO + 1;
    static constexpr size_t BYTES = (size_t)NP * PLANE * 16;
};

}  // namespace

// WM x WN x WK waves: rows x pixels x steps (WK = 2: two waves share a tile, each takes every other
// step, and their sums meet in LDS at the end: for row counts too small to give each wave its own).
// SCATTER: strided backward-data (c_scatter).  CUT: the filter copy holds pieces, else fp32 (only with three pieces).
template <int NP, int TM, int WM, int WK, int NSL, bool SCATTER, bool CUT>
__global__ __launch_bounds__(256, 2) void split_patch_kernel(const IgemmProblem p)
{
    constexpr int WN = 4 / (WM * WK), TN = 128 / (16 * WN), MT = WM * TM * 16, NT = 128;
    static_assert(WM * WN * WK == 4 && TN % 2 == 0, "four waves");
    static_assert(CUT || NP == 3, "fewer pieces take no more room than the values");
    using L = PatchLds<NP, TM, WK, NSL, CUT>;
    extern __shared__ __attribute__((aligned(16))) v4u lds[];        // the pieces of the patch (PatchLds)

    const PatchGeom &pg = p.patch;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = (wave / WM) % WN, wk = wave / (WM * WN);
    const uint32_t m0 = blockIdx.y * MT, g = blockIdx.z;
    const int KK = pg.KH * pg.KW, ncb16 = (int)(pg.Cred + 15) / 16, ngrp = (ncb16 + 1) / 2;
    // this block's pixels: n0..n1, or the rectangle of image bA from (ty0, tx0) on
    const uint32_t P = pg.divP.d;
    uint32_t n0 = 0, n1 = 0, bA, ty0 = 0, tx0 = 0;
    const uint32_t tile = blockIdx.x + pg.tile0;
    const int rs = pg.rect_shift;
    if (pg.tiles_per_img) {
        bA = fdiv(tile, pg.divTpi);
        const uint32_t ti = tile - bA * pg.divTpi.d;
        if (rs) {
            const uint32_t ry = fdiv(ti, pg.divTx);
            ty0 = ry * (uint32_t)(NT >> rs);
            tx0 = (ti - ry * pg.divTx.d) << rs;
        } else {
            n0 = bA * P + ti * NT;
            n1 = min(n0 + NT - 1, (bA + 1) * P - 1);
        }
    } else {
        n0 = tile * NT;
        n1 = min(n0 + NT - 1, p.N - 1);
        bA = fdiv(n0, pg.divP);
    }
    // pixel i of the block: image, row, column, is it one
    struct Pixel { uint32_t b, oy, ox; bool ok; };
    auto pixel = [&](int i) {
        if (rs) {
            const uint32_t oy = ty0 + (uint32_t)(i >> rs), ox = tx0 + (uint32_t)(i & ((1 << rs) - 1));
            return Pixel{bA, oy, ox, oy < (uint32_t)pg.OHo && ox < (uint32_t)pg.OWo};
        }
        const uint32_t n = n0 + (uint32_t)i, b = fdiv(n, pg.divP), rem = n - b * P, oy = fdiv(rem, pg.divOW);
        return Pixel{b, oy, rem - oy * pg.divOW.d, n <= n1};
    };

    const auto rsrcA = buffer_of(p.A.ptr + (int64_t)g * p.A.gstride, (p.A.elems - (uint64_t)g * p.A.gstride) * 4);
    const auto rsrcB = buffer_of(pg.src + (int64_t)g * pg.gstride, (pg.src_elems - (uint64_t)g * pg.gstride) * 4);

    // ---- where this block's pixels sit: images bA..bB, pixel rows oyA (in bA) .. oyB (in bB) -------
    const uint32_t oyA = rs ? ty0 : fdiv(n0 - bA * P, pg.divOW), bB = rs ? bA : fdiv(n1, pg.divP);
    const uint32_t oyB = rs ? ty0 + (uint32_t)(NT >> rs) - 1u : fdiv(n1 - bB * P, pg.divOW);
    // slots of the first image's segment; later images start at R0 + (d-1)*Rfull
    const int32_t R0 = (int32_t)((((bA == bB) ? oyB : (uint32_t)pg.OHo - 1) - oyA) * pg.s + pg.KH) * pg.Wp;

    // global byte offset of every patch slot this lane loads (or out of range: padding, unused slots)
    const int chunk0 = L::RING ? 2 * (wave / 2) : 0;
    uint32_t voff[L::RING ? 2 : NSL];
#pragma unroll
    for (int e = 0; e < (L::RING ? 2 : NSL); ++e) {
        const int32_t j = (chunk0 + e) * 64 + lane;
        const uint32_t d = j < R0 ? 0u : 1u + fdiv((uint32_t)(j - R0), pg.divRfull);
        const int32_t local = j - (d == 0 ? 0 : R0 + (int32_t)(d - 1) * pg.Rfull);
        const uint32_t r = fdiv((uint32_t)local, pg.divWp), c = (uint32_t)local - r * (uint32_t)pg.Wp;
        const uint32_t b = bA + d, oylo = d == 0 ? oyA : 0u;
        const uint32_t oyhi = b == bB ? oyB : (uint32_t)pg.OHo - 1;
        const int32_t sy = (int32_t)(oylo * pg.s) + pg.oy0 + (int32_t)r, sx = (int32_t)(tx0 * pg.s) + pg.ox0 + (int32_t)c;
        const bool ok = b <= bB && r < (oyhi - oylo) * pg.s + pg.KH && (uint32_t)sy < (uint32_t)pg.Hs &&
                        (uint32_t)sx < (uint32_t)pg.Ws;
        voff[e] = ok ? (uint32_t)((int32_t)b * pg.img_stride + sy * pg.Ws + sx) * 4u : OOB_ROW;
    }

    const int q = lane >> 4, l16 = lane & 15;
    const bool second = q >= 2;                 // this lane's eight reduction indices belong to a step's second unit
    // slot of this lane's pixels (their windows' first element)
    int32_t sig[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const Pixel px = pixel((wn * TN + j) * 16 + l16);
        const uint32_t d = px.b - bA, oylo = d == 0 ? oyA : 0u;
        const int32_t sg = (d == 0 ? 0 : R0 + (int32_t)(d - 1) * pg.Rfull) + (int32_t)((px.oy - oylo) * pg.s) * pg.Wp + (int32_t)((px.ox - tx0) * pg.s);
        sig[j] = px.ok ? sg : 0;
    }
    // byte offset of this lane's eight values in a unit of the filter copy [unit][row][16], or in the first piece of
    // [unit][piece][row][16]
    constexpr uint32_t ROW_BYTES = CUT ? 32u : 64u;
    uint32_t arow[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t row = m0 + (uint32_t)((wm * TM + i) * 16 + l16);
        arow[i] = row < p.M ? row * ROW_BYTES + (uint32_t)(q & 1) * (ROW_BYTES / 2) : OOB_ROW;
    }
    const uint32_t piece_bytes = p.M * ROW_BYTES, unit_bytes = piece_bytes * (CUT ? NP : 1);      // unit = tap * ncb16 + 16-channel block

    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // ---- patch: a wave brings eight channels of a group (an octet), 64 slots (a chunk) at a time: wave w all chunks of
    // octet w, or, going round, chunks 2 * (w / 2) and the next of octet w % 2 and, once these are stored, of octet 2 + w % 2 -----
    constexpr bool RING = L::RING;
    constexpr int kStoreHalf = 3;               // of a group's steps, the one in front of which the next one's first half is stored
    constexpr int NCH = RING ? 2 : NSL;         // chunks on their way at a time
    float pr[NCH][8];
    auto load_chunk = [&](auto EC, int grp, int half) {
        constexpr int e = decltype(EC)::value;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int c = grp * 32 + (RING ? half * 2 + wave % 2 : wave) * 8 + t;
            const uint32_t soff = c < (int)pg.Cred ? (uint32_t)(c * pg.chan_stride) * 4u : OOB_K;
            pr[e][t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrcB, voff[e], soff, 0));
        }
    };
    // plane of octet o of the group whose first one lies in plane `first`
    auto plane_of = [&](int first, int o) { return RING && first + o >= L::OCTETS ? first + o - L::OCTETS : first + o; };
    auto store_chunks = [&](int first, int half) {
        const int at = plane_of(first, RING ? half * 2 + wave % 2 : wave) * L::SLOTS + chunk0 * 64 + lane;
#pragma unroll
        for (int e = 0; e < NCH; ++e) {
            v4u pc[NP];
            split8<NP>(pr[e], pc);
#pragma unroll
            for (int k = 0; k < NP; ++k) lds[k * L::PLANE + at + e * 64] = pc[k];
        }
    };

    // ---- steps: (group, index); both units of a step and where they lie -------------------------------
    auto steps_of = [&](int grp) { return 2 * grp + 1 < ncb16 ? KK : (KK + 1) / 2; };
    constexpr int AW = CUT ? NP : 2;            // 16-byte loads of a row: a piece each, or four fp32 values
    using Rows = v4u[TM][AW];
    auto load_a = [&](Rows &ar, int grp, int s) {
        uint32_t u0 = OOB_K, u1 = OOB_K;
        if (grp < ngrp) {
            if (2 * grp + 1 < ncb16) {
                u0 = (uint32_t)(s * ncb16 + 2 * grp) * unit_bytes;
                u1 = u0 + unit_bytes;
            } else {
                u0 = (uint32_t)(2 * s * ncb16 + 2 * grp) * unit_bytes;
                if (2 * s + 1 < KK) u1 = u0 + (uint32_t)ncb16 * unit_bytes;
            }
        }
        const uint32_t u = second ? u1 : u0;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t at = CUT && u >= OOB_K ? OOB_K : arow[i] + u;        // (a piece's offset on top of both marks would wrap)
#pragma unroll
            for (int k = 0; k < AW; ++k)
                ar[i][k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rsrcA, at + (CUT ? 0u : 16u * k), CUT ? k * piece_bytes : 0u, 0));
        }
    };
    auto tap_slot = [&](int t) {                // slot displacement of tap t
        const int ky = (int)fdiv((uint32_t)t, pg.divKW), kx = t - ky * pg.KW;
        return pg.flip ? (pg.KH - 1 - ky) * pg.Wp + (pg.KW - 1 - kx) : ky * pg.Wp + kx;
    };

    if (threadIdx.x < NP) lds[threadIdx.x * L::PLANE + L::ZERO] = v4u{0u, 0u, 0u, 0u};
    static_for<0, NCH>([&](auto EC) { load_chunk(EC, 0, 0); });
    Rows ar;                                    // of the next step
    load_a(ar, 0, wk);
    store_chunks(0, 0);
    if constexpr (RING) {
        static_for<0, NCH>([&](auto EC) { load_chunk(EC, 0, 1); });
        store_chunks(0, 1);
    }
    block_sync_lds();
    int first = 0;                              // plane of this group's first octet

    using Step = MmaStep<NP, TM, TN, TM >= 3 ? 1 : 2>;
    // the products of step s of a group with the rows in `ap`, everything for later steps being on its way
    auto multiply = [&](int grp, int s, const v4u (&ap)[TM][NP]) {
        // where the lane reads: slot displacement of its unit's tap, octet of its channels
        int base;
        int32_t mask = -1;
        if (2 * grp + 1 < ncb16) base = tap_slot(s) + plane_of(first, q) * L::SLOTS;
        else {
            const int t0 = tap_slot(2 * s), t1 = tap_slot(min(2 * s + 1, KK - 1));
            base = (second ? t1 : t0) + plane_of(first, q & 1) * L::SLOTS;
            if (2 * s + 1 >= KK && second) { base = L::ZERO; mask = 0; }     // no second unit: zeros
        }
        auto read_b = [&](int j, v4u (&pc)[NP]) {
            const int idx = (sig[j] & mask) + base;
#pragma unroll
            for (int k = 0; k < NP; ++k) pc[k] = lds[idx + k * L::PLANE];
        };
        Step::run(ap, acc, read_b, typename Step::NoWork{});
    };
    // in front of a step's products: part of the next group's patch, then (by the caller) the next step's filters, so that
    // waiting for those, one step from now, waits for nothing younger.  ls: steps this wave has made of the group
    auto part_of_patch = [&](int grp, int ls) {
        if constexpr (RING) {
            if (ls == kStoreHalf && grp + 1 < ngrp) store_chunks(plane_of(first, 4), 0);
            static_for<0, 2>([&](auto EC) {
                constexpr int e = decltype(EC)::value;
                if (ls == e) load_chunk(EC, grp + 1, 0);
                if (ls == kStoreHalf + e) load_chunk(EC, grp + 1, 1);
            });
        } else static_for<0, NSL>([&](auto EC) { if (ls == decltype(EC)::value) load_chunk(EC, grp + 1, 0); });
    };
    // the group of which this wave has made ls steps is behind it
    auto next_patch = [&](int grp, int ls) {
        const int next = plane_of(first, 4);
        if constexpr (RING) {
            if (ls <= kStoreHalf) {             // (a short group)
                static_for<0, 2>([&](auto EC) { if (ls <= decltype(EC)::value) load_chunk(EC, grp + 1, 0); });
                store_chunks(next, 0);
            }
            static_for<0, 2>([&](auto EC) { if (ls <= kStoreHalf + decltype(EC)::value) load_chunk(EC, grp + 1, 1); });
        } else static_for<0, NSL>([&](auto EC) { if (ls <= decltype(EC)::value) load_chunk(EC, grp + 1, 0); });
        block_sync_lds();                       // every wave is done with this group's patch
        store_chunks(RING ? next : 0, RING ? 1 : 0);
        block_sync_lds();
        if constexpr (RING) first = next;
    };
    if constexpr (NP == 3) {
        // (fp32 rows are cut in one piece in front of the products: cutting them behind the products of the step
        // before, as split_gemm_kernel does, takes 24 more registers.  Two steps a turn with two sets of rows, as below, makes the
        // 192-row tiles spill 200 registers and more: 308 -> 554 us for 256 images, 192 channels of 13x13, 192 rows, 3x3)
        for (int grp = 0; grp < ngrp; ++grp) {
            const int ns = steps_of(grp);
            int ls = 0;
            for (int s = wk; s < ns; s += WK, ++ls) {
                v4u ap[TM][NP];
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if constexpr (CUT) {
#pragma unroll
                        for (int k = 0; k < NP; ++k) ap[i][k] = ar[i][k];
                    } else {
                        float f[8];
#pragma unroll
                        for (int t = 0; t < 8; ++t) f[t] = __uint_as_float(ar[i][t / 4][t % 4]);
                        split8<NP>(f, ap[i]);
                    }
                }
                part_of_patch(grp, ls);
                if (s + WK < ns) load_a(ar, grp, s + WK);
                else load_a(ar, grp + 1, wk);
                multiply(grp, s, ap);
            }
            if (grp + 1 < ngrp) next_patch(grp, ls);
        }
    } else {
        // two steps a turn, so that the rows on their way need not be moved to where the next step reads them
        int grp = 0, s = wk, ls = 0;
        auto step = [&](const Rows &cur, Rows &next) {
            const bool last = s + WK >= steps_of(grp);
            part_of_patch(grp, ls);
            load_a(next, last ? grp + 1 : grp, last ? wk : s + WK);
            multiply(grp, s, cur);
            s += WK;
            ++ls;
            if (!last) return true;
            if (grp + 1 < ngrp) next_patch(grp, ls);
            s = wk;
            ls = 0;
            return ++grp < ngrp;
        };
        Rows other;
        while (step(ar, other) && step(other, ar)) {}
    }
    if constexpr (WK == 2) {
        // the second wave's sums are added to the first's, which stores the tile
        block_sync_lds();                       // the patch's LDS is free
        v4f *const ex = reinterpret_cast<v4f *>(lds) + (wm * WN + wn) * (TM * TN * 64);
        if (wk == 1) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) ex[(i * TN + j) * 64 + lane] = acc[i][j];
        }
        block_sync_lds();
        if (wk == 1) return;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += ex[(i * TN + j) * 64 + lane];
    }
    if constexpr (NP == 3 && !SCATTER) {          // (scattered sums are looked at when they are stored)
        if (not_finite(acc)) sums_in_fp32(acc, [&](int j, auto &&add) {
            // this lane's pixel: its image, position of its window
            const Pixel px = pixel((wn * TN + j) * 16 + l16);
            const int32_t img = (int32_t)px.b * pg.img_stride, wy = (int32_t)(px.oy * pg.s) + pg.oy0, wx = (int32_t)(px.ox * pg.s) + pg.ox0;
            for (int t = 0; t < KK; ++t) {
                const int ky = (int)fdiv((uint32_t)t, pg.divKW), kx = t - ky * pg.KW;
                const int32_t sy = wy + (pg.flip ? pg.KH - 1 - ky : ky), sx = wx + (pg.flip ? pg.KW - 1 - kx : kx);
                const bool ok = px.ok && (uint32_t)sy < (uint32_t)pg.Hs && (uint32_t)sx < (uint32_t)pg.Ws;
                for (int cb = 0; cb < ncb16; ++cb) {
                    // a unit of 16 channels, four consecutive ones a lane, its loads in flight together
                    float a[4][TM], b[4];
                    const uint32_t unit = (uint32_t)(t * ncb16 + cb) * unit_bytes;
                    auto row_of = [&](int i) { return m0 + (uint32_t)((wm * TM + i) * 16 + l16); };
                    v2u pc[TM][CUT ? NP : 1];
                    if constexpr (CUT) {
#pragma unroll
                        for (int i = 0; i < TM; ++i)
#pragma unroll
                            for (int k = 0; k < NP; ++k)
                                pc[i][k] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rsrcA, row_of(i) < p.M ? row_of(i) * ROW_BYTES + unit + 8u * (uint32_t)q : OOB_K, k * piece_bytes, 0));
                    } else {
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const auto f = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, row_of(i) < p.M ? row_of(i) * ROW_BYTES + unit + 16u * (uint32_t)q : OOB_K, 0, 0);
#pragma unroll
                            for (int v = 0; v < 4; ++v) a[v][i] = __uint_as_float((uint32_t)f[v]);
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int c = 16 * cb + 4 * q + v;
                        const uint32_t at = ok && c < (int)pg.Cred ? (uint32_t)(img + c * pg.chan_stride + sy * pg.Ws + sx) * 4u : OOB_K;
                        b[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrcB, at, 0, 0));
                    }
                    if constexpr (CUT) {
                        // the pieces' sum is the value exactly, but for values whose scaled pieces are no finite numbers (from 2^104
                        // up, infinities, NaN): those come from the filters themselves
                        float z = 0.f;
#pragma unroll
                        for (int i = 0; i < TM; ++i)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                float s = 0.f;
#pragma unroll
                                for (int k = 0; k < NP; ++k) s += __uint_as_float(v % 2 ? pc[i][k][v / 2] & 0xffff0000u : pc[i][k][v / 2] << 16);
                                z = fmaf(s, 0.f, z);
                                a[v][i] = s * (1.f / kCutScale);
                            }
                        if (!(z == 0.f)) {
                            const StridedTaps &f = p.taps;
#pragma unroll
                            for (int i = 0; i < TM; ++i)
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const int c = 16 * cb + 4 * q + v, m = pg.flip ? c : (int)row_of(i), ci = pg.flip ? (int)row_of(i) : c;
                                    if (row_of(i) < p.M && c < (int)pg.Cred) a[v][i] = f.w[(((size_t)g * f.Mg + m) * f.Cg + ci) * KK + t];
                                }
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) add(a[v], b[v]);
                }
            }
        });
    }
    store_columns_at<TM, TN, SCATTER>(p, acc, g, 0u, m0 + (uint32_t)(wm * TM * 16), lane, [&](int c) {
        const int i = wn * TN * 16 + c;
        if (rs) {
            const Pixel px = pixel(i);
            return Columns{px.b * P + px.oy * pg.divOW.d + px.ox, px.ok ? min(4u, (uint32_t)pg.OWo - px.ox) : 0u};
        }
        const uint32_t n = n0 + (uint32_t)i;
        return Columns{n, n <= n1 ? min(4u, n1 + 1u - n) : 0u};
    });
}

namespace {

// pixel tiles (blocks along x) of a patch-kernel problem
uint32_t patch_pixel_tiles(const IgemmProblem &p)
{
    return p.patch.tiles_per_img ? (p.N / p.patch.divP.d) * (uint32_t)p.patch.tiles_per_img : (p.N + 127) / 128;
}

template <int NP, int TM, int WM, int WK, int NSL>
int launch_cfg(const IgemmProblem &p, hipStream_t stream)
{
    constexpr int MT = WM * TM * 16, TN = 128 / (16 * (4 / (WM * WK)));
    dim3 grid(p.patch.tile_count ? p.patch.tile_count : patch_pixel_tiles(p), (p.M + MT - 1) / MT, p.groups);
    if (grid.y > 65535u || grid.z > 65535u) return CG_EUNSUPPORTED;
    int rec = -1;
    if (prof_on()) {
        char name[64];
        snprintf(name, sizeof name, NP == 1 ? "igemm_patch%s_kernel<%dx128,%d,bf16>" : NP == 2 ? "igemm_patch%s_kernel<%dx128,%d,bf16x3>" : "igemm_patch%s_kernel<%dx128,%d>",
                 WK == 2 && NP == 3 ? "16" : "", MT, NSL);
        rec = prof_begin(name, p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups, 0.0, stream);
    }
    constexpr size_t patch = PatchLds<NP, TM, WK, NSL, CG_CUT>::BYTES, sums = WK == 2 ? (4 / (WM * WK)) * WM * TM * TN * 64 * 16 : 0, lds = patch > sums ? patch : sums;
    static_assert(2 * lds <= 160 * 1024, "two blocks of this tile do not fit the LDS of a compute unit");
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        CG_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&split_patch_kernel<NP, TM, WM, WK, NSL, CG_SCATTER, CG_CUT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((split_patch_kernel<NP, TM, WM, WK, NSL, CG_SCATTER, CG_CUT>), grid, dim3(256), lds, stream, p);
    prof_end(rec, stream);
    CG_HIP_TRY(hipGetLastError());
    return CG_OK;
}

template <int NP, int NSL> int launch_tiles(const IgemmProblem &p, int mt, hipStream_t stream)
{
    if constexpr (NP == 3) {
        if (mt == 48) return launch_cfg<NP, 3, 1, 2, NSL>(p, stream);
        if (mt == 32) return launch_cfg<NP, 2, 1, 2, NSL>(p, stream);
        if (mt == 16) return launch_cfg<NP, 1, 1, 2, NSL>(p, stream);
    }
    // (what patch_wants_pieces leaves to fp32 filters whatever the size has no instance with three pieces)
    constexpr bool CUT3 = NP == 3 && CG_CUT;
    if (mt == 192) {
        if constexpr (CUT3 && NSL != 4) return CG_EUNSUPPORTED;
        else return launch_cfg<NP, 3, 4, 1, NSL>(p, stream);
    }
    if (mt == 128) {
        if constexpr (CUT3 && NSL == 4 && CG_SCATTER) return CG_EUNSUPPORTED;
        else return launch_cfg<NP, 2, 4, 1, NSL>(p, stream);
    }
    return launch_cfg<NP, 1, 4, 1, NSL>(p, stream);
}

}  // namespace

// This file is compiled once per number of pieces (CG_NP), for scattered rows (CG_SCATTER) and for others, for filters in
// pieces (CG_CUT) and, with three pieces, for fp32 ones, in parallel.
#define CG_CAT_(a, b, c, d, e, f) a##b##c##d##e##f
#define CG_CAT(a, b, c, d, e, f) CG_CAT_(a, b, c, d, e, f)
int CG_CAT(split_patch_tiles_, CG_NP, _, CG_SCATTER, _, CG_CUT)(const IgemmProblem &p, int mt, hipStream_t stream)
{
    if (p.patch.nsl == 4) return launch_tiles<CG_NP, 4>(p, mt, stream);
    if (p.patch.nsl == 5) return launch_tiles<CG_NP, 5>(p, mt, stream);
    return launch_tiles<CG_NP, 6>(p, mt, stream);
}

#if CG_NP == 3 && !CG_SCATTER && !CG_CUT
int split_patch_tiles_1_0_1(const IgemmProblem &p, int mt, hipStream_t stream);
int split_patch_tiles_1_1_1(const IgemmProblem &p, int mt, hipStream_t stream);
int split_patch_tiles_2_0_1(const IgemmProblem &p, int mt, hipStream_t stream);
int split_patch_tiles_2_1_1(const IgemmProblem &p, int mt, hipStream_t stream);
int split_patch_tiles_3_0_1(const IgemmProblem &p, int mt, hipStream_t stream);
int split_patch_tiles_3_1_0(const IgemmProblem &p, int mt, hipStream_t stream);
int split_patch_tiles_3_1_1(const IgemmProblem &p, int mt, hipStream_t stream);

namespace {

int patch_launch_tiles(const IgemmProblem &p, int mt, hipStream_t stream)
{
    if (p.math == CG_MATH_BF16) return p.c_scatter ? split_patch_tiles_1_1_1(p, mt, stream) : split_patch_tiles_1_0_1(p, mt, stream);
    if (p.math == CG_MATH_BF16X3) return p.c_scatter ? split_patch_tiles_2_1_1(p, mt, stream) : split_patch_tiles_2_0_1(p, mt, stream);
    if (p.patch.filter_pieces) return p.c_scatter ? split_patch_tiles_3_1_1(p, mt, stream) : split_patch_tiles_3_0_1(p, mt, stream);
    return p.c_scatter ? split_patch_tiles_3_1_0(p, mt, stream) : split_patch_tiles_3_0_0(p, mt, stream);
}

// Row-tile height.  Two blocks are resident per compute unit (an odd one out runs alone and a little
// slower than a pair); a block's time goes with its rows plus a constant, 18 to 40 rows' worth (bringing
// the patch, the epilogue; 13x13 planes, 384 rows: 64 / 128 / 192-row blocks took 68 / 121 / 190 us).
int patch_mt(uint32_t M, uint32_t N, uint32_t groups)
{
    const int cand[3] = {192, 128, 64};
    int best = 64;
    double best_cost = 1e300;
    const uint64_t units = igemm_resident_blocks() > 1 ? igemm_resident_blocks() / 2 : 1;
    for (int c : cand) {
        const uint64_t tiles = (uint64_t)((M + c - 1) / c) * ((N + 127) / 128) * groups;
        const uint64_t n = (tiles + units - 1) / units;
        const double cost = ((n & 1) ? (double)(n - 1) + 1.2 : (double)n) * (c + 40);
        if (cost < best_cost * 0.999) { best_cost = cost; best = c; }
    }
    return best;
}

int patch_launch(const IgemmProblem &p, hipStream_t stream)
{
    // few rows: a wave takes them all, and the steps are shared out instead (a 64-row tile multiplies 64
    // rows for 48).  The reduced modes have 64-row tiles only.
    if (p.M <= 48 && p.math == CG_MATH_FP32) return patch_launch_tiles(p, (int)(p.M + 15) / 16 * 16, stream);
    int mt = patch_mt(p.M, p.N, p.groups);
    // Two blocks are resident per compute unit, so blocks run in rounds of igemm_resident_blocks() that
    // start and end together.  What a short last round leaves idle is won back in two ways; times with / without, us:
    // - forward, fp32: the pixel tiles of the whole rounds go out as one launch and the rest as a second launch of
    //   64-row tiles.  192-row tiles: 192 rows, 1728 indices, 1.32 rounds 303 / 315; 160 rows, 1296, 1.11 rounds 223 / 253;
    //   320 rows, 2800, 2.09 rounds 726 / 772.  128-row tiles only for a rest of a few blocks (1.04 and 1.14 rounds 0.97;
    //   1.3 - 1.5, 2.1 - 2.5, 4.3 rounds 1.03 - 1.06).  One and two pieces: 1.03 - 1.08 nearly always, so not there.
    //   Not backward-data: it shares the GPU with backward-weight on another stream, whose blocks already
    //   fill those compute units.
    // - backward-data (mirrored taps), one and two pieces, 128-row tiles: 64-row tiles for the whole launch (112 rows, 1344
    //   indices, 1.12 rounds, two pieces 106 / 118; 336 rows 1.63 rounds 162 / 172).  192-row tiles lose by it (1.02 - 1.08),
    //   and three pieces do (256 rows, 3456 indices, 1.32 rounds 498 / 450; 192 rows 346 / 316).  A caller that runs another
    //   stream beside it says so (beside_other_stream) and keeps the large tiles.
    const uint32_t rb = igemm_resident_blocks(), px = patch_pixel_tiles(p), per_px = ((p.M + mt - 1) / mt) * p.groups;
    const uint64_t blocks = (uint64_t)px * per_px;
    const uint32_t rounds = (uint32_t)(blocks / rb), rest = (uint32_t)(blocks - (uint64_t)rounds * rb);
    const bool short_round = mt > 64 && p.patch.tile_count == 0 && rounds >= 1 && rest > 0 && rest < rb * 3 / 4;
    if (short_round && p.patch.flip && p.patch.nsl == 4 && !p.beside_other_stream && p.math != CG_MATH_FP32 && mt == 128) mt = 64;
    else if (short_round && !p.patch.flip && p.math == CG_MATH_FP32 && (mt == 192 || rest <= 80)) {
        const uint32_t px_main = rounds * rb / per_px;
        const uint32_t tail_blocks = (px - px_main) * ((p.M + 63) / 64) * p.groups;
        if (px_main > 0 && px_main < px && tail_blocks <= rb) {
            IgemmProblem a = p, b = p;
            a.patch.tile0 = 0;
            a.patch.tile_count = px_main;
            b.patch.tile0 = px_main;
            b.patch.tile_count = px - px_main;
            const double fl = p.flops > 0 ? p.flops : 2.0 * p.M * (double)p.N * p.K * p.groups;
            a.flops = fl * px_main / px;
            b.flops = fl - a.flops;
            const int rc = patch_launch_tiles(a, mt, stream);
            return rc != CG_OK ? rc : patch_launch_tiles(b, 64, stream);
        }
    }
    return patch_launch_tiles(p, mt, stream);
}

}  // namespace

// Filters in pieces instead of fp32 ones: 1140 random passes, times with fp32 filters over those with pieces.
// - up to 48 rows 1.04 - 1.2 (16-row tiles of four chunks 0.97 - 1.10)
// - 192-row tiles have registers for a second set of pieces only where the patch goes round (PatchLds): 27x27 planes, 96 -> 192
//   channels 5x5, five chunks, 791 / 780 - 818 us; 13x13, two groups, 384 -> 384 3x3, four chunks, 310 / 285
// - 64- and 128-row tiles of five and six chunks 0.99 - 1.12
// - 128-row tiles of four chunks, whose patch goes round: 0.97 - 1.07 where there is a second group of channels, 0.93 - 0.98 where there
//   is none (16 -> 293 channels 3x3, 36 images of 17x17, 21 / 22 us); strided backward-data 0.89 - 1.01 (410 -> 114 3x3 stride 2, eight of
//   34x34, 59 / 64); forward of a round and up to 80 blocks more, which go out as a second launch, 0.92 - 0.99 (128 -> 414 2x2 in two
//   groups, 45 of 21x21, 54 / 59)
// - 64-row tiles of four chunks: strided backward-data 1.01 - 1.08.  The others follow the rounds of resident blocks: up to one round
//   0.93 - 1.0, one to one and a half 0.98 - 1.04, up to two 0.95 - 0.99 (90 -> 300 3x3 in two groups, 150 of 13x13, 57 / 61), beyond
//   0.98 - 1.04; fewer than 450 indices 0.95 - 1.0 whatever the blocks
bool patch_wants_pieces(const IgemmProblem &p)
{
    if (p.M <= 48) return true;
    const int mt = patch_mt(p.M, p.N, p.groups);
    if (p.patch.nsl != 4) return mt != 192;
    if (mt == 192) return true;
    const uint64_t blocks = (uint64_t)patch_pixel_tiles(p) * ((p.M + mt - 1) / mt) * p.groups, rb = igemm_resident_blocks();
    if (mt == 128) return !p.c_scatter && p.patch.Cred > 32 && (p.patch.flip || blocks <= rb || blocks > rb + 80);
    return p.c_scatter || (p.K >= 450 && (blocks > 2 * rb || (blocks > rb && blocks * 2 <= rb * 3)));
}

static std::atomic<uint32_t> g_patch_min_tiles{512};
bool patch_forced() { return g_patch_min_tiles.load(std::memory_order_relaxed) <= 1; }
void patch_set_min_tiles(uint32_t t) { g_patch_min_tiles.store(t, std::memory_order_relaxed); }

bool patch_plan(PatchGeom &g, uint32_t M, uint32_t N, uint32_t groups, int math)
{
    g.nsl = 0;
    const int KK = g.KH * g.KW;
    if (g.Cred == 0 || KK < 4 || g.s <= 0 || g.OHo <= 0 || g.OWo <= 0) return false;
    if (g.src_elems * 4 > kMaxBufferBytes || N >= (1u << 30)) return false;
    if (g.Cred % 16 && (uint64_t)M * groups * ((g.Cred + 15) / 16 * 16) * (uint64_t)KK * 4 > kMaxBufferBytes) return false;     // its filter copy
    g.Wp = (g.OWo - 1) * g.s + g.KW;
    const int64_t rfull = (int64_t)((g.OHo - 1) * g.s + g.KH) * g.Wp;
    if (rfull >= (1 << 24)) return false;
    g.Rfull = (int32_t)rfull;
    const uint32_t P = (uint32_t)g.OHo * (uint32_t)g.OWo;
    g.divP = make_fastdiv(P);
    g.divOW = make_fastdiv((uint32_t)g.OWo);
    g.divWp = make_fastdiv((uint32_t)g.Wp);
    g.divRfull = make_fastdiv((uint32_t)g.Rfull);
    g.divKW = make_fastdiv((uint32_t)g.KW);
    // The kernel has no K slices, and a block alone on a compute unit waits for its own loads: with few tiles the
    // gathered kernel, cut along K, is faster, the more so the longer the reduction.  fp32, tiles of 64 rows, times there /
    // here (285 problems, 3x3 and 5x5 windows): below 256 tiles 0.5 - 1.3; 256 - 384 tiles 0.98 - 1.6 up to 1200 indices,
    // 0.64 - 1.0 beyond for most; 384 - 640 tiles 1.0 - 1.7 below 3200 indices, 0.8 - 1.0 beyond; from 640 tiles 1.0 - 2.2.  Up
    // to 48 rows (waves share the rows and split the steps) 0.9 - 2.6 from 200 tiles; more rows and fewer than 128 indices
    // 0.79 - 0.98 whatever the tiles.
    const uint64_t T = (uint64_t)((M + 63) / 64) * ((N + 127) / 128) * groups, lim = g_patch_min_tiles.load(std::memory_order_relaxed);
    const uint32_t K = g.Cred * (uint32_t)KK;
    const bool enough = M <= 48 ? T * 5 >= lim * 2 : K < 128 ? false : T * 4 >= lim * 5 || (T * 4 >= lim * 3 && K < 3200) || (T * 2 >= lim && K <= 1200);
    if (lim > 1 && !enough) return false;
    // Channels that are no multiple of 16 (zeros are multiplied for the rest) and windows of four taps (a patch is worth
    // little there).  1300 problems in fp32, 260 in each of the other modes, the other kernels' time over this one's: as far as
    // the lines below take them 0.87 - 2.4, geometric mean 1.3, and 1.5 in the other modes; left out: fewer tiles 0.16 - 1.7,
    // most below 0.9; tiles x indices below 200 000 or fewer than 250 indices 0.55 - 1.2; more than 25 % zeros (90 % beside few
    // rows) 0.6 - 1.5; two and
    // three taps, and five in a row, 0.2 - 1.04; four taps of up to 16 rows, whose tiles in one and two pieces are 64 rows,
    // 0.6 - 1.28.  (A problem that split_gemm_kernel runs in tiles of 128 rows stays there, see the callers: 0.8 - 1.2, and its
    // shorter sums are closer to 64 bits.)  The error against 64 bits is 0.15 to 1.0 of what it was.
    const bool padded = g.Cred % 16 != 0;
    if (lim > 1 && (padded || KK == 4)) {
        const uint64_t zeros = (g.Cred + 15) / 16 * 16 * 100ull;
        if (T * K < 200000 || K < 250 || KK == 5 || (KK == 4 && M <= 16) || T < (M <= 16 ? 350 : M <= 48 ? 250 : 400) ||
            zeros > g.Cred * (M <= 48 ? 190ull : 125ull))
            return false;
        // strided backward-data, 17 to 48 rows: by the taps that exist (both kernels multiply the zeros of the others); see below
        const uint64_t real = (uint64_t)K * g.taps / g.tap_slots;
        if (math == CG_MATH_FP32 && g.taps < g.tap_slots && M > 16 && M <= 48 && (real < 270 || T * real < 140000 || zeros > g.Cred * 170ull)) return false;
    }
    // Those problems again, fp32, 780 of them chosen around the lines; times there / here of what is taken out and of what stays:
    // - strided backward-data, 17 to 48 rows: 0.74 - 1.2, 13 of 18 below 0.97 (35 -> 3 channels 11x11 stride 4, 80 images of
    //   156x156, 79 / 88 us; 69 -> 3 7x7, 122 of 196x196, 135 / 171); what stays 0.95 - 1.9
    // - what of a block's products is none of padding, here over there (`share`), is what the times follow where the other kernels
    //   test no window (forward without padding) and a block is all rows: up to 48 rows and fewer than 700 indices they are within
    //   15 % of it, with more indices 1.2 times it, with four taps 0.8 times it, with 25 and more 1.1 - 1.7 times it
    // - more than 48 rows and fewer than 500 tiles: a share below 0.74 0.82 - 0.92 (54 -> 55 channels 3x3, 137 images of 20x22, 56 / 67 us;
    //   26 -> 269 5x5, ten of 31x35, 63 / 69), above 1.05 - 1.6
    // - four taps without padding, 49 to 100 rows, fewer than 500 indices 0.73 - 1.08, median 0.92; beyond 0.94 - 1.23
    const bool few = M <= 48, inside = !g.flip && !g.oy0 && !g.ox0;
    auto worth = [&](uint64_t pixel_tiles) {
        if (lim <= 1 || math != CG_MATH_FP32 || (!padded && KK != 4)) return true;
        if (inside && KK == 4 && !few && M <= 100 && K < 500) return false;
        const double least = inside && few ? (KK == 4 ? 1.2 : KK >= 25 ? 0.7 : K < 700 ? 1. : 0.8) : !few && T < 500 ? 0.74 : 0.;
        auto full = [&](uint32_t tile) { return (double)M / ((M + tile - 1) / tile * tile); };
        const int there = M <= 16 && K >= 180 && T >= 600 ? 16 : gathered_plan(M, N, K, groups).mt;
        const double here = full(few ? 16 : (uint32_t)patch_mt(M, N, groups)) * g.Cred / ((g.Cred + 15) / 16 * 16) * N / (pixel_tiles * 128.);
        return here >= least * full((uint32_t)there);
    };
    // The largest patch any block needs: a fragment read reaches (KH-1)*Wp + KW-1 beyond sigma, and
    // sigma + that stays below the slot count of the block's segments, which is what is counted.
    auto slots = [&](uint32_t n0, uint32_t n1) {
        const uint32_t bA = n0 / P, oyA = (n0 % P) / (uint32_t)g.OWo, bB = n1 / P, oyB = (n1 % P) / (uint32_t)g.OWo;
        if (bA == bB) return (int64_t)((oyB - oyA) * g.s + g.KH) * g.Wp;
        return (int64_t)(((uint32_t)g.OHo - 1 - oyA) * g.s + g.KH) * g.Wp + (int64_t)(bB - bA - 1) * g.Rfull +
               (int64_t)(oyB * g.s + g.KH) * g.Wp;
    };
    int64_t smax = 0;
    for (uint32_t n0 = 0; n0 < N && smax <= 4 * 64; n0 += 128) {
        const int64_t sl = slots(n0, (n0 + 127 < N - 1) ? n0 + 127 : N - 1);
        if (sl > smax) smax = sl;
    }
    g.tiles_per_img = 0;
    g.rect_shift = 0;
    g.divTpi = g.divTx = make_fastdiv(1);
    if (smax <= 4 * 64) { g.nsl = 4; return worth((N + 127) / 128); }
    // large images: blocks that stay inside one image need smaller patches (every image is the same)
    if (N % P) return false;
    int64_t amax = 0;
    for (uint32_t n0 = 0; n0 < P && amax <= 6 * 64; n0 += 128) {
        const int64_t sl = slots(n0, (n0 + 127 < P - 1) ? n0 + 127 : P - 1);
        if (sl > amax) amax = sl;
    }
    if (amax <= 6 * 64) {
        // (six chunks: planes 56 wide with a 3x3 window, four pixel rows, 348 slots)
        g.tiles_per_img = (int32_t)((P + 127) / 128);
        if (lim > 1 && (padded || KK == 4) && P * 4 < (uint32_t)g.tiles_per_img * 128 * 3) return false;       // mostly empty blocks
        g.nsl = amax > 5 * 64 ? 6 : 5;
    } else {
        // Rows too long to keep: rectangles of pixels, the fewest that fit.  170 problems on planes 40 to 240 wide that meet the
        // lines above, the other kernels' time over this one's 0.97 - 3.0, geometric mean 1.4 (57434 pixels, 12 rows, 221 channels
        // 5x5 344 / 114 us; 164892 pixels, 3 rows, 187 channels 5x5 678 / 277).
        for (int rs = 2; rs <= 6; ++rs) {
            const int w = 1 << rs, h = 128 >> rs;
            const int64_t sl = (int64_t)((h - 1) * g.s + g.KH) * ((w - 1) * g.s + g.KW);
            const int32_t tx = (g.OWo + w - 1) / w, tiles = tx * ((g.OHo + h - 1) / h);
            if (sl > 6 * 64 || (g.tiles_per_img && tiles >= g.tiles_per_img)) continue;
            g.tiles_per_img = tiles;
            g.rect_shift = rs;
            g.divTx = make_fastdiv((uint32_t)tx);
            g.nsl = sl > 5 * 64 ? 6 : sl > 4 * 64 ? 5 : 4;
        }
        if (!g.rect_shift) return false;
        const int w = 1 << g.rect_shift;
        g.Wp = (w - 1) * g.s + g.KW;
        g.Rfull = (int32_t)(((128 >> g.rect_shift) - 1) * g.s + g.KH) * g.Wp;
        g.divWp = make_fastdiv((uint32_t)g.Wp);
        g.divRfull = make_fastdiv((uint32_t)g.Rfull);
    }
    g.divTpi = make_fastdiv((uint32_t)g.tiles_per_img);
    return worth((uint64_t)(N / P) * g.tiles_per_img);
}

int split_patch_launch(const IgemmProblem &p, hipStream_t stream)
{
    if (!p.c_ptr || !aligned16(p.c_ptr) || !p.A.ptr || !aligned16(p.A.ptr)) return CG_EINVAL;
    if (p.M == 0 || p.N == 0 || p.K == 0 || p.groups == 0) return CG_EINVAL;
    if (p.M >= (1u << 30) || p.N >= (1u << 30) || p.K >= (1u << 30)) return CG_EUNSUPPORTED;
    if (p.bias_mode && !p.bias) return CG_EINVAL;
    if (p.math != CG_MATH_FP32 && p.math != CG_MATH_BF16 && p.math != CG_MATH_BF16X3) return CG_EINVAL;
    const PatchGeom &g = p.patch;
    if (!g.src || !aligned16(g.src) || g.nsl < 4 || g.nsl > 6 || p.splits != 1 || g.Cred == 0 ||
        p.K != g.Cred * (uint32_t)(g.KH * g.KW) || (p.c_scatter && (!p.taps.dy || !p.taps.w)) ||
        (g.filter_pieces ? g.filter_pieces != (p.math == CG_MATH_BF16 ? 1 : p.math == CG_MATH_BF16X3 ? 2 : 3) || !p.taps.w : p.math != CG_MATH_FP32))
        return CG_EINVAL;
    // the filter copy holds M rows of K values (channels padded to 16) per group, and byte offsets into it stay below the marks
    // that stand for "out of range"
    const uint64_t values = (uint64_t)p.M * ((g.Cred + 15) / 16 * 16) * (uint64_t)(g.KH * g.KW);
    if (p.A.elems * 4 > kMaxBufferBytes || (uint64_t)p.A.gstride * p.groups > p.A.elems ||
        (g.filter_pieces ? values / 2 * g.filter_pieces : values) > (uint64_t)p.A.gstride)
        return CG_EUNSUPPORTED;
    return patch_launch(p, stream);
}

#endif  // CG_NP == 3 && !CG_SCATTER && !CG_CUT

}  // namespace cg
