// Device code of the kernels that multiply fp32 operands in pieces on the bf16 matrix instructions.
#pragma once
#include <type_traits>
#include "cg_internal.h"
#include "igemm_device.h"

namespace cg {
namespace {

// A raw buffer of `bytes` bytes at `base`: reads beyond it return 0.  Both are uniform by construction;
// readfirstlane says so to the compiler, which otherwise wraps every load in a loop over the lanes'
// descriptors where a division on the vector unit was part of the address.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const float *base, uint64_t bytes)
{
    const uint64_t a = (uint64_t)reinterpret_cast<uintptr_t>(base);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>((uintptr_t)u), 0,
                                             (int)__builtin_amdgcn_readfirstlane((uint32_t)bytes), 0x00020000);
}

// Barrier of a block for LDS data: this wave's LDS accesses are done, global loads stay in flight.
__device__ __forceinline__ void block_sync_lds()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef uint32_t v4u __attribute__((ext_vector_type(4)));      // eight bf16: one piece of eight values
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 values cut into NP bf16 pieces, most significant first, each piece the nearest even of what
// the pieces before it left.  Three pieces hold 24 bits.  They are cut from the value times 2^24: the
// smallest fp32 number (2^-149) is then 2^-125, so that every value from there up is held exactly and no
// piece is subnormal; a product of two operands carries 2^48, which MmaStep takes out again.  What
// overflows on the way (an operand from 2^104 up, a sum from 2^80 up) or was no finite number leaves a
// NaN or an infinity in the sum, and sums that end as one are computed anew by fp32 multiply-adds
// (not_finite).  13 vector instructions a pair.
constexpr float kCutScale = 0x1p24f, kProductScale = 0x1p-48f;
template <int NP> __device__ __forceinline__ void split_pair(float x0, float x1, uint32_t (&pc)[NP])
{
    if constexpr (NP == 3) {
        x0 *= kCutScale;
        x1 *= kCutScale;
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        pc[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x0, x1}, bf16x2));
        if (k + 1 < NP) {
            uint32_t h = pc[k];
            asm("" : "+v"(h));             // both values from the pair: else each is converted once more on its own, 17 instructions
            x0 -= __uint_as_float(h << 16);
            x1 -= __uint_as_float(h & 0xffff0000u);
        }
    }
}

// pair t of eight values
template <int NP> __device__ __forceinline__ void split8_pair(const float (&f)[8], int t, v4u (&pc)[NP])
{
    uint32_t p[NP];
    split_pair<NP>(f[2 * t], f[2 * t + 1], p);
#pragma unroll
    for (int k = 0; k < NP; ++k) pc[k][t] = p[k];
}
template <int NP> __device__ __forceinline__ void split8(const float (&f)[8], v4u (&pc)[NP])
{
#pragma unroll
    for (int t = 0; t < 4; ++t) split8_pair<NP>(f, t, pc);
}

// The sums of a wave's tile that are not finite, again, by fp32 matrix instructions from the operands themselves, one
// column tile after the other: for_k(j, add) calls add(a, b) with four reduction indices at a time, one per lane / 16
// (a[i], b: of row 16 i + lane % 16 and of column 16 j + lane % 16).  What infinities, NaN and sums beyond 2^80
// get: a product that is NaN or overflows in fp32 does so here.  Several times slower than the pieces.
// Sums that came out finite stay as they are.
template <int TM, int TN, class ForK> __device__ __forceinline__ void sums_in_fp32(v4f (&acc)[TM][TN], ForK &&for_k)
{
    static_for<0, TN>([&](auto JC) {
        constexpr int j = decltype(JC)::value;
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) z = fmaf(acc[i][j][e], 0.f, z);
        if (!__any(!(z == 0.f))) return;
        v4f s[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) s[i] = v4f{0.f, 0.f, 0.f, 0.f};
        for_k(j, [&](const float (&a)[TM], float b) {
#pragma unroll
            for (int i = 0; i < TM; ++i) s[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(b, a[i], s[i], 0, 0, 0);
        });
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = fmaf(acc[i][j][e], 0.f, 0.f) == 0.f ? acc[i][j][e] : s[i][e];
    });
}

// Products that count, smallest first: number, piece of A, piece of B.
template <int NP> struct Products;
template <> struct Products<1> { static constexpr int N = 1, A[1] = {0}, B[1] = {0}; };
template <> struct Products<2> { static constexpr int N = 3, A[3] = {1, 0, 0}, B[3] = {0, 1, 0}; };
template <> struct Products<3> { static constexpr int N = 6, A[6] = {2, 0, 1, 1, 0, 0}, B[6] = {0, 2, 1, 0, 1, 0}; };

// Columns multiplied together: at least four independent sums, because an instruction that adds to the
// one before it waits about 60 cycles for it and a 16x16x32 multiply takes 16.
template <int TM, int TN> struct ColumnGroup { static constexpr int G = TM >= 3 ? 1 : TM == 2 ? 2 : TN >= 4 ? 4 : 2; };

// One step of 32 reduction indices: acc[i][j] += A tile i times B tile j, all pieces.  B is the FIRST
// operand of the instruction: a lane (q = lane / 16, l = lane % 16) then holds row l and the four
// columns 4q .. 4q+3 of a tile, which it can store as one 16-byte access.  read_b(j, pieces) fetches
// column tile j, one group ahead; work(slot) is other work of the step, spread over the slots 0 ..
// SLOTS-1, one behind each product of a group, whose vector instructions are laid between the matrix
// instructions.
// OWN: a step's products are added up on their own, from zero, and then to the accumulator by four vector
// multiply-adds a tile (which take out the scale of the pieces): the sum is rounded once per 32 terms instead
// of six times, and the instruction, which drops what lies below the last place of the sum it adds to,
// drops it from a sum 32 terms long.  Three pieces always do it.
template <int NP, int TM, int TN, int JG_ = ColumnGroup<TM, TN>::G, bool OWN = NP == 3> struct MmaStep {
    static constexpr int JG = JG_, PR = Products<NP>::N, SLOTS = TN / JG * PR;
    static_assert(TN % JG == 0, "whole groups");
    static_assert(OWN || NP < 3, "the scale of three pieces leaves the sum with the step's own products");
    struct NoWork {};
    template <class ReadB, class Work>
    __device__ __forceinline__ static void run(const v4u (&ap)[TM][NP], v4f (&acc)[TM][TN], ReadB &&read_b, Work &&work)
    {
        v4u bp[2][JG][NP];
#pragma unroll
        for (int jj = 0; jj < JG; ++jj) read_b(jj, bp[0][jj]);
        static_for<0, TN / JG>([&](auto GC) {
            constexpr int g = decltype(GC)::value;
            if constexpr (g + 1 < TN / JG) {
#pragma unroll
                for (int jj = 0; jj < JG; ++jj) read_b((g + 1) * JG + jj, bp[(g + 1) & 1][jj]);
            }
            v4f own[OWN ? TM : 1][OWN ? JG : 1];
            static_for<0, PR>([&](auto PC) {
                constexpr int pi = decltype(PC)::value, a = Products<NP>::A[pi], b = Products<NP>::B[pi];
#pragma unroll
                for (int jj = 0; jj < JG; ++jj)
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        v4f &to = OWN ? own[OWN ? i : 0][OWN ? jj : 0] : acc[i][g * JG + jj];
                        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bp[g & 1][jj][b]), __builtin_bit_cast(bf16x8, ap[i][a]),
                                                                     OWN && pi == 0 ? v4f{0.f, 0.f, 0.f, 0.f} : to, 0, 0, 0);
                        if constexpr (OWN && pi == PR - 1) {
                            if constexpr (NP == 3) {
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[i][g * JG + jj][e] = fmaf(to[e], kProductScale, acc[i][g * JG + jj][e]);
                            } else acc[i][g * JG + jj] += to;
                        }
                    }
                if constexpr (!std::is_same_v<std::decay_t<Work>, NoWork>) {
                    work(std::integral_constant<int, g * PR + pi>{});
                    static_for<0, TM * JG>([&](auto) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one matrix instruction,
                        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);      // three vector ones
                    });
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        });
    }
    // runs items 0 .. N-1 of a step's other work, evenly over the slots
    template <int N, class Item> struct Spread {
        Item item;
        template <class S> __device__ __forceinline__ void operator()(S) const
        {
            constexpr int s = S::value;
            static_for<s * N / SLOTS, (s + 1) * N / SLOTS>(item);
        }
    };
    template <int N, class Item> __device__ __forceinline__ static Spread<N, Item> spread(Item item) { return Spread<N, Item>{item}; }
};

}  // namespace
}  // namespace cg
