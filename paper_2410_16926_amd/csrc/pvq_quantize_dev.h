// Device code shared by the encoders of groups of up to 32 (Sec. 2.5, Sec. 3.3 Steps 3 to 5).  float32, fixed evaluation
// order: the results are part of the format.  The point: project onto the l1 ball of radius K, round to nearest even, then
// move single pulses on the coordinates of largest deviation (lowest coordinate on ties) until the count is K.  No coordinate
// is ever adjusted twice: for finite input the |sum - K| largest deviations are all positive, and an adjusted coordinate
// drops below -1/2.  So the repair takes one round per pulse, with the deviations formed once.
#pragma once

#include <hip/hip_runtime.h>

#include "pvq_exact_dev.h"

namespace pvq_quantize_dev {

using namespace pvq_exact_dev;

// Whether a group's norm l1 is one that all groups but tiny and huge ones have: between 2^-36 and 2^46, so that K / l1 is finite and
// the group has a direction, and the short quotients and roots are right for it: the sum of squares of up to 32 values lies between
// 2^-77 and 2^92, and the square of (y . w) / ||y|| not below 2^-96 (the largest value holds a pulse, K <= 127).  What is not has to
// be looked at closely.
__device__ inline bool ordinary_norm(float l1) { return magnitude_in(l1, 0x1p-36f, 0x1p46f); }

// K / l1; ordinary: whether all groups of the wave are.  degenerate: no direction, which are all zeros, norms whose reciprocal
// overflows, and anything not finite.
__device__ inline float over_norm(float K, float l1, bool &ordinary, bool &degenerate)
{
    float g = small_over(K, l1);
    degenerate = false;
    ordinary = __all(ordinary_norm(l1));
    if (!ordinary) {
        g = K / l1;
        degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(g < INFINITY);
    }
    return g;
}

// The amplitudes, ordinary being whether all groups of the wave are (ordinary_norm): the root of a sum of squares, and a sum of
// products over the root of an integer.
__device__ inline float root_of_squares(float ss, bool ordinary) { return ordinary ? root_of(ss) : sqrtf(ss); }
__device__ inline float over_root(float dot, float n, bool ordinary) { return ordinary ? divide(dot, root_divisor(n)) : dot / sqrtf(n); }

// Sum over adjacent pairs, level by level: ((v0+v1)+(v2+v3))+...  (fixed order, float32).
template <int D>
__device__ inline float tree_sum(float (&v)[D])
{
#pragma unroll
    for (int s = 1; s < D; s *= 2)
#pragma unroll
        for (int i = 0; i < D; i += 2 * s) v[i] = v[i] + v[i + s];
    return v[0];
}

// Three-operand orders of unsigned integers.
__device__ inline uint32_t max3(uint32_t a, uint32_t b, uint32_t c) { return max(max(a, b), c); }
__device__ inline uint32_t min3(uint32_t a, uint32_t b, uint32_t c) { return min(min(a, b), c); }
__device__ inline uint32_t med3(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Clamped to [0, 1] (what is not a number to 0) by the instruction itself.  Additions, multiplications and multiply-adds issue at
// nearly twice the rate of minima, comparisons and selections.
__device__ inline float clamped_product(float a, float b)
{
    float r;
    asm("v_mul_f32_e64 %0, %1, %2 clamp" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float clamped_difference(float a, float b)
{
    float r;
    asm("v_sub_f32_e64 %0, %1, %2 clamp" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// A coordinate's place in the order of deviations as one integer, larger for earlier places: the deviation's bits, scaled down so
// that LOG2D bits are free behind them, and there the coordinate, lower ones first, so that no two places are the same.  The
// scaled bits are the deviation's own from 2^-7 on, which is all that the first `need` places and the one behind them need:
// deviations are at most 1/2 and add up to `need` (to a few parts in 2^20), so the D - need behind the first ones still add up to
// need / 2, and the largest of them is above 1 / 64 for D <= 32.  Smaller ones may come out as equal, and negative ones are zero.
// unit: the sign of the deviations looked for, times order_scale.
template <int LOG2D> __device__ constexpr float order_scale() { return __builtin_bit_cast(float, 1u << (31 - LOG2D)); }
template <int LOG2D>
__device__ inline uint32_t order_of(float deviation, float unit, int i)
{
    return __float_as_uint(clamped_product(deviation, unit)) << LOG2D | (uint32_t)((1 << LOG2D) - 1 - i);
}

// The bits of a place behind all of them, for groups of which no pulse has to move (as a float, infinity).
constexpr uint32_t kNoPlace = 0x7F800000u;

// 1 for a key that is not behind the place `last`, 0 for one that is; before_last: the float with the bits of last - 1.  The keys' bits
// order like the floats that they are too, and the float behind last's is 2^10 on or more where the first places are (LOG2D 3 and 4: a
// deviation of 1 / 64 becomes 2^81 and 2^33), so the difference is at least 1 or not positive.
__device__ inline float taken(uint32_t key, float before_last) { return clamped_difference(__uint_as_float(key), before_last); }

// The repair of Sec. 2.5 for groups of 8: mag[i] += unit for the coordinates that hold the `need` first places (order_of), which
// are those not behind the last of them.  The first three places come out of a network of 21 minima, medians and maxima; a fourth
// (more there are not: eight deviations of at most 1/2 add up to `need`) is looked for in the waves that have such a group, one in seven.
// A round per place, with equal deviations told apart by masks on the scalar unit, took a hundred vector and 75 scalar
// instructions; this takes about 90 and six, and a scalar instruction's turn costs a SIMD as much as a vector one's.  28672 x 8192,
// 2-bit codes: 242 vector and 129 scalar instructions a group, 184 us; now 234 and 46, 152 us.
__device__ inline void adjust_first_places8(const uint32_t (&key)[8], float need, float unit, float (&mag)[8])
{
    const uint32_t a1 = max3(key[0], key[1], key[2]), b1 = med3(key[0], key[1], key[2]), c1 = min3(key[0], key[1], key[2]);
    const uint32_t a2 = max3(key[3], key[4], key[5]), b2 = med3(key[3], key[4], key[5]), c2 = min3(key[3], key[4], key[5]);
    const uint32_t a3 = max(key[6], key[7]), b3 = min(key[6], key[7]);
    // the n-th of two ordered lists is the largest of the minima of places that add up to n
    const uint32_t a = max(a1, a2), b = max3(min(a1, a2), b1, b2), c = max(max3(min(a1, b2), min(b1, a2), c1), c2);
    uint32_t first = max(a, a3), second = max3(min(a, a3), b, b3), third = max3(min(a, b3), min(b, a3), c);
    asm("" : "+v"(first), "+v"(second), "+v"(third));              // (all three at once: no branches)
    uint32_t last = need > 0.0f ? first : kNoPlace;
    last = need > 1.0f ? second : last;
    last = need > 2.0f ? third : last;
    if (__any(need > 3.0f)) {
        uint32_t fourth = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) fourth = max(fourth, key[i] < third ? key[i] : 0u);
        last = need > 3.0f ? fourth : last;
    }
    const float before_last = __uint_as_float(last - 1u);
#pragma unroll
    for (int i = 0; i < 8; i++) mag[i] = __builtin_fmaf(taken(key[i], before_last), unit, mag[i]);
}

// The same repair for any D and signed points (whose zeros have their sign too).  The places come one after the other: with `last`
// the place before, key - last as an unsigned number is largest for the first key behind it (keys not behind it stay below
// 2^31), so a round is a subtraction for a coordinate and half a three-operand maximum, and needs no masks.  A wave runs as many
// rounds as its lane with the largest `need`, about three for D = 16 and four for D = 32.  (Marks as masks, the key of a place that is
// taken set to -1: 8192 x 8192, D = 16, 48 bits, float32 amplitudes 54.3 us, now 44.7; D = 32, 96 bits, 2-bit codes 82.4, now 69.8.)
template <int D>
__device__ inline void adjust_first_places(const uint32_t (&key)[D], float need, float unit, float (&y)[D])
{
    uint32_t last = max(key[0], key[1]);
#pragma unroll
    for (int i = 2; i < D; i += 2) last = max3(last, key[i], key[i + 1]);
    last = need > 0.0f ? last : kNoPlace;
#pragma unroll 1
    for (float round = 1.0f; round < (float)D && __any(need > round); round += 1.0f) {
        uint32_t behind = max(key[0] - last, key[1] - last);
#pragma unroll
        for (int i = 2; i < D; i += 2) behind = max3(behind, key[i] - last, key[i + 1] - last);
        last = need > round ? last + behind : last;
    }
    const float before_last = __uint_as_float(last - 1u);
#pragma unroll
    for (int i = 0; i < D; i++) {
        float mag;
        if constexpr (D <= 16) mag = __builtin_fmaf(taken(key[i], before_last), unit, fabsf(y[i]));
        else mag = fabsf(y[i]) + (key[i] >= last ? unit : 0.0f);
        y[i] = copysignf(mag, y[i]);
    }
}

// ---- sums and fields over the lanes of a wave ----------------------------------------------------------------------
constexpr int kWave = 64;

// v + (v moved across lanes by one data-parallel-primitive pattern); lanes outside ROWS add zero
template <int CTRL, int ROWS = 0xF>
__device__ inline float dpp_add(float v)
{
    const int moved = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false);
    return v + __builtin_bit_cast(float, moved);
}

// Sum of the 64 lanes' values over adjacent pairs, level by level (lanes 2i and 2i+1, then pairs of
// pairs, ...), valid in lane 63.  Each level adds the two halves' sums, in whichever operand order
// the lane pattern gives (addition commutes exactly), so the result is the pair-level sum bit for bit.
__device__ inline float wave_pair_sum(float v)
{
    v = dpp_add<0xB1>(v);          // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);          // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);         // row_half_mirror
    v = dpp_add<0x140>(v);         // row_mirror
    v = dpp_add<0x142, 0xA>(v);    // row_bcast15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);    // row_bcast31 into rows 2 and 3
    return v;
}

// OR of v over aligned runs of N lanes (a power of two up to 32), in every lane of the run: the first four levels by lane
// patterns inside a row of 16 lanes (within a quad; then, the quads being uniform, the mirror images inside 8 and 16
// lanes bring the other half), the fifth across rows.
template <int CTRL>
__device__ inline uint32_t dpp_or(uint32_t v)
{
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
template <int N>
__device__ inline uint32_t or_over_lanes(uint32_t v)
{
    v = dpp_or<0xB1>(v);                              // quad_perm [1,0,3,2]
    if constexpr (N > 2) v = dpp_or<0x4E>(v);         // quad_perm [2,3,0,1]
    if constexpr (N > 4) v = dpp_or<0x141>(v);        // row_half_mirror
    if constexpr (N > 8) v = dpp_or<0x140>(v);        // row_mirror
    if constexpr (N > 16) v |= __shfl_xor(v, 16, kWave);
    return v;
}

// ---- amplitude codes (Sec. 3.3 Step 5): how many of the 2^bits - 1 ascending edges are <= u ----------------------
// A tree of nodes of three edges, one 16-byte read and three comparisons for two bits of the code (a bisection takes a
// dependent read per bit): node v of level l holds every 4^(L-l-1)-th edge of the 4^(L-l) - 1 under it, L = (bits + 1) / 2
// levels.  Absent edges (the fourth word, and two of three with one bit) are NaN, which no u reaches.
constexpr int kEdgeNodes = 85;
__device__ constexpr int edge_level_base(int l) { return ((1 << 2 * l) - 1) / 3; }

__device__ inline void fill_edge_tree(float4 *tree, const float *__restrict__ edges, int bits, int tid, int lanes)
{
    const int L = (bits + 1) / 2;
    for (int e = tid; e < 4 * edge_level_base(L); e += lanes) {
        const int n = e >> 2, j = e & 3;
        const int l = n < 1 ? 0 : n < 5 ? 1 : n < 21 ? 2 : 3;
        const int at = ((n - edge_level_base(l)) * 4 + j + 1) * (1 << 2 * (L - l - 1)) - 1;
        reinterpret_cast<float *>(tree)[e] = j < 3 && at < (1 << bits) - 1 ? edges[at] : __builtin_nanf("");
    }
}

template <int BITS>
__device__ inline uint32_t count_edges(const float4 *tree, float u)
{
    uint32_t v = 0;
#pragma unroll
    for (int l = 0; 2 * l < BITS; l++) {
        const float4 n = tree[edge_level_base(l) + v];
        v = 4 * v + (n.x <= u ? 1u : 0u) + (n.y <= u ? 1u : 0u) + (n.z <= u ? 1u : 0u);
    }
    return v;
}

// The row's amplitude codes (Sec. 3.3 Step 5): code = number of quantile edges <= u, u = ss_g / rowss.  The wave's groups are runs
// of 64, number first, first + waves, ... of the row, and nobody else touches their sums of squares.  A lane takes N neighbouring
// groups, of N runs at a time: the codes come together in the lane (with eight bits and N = 4 all of a word, else an OR over
// 32 / (SB N) lanes), the waits fill each other, and the loop runs once for N of the wave's tiles.  N is chosen with the kernel: a
// second form of this in the same kernel costs the loops around it registers.  (28672 x 8192 with 2-bit codes, four runs a wave: 163 us
// with N = 1, 154 with 4, 160 with both forms.)
template <int SB, int N>
__device__ inline void write_codes(const float *ss_row, float rowss, const float4 *tree, uint32_t *srow, int G, int first, int waves, int lane)
{
    constexpr int kLanes = 32 / (SB * N), kRunLanes = kWave / N;          // lanes of a word and of a run
    // The short quotient is right for row sums like these and sums of squares that are zero or not below 2^-70; none is above its row's.
    // (Divisions for all, and comparisons and selections in the repair: 14336 x 4096 bf16 with 8-bit codes 48.1 us, 8192 x 8192 in groups of 16,
    // 32-bit indices, 2-bit codes 51.5, in groups of 32, 104-bit indices, float32, 87.0; now 45.3, 46.5 and 75.1.)
    const bool ordinary = magnitude_in(rowss, 0x1p-60f, 0x1p30f);
    const divisor sum = divisor_of(rowss, reciprocal(rowss));
    for (int run = first; run * kWave < G; run += N * waves) {
        const int g = (run + lane / kRunLanes * waves) * kWave + N * (lane % kRunLanes);
        const float nan = __builtin_nanf("");                             // (no edge is reached: absent groups leave zeros)
        float u[N];
#pragma unroll
        for (int i = 0; i < N; i++) u[i] = nan;
        if (g < G) {
            typedef float part __attribute__((ext_vector_type(N)));
            const part v = *reinterpret_cast<const part *>(ss_row + g);
#pragma unroll
            for (int i = 0; i < N; i++) u[i] = g + i < G ? v[i] : nan;
        }
        // (a zero less one is large; what is not a number is not small)
        uint32_t least = __float_as_uint(u[0]) - 1u;
#pragma unroll
        for (int i = 1; i < N; i++) least = min(least, __float_as_uint(u[i]) - 1u);
        if (ordinary && __all(least >= __float_as_uint(0x1p-70f) - 1u)) {
#pragma unroll
            for (int i = 0; i < N; i++) u[i] = divide(u[i], sum);
        } else {
#pragma unroll
            for (int i = 0; i < N; i++) u[i] = u[i] / rowss;
        }
        uint32_t word = 0;
#pragma unroll
        for (int i = 0; i < N; i++) word |= count_edges<SB>(tree, u[i]) << (SB * i);
        if constexpr (kLanes > 1) word = or_over_lanes<kLanes>(word << (N * SB * (lane & (kLanes - 1))));
        if ((lane & (kLanes - 1)) == 0 && g < G) srow[((uint32_t)g * SB) >> 5] = word;
    }
}
// (the width of a code is the same for all lanes; a branch per row, so that no loop keeps its conditions in registers)
template <int N>
__device__ inline void write_codes(int sb, const float *ss_row, float rowss, const float4 *tree, uint32_t *srow, int G, int first, int waves, int lane)
{
    switch (sb) {
    case 1: write_codes<1, N>(ss_row, rowss, tree, srow, G, first, waves, lane); break;
    case 2: write_codes<2, N>(ss_row, rowss, tree, srow, G, first, waves, lane); break;
    case 4: write_codes<4, N>(ss_row, rowss, tree, srow, G, first, waves, lane); break;
    default: write_codes<8, N>(ss_row, rowss, tree, srow, G, first, waves, lane); break;
    }
}

// A float whose bits are the integer n (subnormal for the n used here): small integers times bytes(1) add and multiply
// exactly, so one fused multiply-add steps a byte address, and its result's bits are the address.
__device__ constexpr float bytes(uint32_t n) { return __builtin_bit_cast(float, n); }

}  // namespace pvq_quantize_dev
