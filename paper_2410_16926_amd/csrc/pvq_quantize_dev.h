// Device code shared by the encoders of groups of up to 32 (Sec. 2.5, Sec. 3.3 Steps 3 to 5).  float32, fixed evaluation
// order: the results are part of the format.  The point: project onto the l1 ball of radius K, round to nearest even, then
// move single pulses on the coordinates of largest deviation (lowest coordinate on ties) until the count is K.  No coordinate
// is ever adjusted twice: for finite input the |sum - K| largest deviations are all positive, and an adjusted coordinate
// drops below -1/2.  So the repair takes one round per pulse, with the deviations formed once.
#pragma once

#include <hip/hip_runtime.h>

namespace pvq_quantize_dev {

// Whether a group's norm l1 is one that all groups but tiny and huge ones have: finite, not zero, and with K / l1 finite for
// every K up to MAX_K.  What is not has to be looked at closely, and what is has a direction.  From a power of two 2^(f - 127)
// on, f the exponent's field, K / l1 <= MAX_K 2^(127 - f), which is finite if MAX_K < 2^(f + 1).  (K / l1 overflows up to
// l1 = K 2^-128, which is 2^-124 for K = 16: above the smallest normal float.)  Up to 2^127, so that infinities and NaN,
// whose bits lie above, are not among them.
__device__ constexpr uint32_t ordinary_norm_from(int max_k)
{
    uint32_t f = 1;
    while (max_k >> (f + 1)) f++;
    return f << 23;
}
template <int MAX_K>
__device__ inline bool ordinary_norm(float l1)
{
    constexpr uint32_t from = ordinary_norm_from(MAX_K), to = 0x7F000000u;
    static_assert(MAX_K / __builtin_bit_cast(float, from) <= __FLT_MAX__, "K over the smallest ordinary norm is finite");
    return __float_as_uint(l1) - from < to - from;
}

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

// The repair of Sec. 2.5 for groups of 8: mag[i] += unit for the coordinates that hold the `need` first places in the order
// of keys (largest first, lower coordinate first on ties; the bits of floats, of which the first `need` are positive).  A
// round takes the largest key left (three-operand maxima), marks the first coordinate that has it and takes its key out; a
// wave runs as many rounds as its lane with the largest `need`, two or three for groups of 8 (counting every coordinate's
// place with 28 comparisons takes a hundred instructions).  The first two rounds keep their marks as masks (scalar registers;
// those of more rounds do not fit there).  Changes key.
__device__ inline void adjust_first_places8(int (&key)[8], float need, float unit, float (&mag)[8])
{
    bool adj[8];
#pragma unroll
    for (int i = 0; i < 8; i++) adj[i] = false;
    auto mark = [&](bool open) {                  // (a lane that needs no more takes nothing)
        const int best = max(max(max(max(key[0], key[1]), key[2]), max(max(key[3], key[4]), key[5])), max(key[6], key[7]));
        bool taken = !open;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const bool equal = key[i] == best;
            adj[i] = adj[i] || (equal && !taken);
            taken = taken || equal;
        }
    };
    mark(need > 0.0f);
    if (__any(need > 1.0f)) {
#pragma unroll
        for (int i = 0; i < 8; i++) key[i] = adj[i] ? INT32_MIN : key[i];
        mark(need > 1.0f);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) mag[i] += adj[i] ? unit : 0.0f;
    if (__any(need > 2.0f)) {
#pragma unroll 1
        for (float round = 2.0f; round < 8.0f && __any(need > round); round += 1.0f) {
#pragma unroll
            for (int i = 0; i < 8; i++) { key[i] = adj[i] ? INT32_MIN : key[i]; adj[i] = false; }
            mark(need > round);
#pragma unroll
            for (int i = 0; i < 8; i++) mag[i] += adj[i] ? unit : 0.0f;
        }
    }
}

// The same repair for any D and signed points (whose zeros have their sign too), in one loop for all rounds: a place that is taken gets the key -1 (below every positive float,
// and the bits of no deviation), which shows at the end where a pulse moved.  A wave runs as many rounds as its lane with the
// largest `need`, about three for D = 16 and five for D = 32.
template <int D>
__device__ inline void adjust_first_places(int (&key)[D], float need, float unit, float (&y)[D])
{
#pragma unroll 1
    for (float round = 0.0f; round < (float)D && __any(need > round); round += 1.0f) {
        int best = max(key[0], key[1]);
#pragma unroll
        for (int i = 2; i < D; i += 2) best = max(max(best, key[i]), key[i + 1]);
        bool taken = !(need > round);             // (a lane that needs no more takes nothing)
#pragma unroll
        for (int i = 0; i < D; i++) {
            const bool equal = key[i] == best;
            key[i] = equal && !taken ? -1 : key[i];
            taken = taken || equal;
        }
    }
#pragma unroll
    for (int i = 0; i < D; i++) y[i] = copysignf(fabsf(y[i]) + (key[i] == -1 ? unit : 0.0f), y[i]);
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

// OR of v over aligned runs of N lanes (N = 4, 8, 16, 32), in every lane of the run: the first four levels by lane
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
    v = dpp_or<0x4E>(v);                              // quad_perm [2,3,0,1]
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

// The row's amplitude codes (Sec. 3.3 Step 5): code = number of quantile edges <= u, u = ss_g / rowss, packed 32/SB lanes to
// a dword by an OR butterfly.  first, step: the lane's first group and the distance to its next.
template <int SB>
__device__ inline void write_codes(const float *ss_row, float rowss, const float4 *tree, uint32_t *srow, int G, int first, int step, int lane)
{
    for (int g = first; g - lane < G; g += step) {
        const float ss = g < G ? ss_row[g] : __builtin_nanf("");          // (no edge is reached: absent groups leave zeros)
        const uint32_t code = count_edges<SB>(tree, ss / rowss);
        const uint32_t word = or_over_lanes<32 / SB>(code << ((lane * SB) & 31));
        if ((lane & (32 / SB - 1)) == 0 && g < G) srow[((uint32_t)g * SB) >> 5] = word;
    }
}
// (the width of a code is the same for all lanes; a branch per row, so that no loop keeps its conditions in registers)
__device__ inline void write_codes(int sb, const float *ss_row, float rowss, const float4 *tree, uint32_t *srow, int G, int first, int step, int lane)
{
    switch (sb) {
    case 1: write_codes<1>(ss_row, rowss, tree, srow, G, first, step, lane); break;
    case 2: write_codes<2>(ss_row, rowss, tree, srow, G, first, step, lane); break;
    case 4: write_codes<4>(ss_row, rowss, tree, srow, G, first, step, lane); break;
    default: write_codes<8>(ss_row, rowss, tree, srow, G, first, step, lane); break;
    }
}

// A float whose bits are the integer n (subnormal for the n used here): small integers times bytes(1) add and multiply
// exactly, so one fused multiply-add steps a byte address, and its result's bits are the address.
__device__ constexpr float bytes(uint32_t n) { return __builtin_bit_cast(float, n); }

}  // namespace pvq_quantize_dev
