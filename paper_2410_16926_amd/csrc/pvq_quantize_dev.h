// Device code shared by the kernels that quantise a group onto the pyramid (Sec. 2.5): the encoders and
// the error correction of Sec. 3.3 Step 6.  float32, fixed evaluation order: the results are part of the
// format.  The point: project onto the l1 ball of radius K, round to nearest even, then move single pulses on
// the coordinates of largest deviation (lowest coordinate on ties) until the count is K.  quantize_group8 finds
// it without branches for D = 8 (count_wins); the D = 8 encoder and quantize_group_select<D>, for any D, take one
// round per pulse to move (adjust_first_places8 for D = 8).
#pragma once

#include <hip/hip_runtime.h>

namespace pvq_quantize_dev {

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

// Position of every coordinate in the order of keys (largest first, lower coordinate first on
// ties): wins[i] = number of coordinates that i comes before.  One comparison per pair feeds two
// counters through its carry: i's wins over later coordinates and j's losses against earlier ones.
__device__ inline void count_wins(const float (&key)[8], int (&wins)[8])
{
    constexpr int D = 8;
    int lose[D];
#pragma unroll
    for (int i = 0; i < D; i++) { wins[i] = 0; lose[i] = 0; }
#pragma unroll
    for (int i = 0; i < D; i++)
#pragma unroll
        for (int j = i + 1; j < D; j++) {
            const int first = key[i] >= key[j] ? 1 : 0;
            wins[i] += first;
            lose[j] += first;
        }
#pragma unroll
    for (int j = 0; j < D; j++) wins[j] += j - lose[j];   // j beat every earlier coordinate it did not lose to
}

// The repair of Sec. 2.5 for groups of 8: mag[i] += unit for the coordinates that hold the `need` first places in the order
// of keys (largest first, lower coordinate first on ties; the bits of floats, of which the first `need` are positive).  A
// round takes the largest key left (three-operand maxima), marks the first coordinate that has it and takes its key out; a
// wave runs as many rounds as its lane with the largest `need`, two or three for groups of 8, against a hundred
// instructions for count_wins: the form for kernels that are short of vector instructions (the encoders).  The first two
// rounds keep their marks as masks (scalar registers; those of more rounds do not fit there).  Changes key.
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

// Groups of 8 without branches (for the error correction, whose waves wait for one group after the other: rounds
// with a wave-wide vote measured 2 % slower there): the coordinates' places in the order of deviations are counted
// with 28 comparisons and the |sum - K| first places are adjusted, which equals the one-at-a-time repair because no
// coordinate is ever adjusted twice (for finite input the |sum - K| largest deviations are all positive, and an
// adjusted coordinate drops below -1/2).  Returns the sum of squares; y gets the signed point.  Weights that are
// not finite give (0, ..., 0, K).
__device__ inline float quantize_group8(const float (&w)[8], int K, int (&y)[8])
{
    constexpr int D = 8;
    float a[D], tmp[D];
#pragma unroll
    for (int i = 0; i < D; i++) { a[i] = fabsf(w[i]); tmp[i] = a[i]; }
    const float l1 = tree_sum<D>(tmp);
#pragma unroll
    for (int i = 0; i < D; i++) tmp[i] = w[i] * w[i];
    const float ss = tree_sum<D>(tmp);
    const float g = (float)K / l1;
    const bool degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(g < INFINITY);
    float t[D], yf[D];
    float S = 0.0f;
#pragma unroll
    for (int i = 0; i < D; i++) {
        t[i] = a[i] * g;
        yf[i] = rintf(t[i]);
        S += yf[i];                       // small integers: exact in any order
    }
    const float m = (float)K - S;         // > 0: pulses to add, < 0: pulses to take away
    float key[D];
#pragma unroll
    for (int i = 0; i < D; i++) {
        const float d = t[i] - yf[i];
        key[i] = m < 0.0f ? -d : d;
    }
    int wins[D];
    count_wins(key, wins);
    const int need = (int)fabsf(m);
    const float unit = m < 0.0f ? -1.0f : 1.0f;
    int k = K;
#pragma unroll
    for (int i = 0; i < D; i++) {
        const bool adjust = wins[i] + need >= D;      // place = D-1-wins < need
        int mag = (int)(yf[i] + (adjust ? unit : 0.0f));
        if (degenerate) mag = 0;
        if (i == D - 1) mag = k;                      // the last coordinate takes what is left
        y[i] = (w[i] < 0.0f && !degenerate) ? -mag : mag;
        k -= mag;
    }
    return ss;
}

// The same point for any D, without the two repair loops' re-evaluation of every deviation: the deviations are
// formed once (as keys, negated when pulses have to be taken away), and each of the |sum - K| rounds picks the
// largest key, lowest coordinate on ties, adjusts that coordinate and takes its key out.  This is the one-at-a-time
// repair itself, since an adjusted coordinate never comes up again (see quantize_group8); a wave runs as many rounds
// as its lane with the largest |sum - K| needs, two to five for D = 16 and 32 (re-evaluating all deviations in every
// round, in one loop for pulses to take away and one for pulses to add, took 2.5 times the instructions).
// Weights that are not finite give (0, ..., 0, K).
template <int D>
__device__ inline float quantize_group_select(const float (&w)[D], int K, int (&y)[D])
{
    float a[D], tmp[D];
#pragma unroll
    for (int i = 0; i < D; i++) { a[i] = fabsf(w[i]); tmp[i] = a[i]; }
    const float l1 = tree_sum<D>(tmp);
#pragma unroll
    for (int i = 0; i < D; i++) tmp[i] = w[i] * w[i];
    const float ss = tree_sum<D>(tmp);
    const float g = (float)K / l1;
    const bool degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(g < INFINITY);
    float key[D], yf[D];
    float S = 0.0f;
#pragma unroll
    for (int i = 0; i < D; i++) {
        const float t = a[i] * g;
        yf[i] = rintf(t);
        S += yf[i];                       // small integers: exact in any order
        key[i] = t - yf[i];
    }
    const float m = (float)K - S;         // > 0: pulses to add, < 0: pulses to take away
    const float unit = m < 0.0f ? -1.0f : 1.0f;
    if (m < 0.0f) {
#pragma unroll
        for (int i = 0; i < D; i++) key[i] = -key[i];
    }
    const int need = degenerate ? 0 : (int)fminf(fabsf(m), (float)D);
    for (int round = 0; round < D; round++) {
        if (!__any(round < need)) break;
        float best = key[0];
        int at = 0;
#pragma unroll
        for (int i = 1; i < D; i++) {
            const bool take = key[i] > best;
            best = take ? key[i] : best;
            at = take ? i : at;
        }
        if (round < need) {
#pragma unroll
            for (int i = 0; i < D; i++) {
                const bool hit = i == at;
                yf[i] += hit ? unit : 0.0f;
                key[i] = hit ? -INFINITY : key[i];
            }
        }
    }
    int k = K;
#pragma unroll
    for (int i = 0; i < D; i++) {
        int mag = degenerate ? 0 : (int)yf[i];
        if (i == D - 1) mag = k;                      // the last coordinate takes what is left
        y[i] = (w[i] < 0.0f && !degenerate) ? -mag : mag;
        k -= mag;
    }
    return ss;
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

}  // namespace pvq_quantize_dev
