// PVQ of long groups, D = 64 or 128 values with indices of up to 512 bits: the setting of on-the-fly
// quantisation of activations (Sec. 3.2, Sec. 4.3), e.g. D = 128, K = 187 for
// 3 bits per value (384-bit indices).  Amplitudes are float32 (Sec. 3.3 Step 5 quantises them only for
// small groups).  The size table no longer fits LDS (1.2 MB for (128,187)); it is read from device
// memory, where the L2 keeps it.
//
// One table of W-word integers (W = 4, 8, 12 or 16) serves both directions: the thresholds T_j of every row
// (pvq_internal.h), of which a coordinate of the point is one, so that N(D,K) - 1 - index is the sum over the
// coordinates.
//
// Encoding (Sec. 2.5 for the point, App. B.2 for its index): 16 lanes per group, lane l holds coordinates
// CP*l .. CP*l+CP-1 (CP = D/16).  The quantiser's sums run over adjacent pairs level by level (in the
// lane, then across lanes by data-parallel-primitive moves, no LDS traffic), the repair of the pulse
// count takes the largest deviation of the group per step (lowest coordinate on ties).  The index is a sum of
// per-coordinate thresholds that depend on the coordinate's magnitude, sign and the pulses left before it only; a
// prefix sum over the magnitudes gives the latter.
//
// Decoding (App. B.3): coordinate by coordinate, q = N(D,K) - 1 - index first; a coordinate is the last
// threshold of its row that is not above q, and q loses it.  Few groups: a wave per group
// (decode_wide_wave_kernel); many: a lane per group, the rows in LDS (decode_wide_rows_kernel) or, for many pulses (rows_in_lds), in
// device memory (decode_wide_kernel).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cmath>

#include "pvq_exact_dev.h"
#include "pvq_hadamard_dev.h"
#include "pvq_internal.h"

namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// A lane's value moved by one data-parallel-primitive pattern; lanes whose row is not in ROWS, or whose
// source lies outside their row, get `idle`.
template <int CTRL, int ROWS = 0xF>
__device__ inline uint32_t dpp_move(uint32_t v, uint32_t idle = 0)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)idle, (int)v, CTRL, ROWS, 0xF, false);
}

// The six steps that bring a combination of all 64 lanes' values to lane 63: lane^1, lane^2 (quad
// permutations), the other quad of the half row and the other half of the row (mirror patterns: the
// partner holds the same value as every lane of its group by then), row 0 into 1 and 2 into 3, rows 0..1
// into 2..3.  No LDS traffic.
#define PVQ_WAVE_STEPS(STEP)                                       \
    STEP(0xB1, 0xF) STEP(0x4E, 0xF) STEP(0x141, 0xF) STEP(0x140, 0xF) STEP(0x142, 0xA) STEP(0x143, 0xC)

struct encode_wide_params {
    const void *X;
    int64_t ldx, groups, index_row_words;
    int K, bits, tile_groups, tiles_per_row, ls;
    const uint32_t *tab_t;   // thresholds [D][row_len][W]
    int row_len;
    uint32_t last_index[16]; // N(D,K) - 1
    uint32_t *index_out;
    float *scale_out;
    int8_t *pulses_out;
    int64_t cols;
};

// Encoding, 16 lanes per group and four groups per wave (lane = 16 * group + sub, sub holds coordinates CP*sub ..
// CP*sub+CP-1, CP = D/16): the sums, the largest deviation, the prefix sum and the multi-word total need four cross-lane
// levels, all of them permutations inside a row of 16 lanes after which every lane of the row holds the result, and a lane's
// own coordinates (four or eight) are independent work in between.
// Bound by instructions (906 on the vector and 155 on the scalar unit a wave at D = 128, K = 187, with the rotation in front)
// and the gathers of thresholds.  2048 rows of 8192 rotated and encoded: 79 us, K = 84: 54 us; 2048 x 8192 encoded, D = 64,
// K = 96: 44 us from bfloat16, 45 from float32.  With the places of the repair marked in every step, general division and root
// (1025 and 254 instructions): 84, 59, 44 and 47 us; with 90 instructions a step besides, and a lane reading all of an entry's
// pieces: 101, 100, 64 (bfloat16).  A wave per group, the form of small batches before: 7.7 and 11 us for 32 and 4096 groups
// (D = 128, K = 187), this one 6.9 and 7.7.
#define PVQ_ROW_STEPS(STEP) STEP(0xB1) STEP(0x4E) STEP(0x141) STEP(0x140)

__device__ inline float row_sum_pairs(float v)
{
#define PVQ_STEP(CTRL) v = v + __uint_as_float(dpp_move<CTRL>(__float_as_uint(v)));
    PVQ_ROW_STEPS(PVQ_STEP)
#undef PVQ_STEP
    return v;
}
// sum of CP values over adjacent pairs, level by level
template <int CP>
__device__ inline float tree_sum(const float (&x)[CP])
{
    float t[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) t[j] = x[j];
#pragma unroll
    for (int st = 1; st < CP; st *= 2)
#pragma unroll
        for (int j = 0; j < CP; j += 2 * st) t[j] = t[j] + t[j + st];
    return t[0];
}

// One group of 16 * CP values held by 16 lanes (lane `sub` of the group: coordinates CP*sub .. CP*sub+CP-1):
// the point, the amplitude, the index, and the index's words into the tile's bit stream in LDS at group
// position gl.  `on` = false: the lanes go through the motions (every cross-lane step needs them) and
// write nothing.  K and D = 16 * CP as in the context.  DISTINCT: deviations are seldom equal (float32 values: bfloat16 ones
// often have the same magnitude twice in a group).
template <int CP, int W, bool DISTINCT>
__device__ inline void encode_group16(const float (&w)[CP], int sub, bool on, int gl, int64_t row, int64_t g,
                                      const encode_wide_params &p, uint32_t *stream, int tile_words)
{
    constexpr int D = 16 * CP;
    // ---- the point (Sec. 2.5): the magnitudes as floats, which add and multiply at twice the rate of integers
    const float K = (float)p.K;
    float tmp[CP], t[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) tmp[j] = fabsf(w[j]);
    const float l1 = row_sum_pairs(tree_sum<CP>(tmp));
#pragma unroll
    for (int j = 0; j < CP; j++) tmp[j] = w[j] * w[j];
    const float ss = row_sum_pairs(tree_sum<CP>(tmp));
    // no direction: the point is (0, ..., 0, +K), zeros here until the pulses have been moved  (looked at, and the general
    // division and root taken, only where a group's norm is not between 2^-40 and 2^46: between them its sum of squares lies
    // between 2^-87 and 2^92.  bfloat16 sources: always, the two forms beside the steps below cost them 1 %)
    const bool ordinary = DISTINCT && __all(pvq_exact_dev::magnitude_in(l1, 0x1p-40f, 0x1p46f));
    float gain = pvq_exact_dev::integer_over(K, l1);
    bool degenerate = false;
    if (!ordinary) {
        gain = K / l1;
        degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(gain < INFINITY);
    }
    const bool any_degenerate = !ordinary && __any(degenerate);
#pragma unroll
    for (int j = 0; j < CP; j++) t[j] = fabsf(w[j]) * gain;
    if (any_degenerate) {
#pragma unroll
        for (int j = 0; j < CP; j++) t[j] = degenerate ? 0.0f : t[j];
    }
    float m[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) { m[j] = rintf(t[j]); tmp[j] = m[j]; }
    // pulses to add (> 0) or to take away (< 0)   (small integers: exact in any order)
    const float miss = (degenerate ? 0.0f : K) - row_sum_pairs(tree_sum<CP>(tmp));
    const float unit = miss < 0.0f ? -1.0f : 1.0f, need = fabsf(miss);
    // deviations (negated where pulses have to go), as bits of floats: the `need` largest are positive
    int key[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) key[j] = (int)__float_as_uint((t[j] - m[j]) * unit);
    if constexpr (DISTINCT) {
        // The largest, the largest below it, ...: with `last` the one before, key - last as an unsigned number is largest for the
        // first key below it.  After as many steps as the group has pulses to move, the keys not below the last are moved,
        // unless some of them were equal: then the sum tells.  (The wave goes on while any of its four groups has a step left,
        // about five at D = 128; a step's masks on the scalar unit cost as much as its vector instructions, and this has none.)
        uint32_t place[CP];
#pragma unroll
        for (int j = 0; j < CP; j++) place[j] = (uint32_t)max(key[j], 0);
        uint32_t last = 0x80000000u;                // (above all of them)
#pragma unroll 1
        for (float step = 0.0f; step < (float)D && __any(need > step); step += 1.0f) {
            uint32_t next = max(place[0] - last, place[1] - last);
#pragma unroll
            for (int j = 2; j < CP; j += 2) next = max(max(next, place[j] - last), place[j + 1] - last);
#define PVQ_STEP(CTRL) next = max(next, dpp_move<CTRL>(next));
            PVQ_ROW_STEPS(PVQ_STEP)
#undef PVQ_STEP
            last = need > step ? last + next : last;
        }
        float moved[CP];
#pragma unroll
        for (int j = 0; j < CP; j++) {
            moved[j] = m[j] + (place[j] >= last ? unit : 0.0f);
            tmp[j] = moved[j];
        }
        if (!__all(row_sum_pairs(tree_sum<CP>(tmp)) == (degenerate ? 0.0f : K))) {
            // Equal deviations, so that too many are not below `last`: it goes up again while those above it are enough.  (A
            // group with fewer different deviations than pulses to move has come to its largest again, and starts at the lowest.)
            // Taking every step again with masks instead, 2048 x 8192 float32 values that are bfloat16's, K = 84: 53.8 us, now
            // 47.0; 64 x 8192 of which one in a thousand is not zero, rotated: 17.2, now 14.5.
            auto count = [&](auto is) {
                float n = 0.0f;
#pragma unroll
                for (int j = 0; j < CP; j++) n += is(place[j]) ? 1.0f : 0.0f;
                return n;
            };
            float above = row_sum_pairs(count([&](uint32_t v) { return v >= last; })), equal;
            if (above < need) { last = 0; above = (float)D; }
            for (bool up = true; __any(up);) {
                equal = row_sum_pairs(count([&](uint32_t v) { return v == last; }));
                uint32_t next = ~0u;
#pragma unroll
                for (int j = 0; j < CP; j++) next = min(next, place[j] > last ? place[j] : ~0u);
#define PVQ_STEP(CTRL) next = min(next, dpp_move<CTRL>(next));
                PVQ_ROW_STEPS(PVQ_STEP)
#undef PVQ_STEP
                up = above > need && above - equal >= need;
                last = up ? next : last;
                above -= up ? equal : 0.0f;
            }
            // of those equal to `last` the lowest coordinates, as many as are missing: the lane's share is what the lanes in front
            // of it leave
            float incl = count([&](uint32_t v) { return v == last; });
            const float mine = incl;
            incl += __uint_as_float(dpp_move<0x111>(__float_as_uint(incl)));        // row_shr:1
            incl += __uint_as_float(dpp_move<0x112>(__float_as_uint(incl)));        // row_shr:2
            incl += __uint_as_float(dpp_move<0x114>(__float_as_uint(incl)));        // row_shr:4
            incl += __uint_as_float(dpp_move<0x118>(__float_as_uint(incl)));        // row_shr:8
            float left = need - (above - equal) - (incl - mine);
#pragma unroll
            for (int j = 0; j < CP; j++) {
                const bool is = place[j] == last;
                moved[j] = m[j] + (place[j] > last || (is && left > 0.0f) ? unit : 0.0f);
                left -= is ? 1.0f : 0.0f;
            }
        }
#pragma unroll
        for (int j = 0; j < CP; j++) m[j] = moved[j];
    } else {
        // One pulse per step and group on the largest deviation, lowest coordinate on ties; none comes up twice (a place taken
        // gets the key -1, the bits of no deviation).
#pragma unroll 1
        for (float step = 0.0f; step < (float)D && __any(need > step); step += 1.0f) {
            const bool open = need > step;      // the same in the 16 lanes of a group
            int largest = max(key[0], key[1]);
#pragma unroll
            for (int j = 2; j < CP; j += 2) largest = max(max(largest, key[j]), key[j + 1]);
            int best = largest;
#define PVQ_STEP(CTRL) best = max(best, (int)dpp_move<CTRL>((uint32_t)best, 0x80000000u));
            PVQ_ROW_STEPS(PVQ_STEP)
#undef PVQ_STEP
            bool taken = !(open && largest == best);
            if (16 * __popcll(__ballot(!taken)) != __popcll(__ballot(open))) {      // a tie between lanes of a group
                int first = taken ? 16 : sub;
#define PVQ_STEP(CTRL) first = min(first, (int)dpp_move<CTRL>((uint32_t)first, 0x7FFFFFFFu));
                PVQ_ROW_STEPS(PVQ_STEP)
#undef PVQ_STEP
                taken = taken || first != sub;
            }
#pragma unroll
            for (int j = 0; j < CP; j++) {
                const bool equal = key[j] == best;
                key[j] = equal && !taken ? -1 : key[j];
                taken = taken || equal;
            }
        }
#pragma unroll
        for (int j = 0; j < CP; j++) m[j] += key[j] == -1 ? unit : 0.0f;
    }
    float y[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) {
        y[j] = copysignf(m[j], w[j]);
    }
    if (any_degenerate && degenerate && sub == 15) {
        m[CP - 1] = K;
        y[CP - 1] = K;                       // (positive whatever the value's sign)
    }

    // ---- amplitude (Sec. 2.3, or Sec. 3.3 Step 4)
    float amp;
    if (p.ls) {
        float pr[CP];
#pragma unroll
        for (int j = 0; j < CP; j++) {
            pr[j] = y[j] * w[j];
            tmp[j] = m[j] * m[j];
        }
        if (any_degenerate) {
            // zeros of the point are positive (the sign of a sum of zeros is theirs)
#pragma unroll
            for (int j = 0; j < CP; j++) pr[j] = m[j] == 0.0f ? 0.0f * w[j] : pr[j];
        }
        amp = row_sum_pairs(tree_sum<CP>(pr)) / sqrtf(row_sum_pairs(tree_sum<CP>(tmp)));
    } else {
        amp = ordinary ? pvq_exact_dev::root_of(ss) : sqrtf(ss);
    }
    if (on && sub == 0) p.scale_out[row * p.groups + g] = amp;
    if (on && p.pulses_out) {
#pragma unroll
        for (int j = 0; j < CP; j++) p.pulses_out[row * p.cols + g * D + CP * sub + j] = (int8_t)(int)y[j];
    }

    // ---- the index (App. B.2): the bytes of the coordinates' thresholds in the table, as floats whose bits are the integers
    // (below 2^24, to which they add and multiply exactly)
    constexpr uint32_t kEntry = 4 * W;
    const uint32_t row_bytes = (uint32_t)p.row_len * kEntry;
    float mine = tree_sum<CP>(m), incl = mine;   // inclusive prefix sum over the 16 lanes of the group
    incl += __uint_as_float(dpp_move<0x111>(__float_as_uint(incl)));        // row_shr:1
    incl += __uint_as_float(dpp_move<0x112>(__float_as_uint(incl)));        // row_shr:2
    incl += __uint_as_float(dpp_move<0x114>(__float_as_uint(incl)));        // row_shr:4
    incl += __uint_as_float(dpp_move<0x118>(__float_as_uint(incl)));        // row_shr:8
    float left = K - (incl - mine);              // pulses left in front of the lane's first coordinate
    float trow = __uint_as_float((uint32_t)(D - 1 - CP * sub) * row_bytes);
    uint32_t from[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) {
        left -= m[j];
        const float k = __builtin_amdgcn_fmed3f(left, 0.0f, K);              // (in range whatever the input)
        const float positive = __builtin_amdgcn_fmed3f(y[j], 0.0f, 1.0f);
        from[j] = __float_as_uint(fmaf(positive, __uint_as_float(kEntry), fmaf(k, __uint_as_float(2 * kEntry), trow)));
        trow -= __uint_as_float(row_bytes);
    }
    // An entry is read by neighbouring lanes, 16 bytes each: a gather of 16 bytes a lane costs the vector memory path a cycle
    // per lane, three of them for an entry of 12 words, and the lanes of a quad beside one another little more than one for
    // all.  So lane i of a quad adds up piece i (of two pieces: i mod 2) of its quad's entries, with a word for what overflows.
    constexpr int NP = W / 4, kLanes = NP == 3 ? 4 : NP;
    const int i4 = sub & 3, piece = kLanes == 4 ? min(i4, NP - 1) : i4 & (kLanes - 1);
    uint32_t acc[5] = {};
    const unsigned char *base = reinterpret_cast<const unsigned char *>(p.tab_t);
    u32x4 e[2][kLanes];
    auto request = [&](u32x4 (&e)[kLanes], uint32_t at) {
        uint32_t a[kLanes];
        if constexpr (kLanes == 4) {
            a[0] = dpp_move<0x00>(at); a[1] = dpp_move<0x55>(at); a[2] = dpp_move<0xAA>(at); a[3] = dpp_move<0xFF>(at);
        } else if constexpr (kLanes == 2) {
            a[0] = dpp_move<0x50>(at); a[1] = dpp_move<0xFA>(at);             // lanes 0 0 1 1, 2 2 3 3
        } else {
            a[0] = at;
        }
#pragma unroll
        for (int l = 0; l < kLanes; l++) e[l] = *reinterpret_cast<const u32x4 *>(base + (a[l] + 16u * piece));
    };
    auto add5 = [&](uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t w4) {
        uint32_t c;
        acc[0] = __builtin_addc(acc[0], w0, 0u, &c);
        acc[1] = __builtin_addc(acc[1], w1, c, &c);
        acc[2] = __builtin_addc(acc[2], w2, c, &c);
        acc[3] = __builtin_addc(acc[3], w3, c, &c);
        acc[4] = __builtin_addc(acc[4], w4, c, &c);
    };
    request(e[0], from[0]);
#pragma unroll
    for (int j = 0; j < CP; j++) {
        if (j + 1 < CP) request(e[(j + 1) & 1], from[j + 1]);
#pragma unroll
        for (int l = 0; l < kLanes; l++) add5(e[j & 1][l].x, e[j & 1][l].y, e[j & 1][l].z, e[j & 1][l].w, 0u);
    }
#define PVQ_STEP(CTRL) add5(dpp_move<CTRL>(acc[0]), dpp_move<CTRL>(acc[1]), dpp_move<CTRL>(acc[2]), dpp_move<CTRL>(acc[3]), dpp_move<CTRL>(acc[4]));
    if constexpr (kLanes < 2) { PVQ_STEP(0xB1) }
    if constexpr (kLanes < 4) { PVQ_STEP(0x4E) }
    PVQ_STEP(0x124) PVQ_STEP(0x128)              // the quads of the group: rotations by 4 and 8
#undef PVQ_STEP

    // N(D,K) - 1 less the sum: every piece by itself, then what it owes the next
    uint32_t d[4], owed = 0;
#pragma unroll
    for (int x = 0; x < 4; x++) {
        uint32_t last = p.last_index[x];
#pragma unroll
        for (int n = 1; n < NP; n++) last = i4 == n ? p.last_index[4 * n + x] : last;
        d[x] = __builtin_subc(last, acc[x], owed, &owed);
    }
    owed += acc[4];
#pragma unroll
    for (int n = 1; n < NP; n++) {
        uint32_t c, in = dpp_move<0x90>(owed);                               // of the lane before in the quad (all lanes move)
        in = i4 == 0 ? 0u : in;
        d[0] = __builtin_subc(d[0], in, 0u, &c);
        d[1] = __builtin_subc(d[1], 0u, c, &c);
        d[2] = __builtin_subc(d[2], 0u, c, &c);
        d[3] = __builtin_subc(d[3], 0u, c, &owed);
    }
    // ---- into the tile's bit stream: of quad x, lane i takes word 4 i + x of the index, the last of them what it shifts out
    const int quad = sub >> 2;
    uint32_t before = dpp_move<0x90>(d[3]);
    before = i4 == 0 ? 0u : before;
    const uint32_t word = quad == 0 ? d[0] : quad == 1 ? d[1] : quad == 2 ? d[2] : d[3];
    const uint32_t prev = quad == 0 ? before : quad == 1 ? d[0] : quad == 2 ? d[1] : d[2];
    const int off = gl * p.bits, sh = off & 31, w0 = off >> 5, at = 4 * i4 + quad;
    const uint32_t out = sh ? (word << sh) | (prev >> (32 - sh)) : word;
    if (on && at < W && w0 + at < tile_words && out) atomicOr(&stream[w0 + at], out);
    const uint32_t over = sh ? word >> (32 - sh) : 0u;
    if (on && at == W - 1 && w0 + W < tile_words && over) atomicOr(&stream[w0 + W], over);
}

template <int TIN, int CP, int W>
__global__ __launch_bounds__(512) void encode_wide16_kernel(encode_wide_params p)
{
    extern __shared__ __align__(16) uint32_t stream[];
    constexpr int D = 16 * CP;
    const int lane = threadIdx.x & 63, sub = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int64_t row = blockIdx.x / p.tiles_per_row;
    const int tile = blockIdx.x - (int)(row * p.tiles_per_row);
    const int64_t g0 = (int64_t)tile * p.tile_groups;
    const int ng = (int)min((int64_t)p.tile_groups, p.groups - g0);
    const int tile_words = (int)(((int64_t)ng * p.bits + 31) / 32);
    const int64_t first_word = g0 * p.bits / 32;   // exact: tile_groups * bits is a multiple of 32

    for (int i = threadIdx.x; i < tile_words; i += blockDim.x) stream[i] = 0;
    __syncthreads();

    for (int gi = 4 * wave; gi < ng; gi += 4 * nwaves) {
        const int gl = gi + quarter;           // this quarter's group inside the tile
        const bool on = gl < ng;               // quarters beyond the tile work on its first group again, unused
        const int64_t g = g0 + (on ? gl : gi);
        float w[CP];
        if constexpr (TIN == PVQ_F32) {
            const float4 *src = reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(p.X) + row * p.ldx + g * D + CP * sub);
#pragma unroll
            for (int j = 0; j < CP / 4; j++) {
                const float4 v = src[j];
                w[4 * j] = v.x; w[4 * j + 1] = v.y; w[4 * j + 2] = v.z; w[4 * j + 3] = v.w;
            }
        } else {
            const uint2 *src = reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(p.X) + row * p.ldx + g * D + CP * sub);
#pragma unroll
            for (int j = 0; j < CP / 4; j++) {
                const uint2 v = src[j];
                w[4 * j] = __uint_as_float(v.x << 16); w[4 * j + 1] = __uint_as_float(v.x & 0xFFFF0000u);
                w[4 * j + 2] = __uint_as_float(v.y << 16); w[4 * j + 3] = __uint_as_float(v.y & 0xFFFF0000u);
            }
        }

        encode_group16<CP, W, TIN == PVQ_F32>(w, sub, on, gl, row, g, p, stream, tile_words);
    }
    __syncthreads();
    uint32_t *dst = p.index_out + row * p.index_row_words + first_word;
    for (int i = threadIdx.x; i < tile_words; i += blockDim.x) dst[i] = stream[i];
}

// Rotation and quantisation of activations in one kernel (Sec. 3.3 Step 1 in front of the encoder): a
// workgroup of L lanes takes 8L consecutive values of a row, 8 per lane, runs the block Walsh-Hadamard
// transform of the rotation kernel on them (same stages, same order, float32), and, since a lane ends with
// 8 consecutive rotated values, 16 neighbouring lanes hold one group of 128: the group encoder above
// takes them from the registers.  The rotated values are never written.
struct rotate_encode_params {
    const void *X;
    int64_t ldx, cols;
    int log2n, chunks_per_row;
    const uint8_t *signs;
    float scale;
    encode_wide_params e;
};

template <int TIN, int W, int LOG2N>
__global__ __launch_bounds__(1024, 8) void rotate_encode16_kernel(rotate_encode_params p)
{
    extern __shared__ __align__(16) float smem[];
    const int L = blockDim.x;
    const int lane = threadIdx.x;
    const int64_t row = blockIdx.x / p.chunks_per_row;
    const int chunk = blockIdx.x - (int)(row * p.chunks_per_row);
    const int64_t col0 = (int64_t)chunk * 8 * L + 8 * pvq_hadamard_dev::load_lane<LOG2N>(lane);   // first of the 8 columns that the lane loads
    const bool live = col0 < p.cols;                           // whole blocks and groups: a lane is in or out

    float v[8];
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = 0.0f;
    if (live) {
        if constexpr (TIN == PVQ_F32) {
            const float *src = reinterpret_cast<const float *>(p.X) + row * p.ldx + col0;
            const float4 a = *reinterpret_cast<const float4 *>(src), b = *reinterpret_cast<const float4 *>(src + 4);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        } else {
            const uint4 q = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(p.X) + row * p.ldx + col0);
            const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                v[2 * j] = __uint_as_float(u[j] << 16);
                v[2 * j + 1] = __uint_as_float(u[j] & 0xFFFF0000u);
            }
        }
        if (p.signs) {
            const uint2 bits = pvq_hadamard_dev::sign_bits(*reinterpret_cast<const uint2 *>(p.signs + col0));
#pragma unroll
            for (int j = 0; j < 8; j++) v[j] = pvq_hadamard_dev::with_sign(v[j], bits, j);
        }
    }
    pvq_hadamard_dev::hadamard_stages<LOG2N, false>(v, lane, p.log2n, smem);
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = v[j] * p.scale;

    // the chunk's groups are a tile of the index plane (whole words: the host checks it)
    uint32_t *stream = reinterpret_cast<uint32_t *>(smem) + (LOG2N > 9 ? pvq_hadamard_dev::pad(8u * (uint32_t)L) + 1u : 0u);
    const int per_chunk = L / 16;
    const int64_t g0 = (int64_t)chunk * per_chunk;
    const int ng = (int)min((int64_t)per_chunk, p.e.groups - g0);
    const int tile_words = ng > 0 ? (int)(((int64_t)ng * p.e.bits + 31) / 32) : 0;
    const int64_t first_word = g0 * p.e.bits / 32;
    for (int i = threadIdx.x; i < tile_words; i += blockDim.x) stream[i] = 0;
    __syncthreads();
    const int sub = lane & 15, gl = lane >> 4;
    const bool on = gl < ng;
    encode_group16<8, W, true>(v, sub, on, gl, row, g0 + (on ? gl : 0), p.e, stream, tile_words);
    __syncthreads();
    uint32_t *dst = p.e.index_out + row * p.e.index_row_words + first_word;
    for (int i = threadIdx.x; i < tile_words; i += blockDim.x) dst[i] = stream[i];
}

struct decode_wide_params {
    const uint32_t *index;
    const float *scale;
    int64_t groups, total_groups, index_row_words, ldw;
    int K, bits, row_len, key_len, buckets, out_dtype;
    const uint32_t *tab_t, *tab_key;
    const uint16_t *tab_guess;
    const double *tab_near;
    uint32_t last_index[16];
    void *W_out;
    int64_t first_group;       // of the launch (decode_wide_rows_kernel)
};

// word i of the W-word index of group g of a row (zero beyond the index)
__device__ inline uint32_t index_word(const uint32_t *row, const decode_wide_params &p, int64_t g, int i)
{
    const int left = p.bits - 32 * i;
    const int64_t at = g * p.bits + 32 * i, wi = at >> 5;
    const int sh = (int)(at & 31);
    // (both words are read whatever the field needs, inside the row: no read waits for another)
    const uint32_t lo = row[std::min(wi, p.index_row_words - 1)], hi = row[std::min(wi + 1, p.index_row_words - 1)];
    const uint32_t v = __builtin_amdgcn_alignbit(hi, lo, sh);
    return left >= 32 ? v : left <= 0 ? 0u : v & ((1u << left) - 1u);
}

// CP neighbouring values of a decoded group
template <int CP>
__device__ inline void store_values(const decode_wide_params &p, int64_t at, const float (&v)[CP])
{
    if (p.out_dtype == PVQ_F32) {
        float *o = reinterpret_cast<float *>(p.W_out) + at;
        if constexpr (CP == 2) *reinterpret_cast<float2 *>(o) = make_float2(v[0], v[1]);
        else o[0] = v[0];
    } else if (p.out_dtype == PVQ_F16) {
        __half *o = reinterpret_cast<__half *>(p.W_out) + at;
        if constexpr (CP == 2) *reinterpret_cast<__half2 *>(o) = __halves2half2(__float2half_rn(v[0]), __float2half_rn(v[1]));
        else o[0] = __float2half_rn(v[0]);
    } else {
        uint16_t *o = reinterpret_cast<uint16_t *>(p.W_out) + at;
        const f32x2_t pair = {v[0], CP == 2 ? v[CP - 1] : 0.0f};
        const uint32_t bits = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2_t));
        if constexpr (CP == 2) *reinterpret_cast<uint32_t *>(o) = bits;
        else o[0] = (uint16_t)bits;
    }
}

// ---- many groups: a lane per group -------------------------------------------------------------------

// q of one lane's group.
template <int W>
struct lane_q {
    uint32_t q[W];

    // pvq_wide_key of q, which lies below 2^(32 WP); `lower`: its leading word is not among the upper four, and it has another key
    template <int WP>
    __device__ inline uint32_t key_of_q(bool &lower) const
    {
        constexpr int w1 = WP > 1 ? WP - 2 : 0, w2 = WP > 2 ? WP - 3 : 0, w3 = WP > 3 ? WP - 4 : 0;
        uint32_t a = q[WP - 1], b = WP > 1 ? q[w1] : 0u;
        int length = 32 * WP;
        if (WP > 2) {
            const bool none = a == 0 && b == 0;                    // both upper words
            const uint32_t c = none ? (WP > 4 ? q[WP > 4 ? WP - 5 : 0] : 0u) : q[w2];
            a = none ? q[w2] : a; b = none ? (WP > 3 ? q[w3] : 0u) : b; length = none ? 32 * (WP - 2) : length;
            const bool second = a == 0;
            a = second ? b : a; b = second ? c : b; length -= second ? 32 : 0;
        } else if (WP > 1) {
            const bool second = a == 0;
            a = second ? b : a; b = second ? 0u : b; length -= second ? 32 : 0;
        }
        const int lead = __builtin_clz(a | 1u);
        const uint32_t from_one = (uint32_t)((((uint64_t)a << 32 | b) << lead) >> 32);   // the 32 bits from the leading one on
        const uint32_t key = __builtin_amdgcn_alignbit((uint32_t)(length - lead), from_one, 10);
        lower = WP > 4 && a == 0;
        return WP > 4 || a != 0 ? key : 0u;
    }
    template <int WP>
    __device__ inline uint32_t key_of_q() const
    {
        bool lower;
        const uint32_t key = key_of_q<WP>(lower);
        return lower ? pvq_wide_key(q, WP) : key;
    }

    // The coordinate's place in a row by the tables in device memory, two dependent trips: the guess of q's bucket, the four
    // keys behind it.  (Equal keys: one too high, which the subtraction shows by its borrow.)
    __device__ inline static uint32_t place_by_guess(const decode_wide_params &p, uint32_t row, uint32_t kq, int k)
    {
        const uint32_t *keys = p.tab_key + row * (uint32_t)p.key_len;
        uint32_t j = p.tab_guess[row * (uint32_t)p.buckets + (kq >> 19 & ~7u) + (kq >> 18 & 7u)];
        uint32_t more;
        do {
            uint32_t ke[4];
            __builtin_memcpy(ke, keys + j + 1, 16);
            more = (ke[0] <= kq ? 1u : 0u) + (ke[1] <= kq ? 1u : 0u) + (ke[2] <= kq ? 1u : 0u) + (ke[3] <= kq ? 1u : 0u);
            j += more;
        } while (__any(more == 4));                                // (ends: the keys behind a row are all ones)
        return min(j, (uint32_t)(2 * k + 1));
    }

    // the first WP words (in whole fours) of threshold j of a row in device memory
    template <int WP>
    __device__ inline static void read_threshold(const decode_wide_params &p, uint32_t row, uint32_t j, uint32_t (&t)[(WP + 3) / 4 * 4])
    {
        const uint32_t *trow = p.tab_t + row * (uint32_t)(p.row_len * W);
#pragma unroll
        for (int x = 0; x < (WP + 3) / 4; x++) {
            const uint4 v = *reinterpret_cast<const uint4 *>(trow + (j * W + 4 * x));
            t[4 * x] = v.x; t[4 * x + 1] = v.y; t[4 * x + 2] = v.z; t[4 * x + 3] = v.w;
        }
    }

    // q -= t, the threshold of place j of the row, or of the place below where that one is above q
    template <int WP>
    __device__ inline void subtract(const decode_wide_params &p, uint32_t row, uint32_t &j, uint32_t (&t)[(WP + 3) / 4 * 4])
    {
        uint32_t br = 0;
#pragma unroll
        for (int x = 0; x < WP; x++) q[x] = __builtin_subc(q[x], t[x], br, &br);
        while (br) {                                               // (ends: T_0 = 0)
            uint32_t c = 0;
#pragma unroll
            for (int x = 0; x < WP; x++) q[x] = __builtin_addc(q[x], t[x], c, &c);
            j--;
            read_threshold<WP>(p, row, j, t);
            br = 0;
#pragma unroll
            for (int x = 0; x < WP; x++) q[x] = __builtin_subc(q[x], t[x], br, &br);
        }
    }
};

// ---- many groups: a lane per group, the rows of the tables in LDS ------------------------------------------
// All lanes of a workgroup are at the same coordinate, so they need the same row, of it the places from their largest 2 k + 1
// down (k pulses left; a coordinate of magnitude m is 2 m places below 2 k), and rows of fewer dimensions in fewer words.  The
// rows go through LDS in turn, brought by a wave of their own, two rows for every barrier; the window is a matter of the
// workgroup's largest and smallest k, looked at every eighth coordinate (k only falls, the margin below covers the rest).
// A coordinate takes three keys (places 3, 7 and 11 below 2 k), the four keys of the block of places they point to, and the
// threshold: three dependent reads of LDS.  A lane whose place is further down, or lies below the window (points that have
// nearly all their pulses in a few coordinates), looks it up in device memory.
// Bound by the walk's chain, about 100 instructions and the three reads a coordinate, 0.41 us of a wave alone; from two waves a
// SIMD on by their issue as well.  D = 128, K = 187, 8192-wide rows, 512 / 1024 / 2048 / 4096 of them: 54 / 60 / 70 / 89 us; with
// every wave requesting its share of every row (45 scalar instructions a coordinate), a barrier for every coordinate, comparisons and
// carries that wait for one another, and three branches where one is now, 72 / 75 / 85 / 110; with guess, keys and thresholds in
// device memory 95 / 100 / 155 / 161.  D = 64, K = 96: 31 / 35 / 46 / 89, before 37 / 41 / 53 / 99 and 55 / 57 / 86 / 104.  Four
// coordinates share a turn of the loop, so that shifts are known when it is compiled.
constexpr int kRowWindow = 256;       // places of a row in LDS
constexpr int kRowMargin = 96;        // of them below the smallest 2 k when the window is set
constexpr int kRowPad = 16;           // keys in front of them: zeros

// A row in LDS: the keys behind their padding, the thresholds.  (The places that step looks for lie at most 17 below the
// window: in the keys.)
constexpr int kPointWords = 19;       // 64 coordinates on their way out: 16 words of magnitudes, 2 of signs, and one for the banks' sake
constexpr uint32_t kRowKeys = 4 * kRowPad, kRowThresholds = kRowKeys + 4 * kRowWindow;
constexpr uint32_t row_bytes(int W) { return kRowThresholds + 4 * kRowWindow * W; }
static_assert(kRowThresholds >= 17 * 4 * 16, "a place below the window");
// Rows in LDS: the present pair's, the next one's, and the pair on its way; with integers of 16 words without the last, so that
// two workgroups fit a unit, with 8 words so that three do (D = 64, K = 96, 2048 / 3072 tokens 46 / 69 us; six rows in LDS 47 / 72).
constexpr int row_slots(int W) { return W == 8 || W == 16 ? 4 : 6; }
constexpr int rows_ahead(int W) { return row_slots(W) / 2 - 1; }   // pairs
constexpr size_t decode_rows_lds(int W, int lanes)
{
    const size_t rows = (size_t)row_slots(W) * row_bytes(W) + (lanes / 64) * 8 + 4;
    return std::max(rows, (size_t)4 * kPointWords * lanes);
}

// The wave that brings the rows.  It has W + 1 loads on their way for a row (lanes past the window load its end once more) and
// waits for them by that number, in order; the compiler does not see that they write LDS.
template <int D, int W, int LANES>
__device__ inline void bring_rows(const decode_wide_params &p, uint32_t slots, int *stat, int lane)
{
    constexpr int kSlots = row_slots(W), kAhead = rows_ahead(W);
    int lo = 0;
    uint32_t from[W], key_from = 0;                                // the lane's places of every load
    auto set_window = [&](int most2, int least2) {
        // (read behind one of the next barriers; the first place a multiple of four, as the keys come in fours)
        lo = __builtin_amdgcn_readfirstlane(max(max(least2 - kRowMargin, most2 + 2 - kRowWindow), 0) + 3 & ~3);
        stat[2 * (LANES / 64)] = lo;
        const int count = __builtin_amdgcn_readfirstlane(most2 + 2) - lo;
#pragma unroll
        for (int x = 0; x < W; x++) from[x] = (uint32_t)min(1024 * x + 16 * lane, count * 4 * W - 16);
        key_from = (uint32_t)min(16 * lane, (count + 3 & ~3) * 4 - 16);
    };
    int c = 0;
    uint32_t slot = slots;
    // row of coordinate c (past the last: row 0, not used) into the next slot
    auto request = [&]() {
        lo = __builtin_amdgcn_readfirstlane(lo); slot = __builtin_amdgcn_readfirstlane(slot); c = __builtin_amdgcn_readfirstlane(c);
        const uint32_t row = (uint32_t)max(D - 1 - c, 0);
        const unsigned char *t = reinterpret_cast<const unsigned char *>(p.tab_t) + (row * (uint32_t)p.row_len + (uint32_t)lo) * (4u * W);
        const unsigned char *key = reinterpret_cast<const unsigned char *>(p.tab_key) + (row * (uint32_t)p.key_len + (uint32_t)lo) * 4u;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     : : "s"(slot + kRowKeys), "v"(key_from), "s"(key) : "memory", "m0");
#pragma unroll
        for (int x = 0; x < W; x++) {
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         : : "s"(slot + kRowThresholds + 1024u * x), "v"(from[x]), "s"(t) : "memory", "m0");
        }
        c++;
        slot = slot == slots + (kSlots - 1) * row_bytes(W) ? slots : slot + row_bytes(W);
    };
    set_window(2 * p.K, 2 * p.K);
#pragma unroll 1
    for (int x = 0; x < 2 * kAhead; x++) request();
#pragma unroll 1
    for (int pair = 0; pair < D / 2; pair++) {
        // the pair's rows are in LDS once only the later ones' loads are on their way; behind the barrier the pair before has been used
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((kAhead - 1) * 2 * (W + 1)) : "memory");
        if ((pair & 3) == 0 && pair > 0) {
            int most2 = 0, least2 = 2 * p.K;
#pragma unroll
            for (int w = 0; w < LANES / 64; w++) { most2 = max(most2, stat[2 * w]); least2 = min(least2, stat[2 * w + 1]); }
            set_window(most2, min(least2, most2));
        }
        request();
        request();
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");             // (LDS is used otherwise behind this)
}

template <int CP, int W, int LANES>
struct rows_walk : lane_q<W> {
    using lane_q<W>::q;
    static constexpr int D = 64 * CP;
    const decode_wide_params &p;
    const uint32_t slots;             // LDS address of the rows
    int *const stat;                  // LDS: every wave's largest and smallest 2 k, the window's first place
    const int tid, wave;
    const bool walks;                 // the wave has a group to walk for
    int k2, n2, i;                    // 2 k, 4 sum m^2
    uint32_t sign, mag;               // the last coordinates' places' lowest bits, the latest on top; their magnitudes, a byte each
    uint32_t slot;                    // the coordinate's row
    int first;                        // the first place of its window

    template <typename T>
    __device__ __forceinline__ static T from_lds(uint32_t at) { return *reinterpret_cast<const __attribute__((address_space(3))) T *>(at); }

    // coordinate i + S, i a multiple of four; every q of the wave lies below 2^(32 WP)
    template <int WP, int S>
    __device__ inline void step()
    {
        slot = __builtin_amdgcn_readfirstlane(slot);               // (the same for the workgroup)
        bool unknown;
        const uint32_t kq = this->template key_of_q<WP>(unknown);
        // places below 2 k whose threshold is above q: three keys, then the four of the block of places they point to
        const int top = max(k2 - first, -1);
        uint32_t keys = slot + (kRowKeys - 4 * 11);
        asm volatile("" : "+s"(keys));                             // (one address for the reads' small offsets)
        const uint32_t at = keys + 4u * (uint32_t)top;
        // (differences of keys, which lie below 2^31, by their signs (the integers have at most 438 bits): a comparison's result may be used
        // two instructions later only
        auto above = [&](uint32_t place) { return (int)(kq - from_lds<uint32_t>(place)) >> 31; };
        int down = 4 * (above(at + 32) + above(at + 16) + above(at));
        const uint32_t block = keys + 4u * (uint32_t)(top + down);
        down += (above(block + 44) + above(block + 40)) + (above(block + 36) + above(block + 32));
        const int in_window = top + down;
        uint32_t j = (uint32_t)(first + in_window);
        const uint32_t entry = slot + (uint32_t)__mul24(in_window, 4 * W);
        uint32_t t[(WP + 3) / 4 * 4];
#pragma unroll
        for (int x = 0; x < (WP + 3) / 4; x++) {
            const u32x4 v = from_lds<u32x4>(entry + (kRowThresholds + 16 * x));
            t[4 * x] = v[0]; t[4 * x + 1] = v[1]; t[4 * x + 2] = v[2]; t[4 * x + 3] = v[3];
        }
        // q - t in three parts side by side, and what a part owes the next
        constexpr int kParts = WP >= 6 ? 3 : 1, kPart = (WP + kParts - 1) / kParts;
        uint32_t owes[kParts] = {};
#pragma unroll
        for (int y = 0; y < kPart; y++)
#pragma unroll
            for (int part = 0; part < kParts; part++)
                if (const int x = part * kPart + y; x < WP) q[x] = __builtin_subc(q[x], t[x], owes[part], &owes[part]);
        uint32_t br = owes[kParts - 1];
#pragma unroll
        for (int part = 1; part < kParts; part++) {
            uint32_t far;                                          // owed further than a word
            q[part * kPart] = __builtin_subc(q[part * kPart], 0u, owes[part - 1], &far);
            br |= far;
        }
        // below the window, or further down than the keys that were looked at; another key; equal keys: by the tables in device memory
        if (min(in_window, down + 15) < 0 || unknown || br) {
#pragma unroll
            for (int part = 0; part < kParts; part++) {
                q[part * kPart] += part > 0 ? owes[part > 0 ? part - 1 : 0] : 0u;
                uint32_t c = 0;
#pragma unroll
                for (int x = part * kPart; x < WP && x < (part + 1) * kPart; x++) q[x] = __builtin_addc(q[x], t[x], c, &c);
            }
            const uint32_t row = (uint32_t)(D - 1 - S - i);
            j = lane_q<W>::place_by_guess(p, row, this->template key_of_q<WP>(), k2 >> 1);
            lane_q<W>::template read_threshold<WP>(p, row, j, t);
            this->template subtract<WP>(p, row, j, t);
        }
        const int left2 = (int)(j & ~1u), d = k2 - left2;
        k2 = left2;
        n2 = (int)__umul24((uint32_t)d, (uint32_t)d) + n2;
        mag = S == 0 ? (uint32_t)d >> 1 : (uint32_t)d << (8 * S - 1) | mag;
        sign = __builtin_amdgcn_alignbit(j, sign, 1);
        slot = slot == slots + (row_slots(W) - 1) * row_bytes(W) ? slots : slot + row_bytes(W);
    }
    template <int WP, int S>
    __device__ __forceinline__ void two_steps()
    {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
        // the rows from this pair on have another window than those before
        constexpr int kAhead = rows_ahead(W);
        if ((S == 0 && i == 0) || (S == (kAhead == 1 ? 2 : 0) && (i & 4) == (kAhead == 1 ? 0 : 4)))
            first = __builtin_amdgcn_readfirstlane(stat[2 * (LANES / 64)]);
        if (walks) { step<WP, S>(); step<WP, S + 1>(); }
    }

    // mags, signs: the point
    template <int WP>
    __device__ __forceinline__ void four_steps(uint32_t (&mags)[D / 4], uint32_t (&signs)[D / 32])
    {
        two_steps<WP, 0>(); two_steps<WP, 2>();
        const int at = __builtin_amdgcn_readfirstlane(i) >> 2;
        mags[at] = mag;
#pragma unroll
        for (int x = 0; x < D / 32; x++) signs[x] = at == 8 * x + 7 ? ~sign : signs[x];
        if (i & 4) {
            uint32_t most2 = walks ? (uint32_t)k2 : 0u, least2 = walks ? (uint32_t)k2 : ~0u;
#define PVQ_STEP(CTRL, ROWS) most2 = max(most2, dpp_move<CTRL, ROWS>(most2, 0u)); least2 = min(least2, dpp_move<CTRL, ROWS>(least2, ~0u));
            PVQ_WAVE_STEPS(PVQ_STEP)
#undef PVQ_STEP
            if ((tid & 63) == 63) { stat[2 * wave] = (int)most2; stat[2 * wave + 1] = (int)min(least2, 0x7FFFFFFFu); }
        }
        i += 4;
    }

    // q shrinks as it goes: the walk runs in as many words as the wave's largest q needs, or one more
    template <int WP>
    __device__ __forceinline__ void walk(uint32_t (&mags)[D / 4], uint32_t (&signs)[D / 32])
    {
        while (i < D && (WP <= 2 || __builtin_amdgcn_ballot_w64((q[WP - 1] | q[WP - 2]) != 0))) four_steps<WP>(mags, signs);
        if constexpr (WP > 2) walk<WP - 2>(mags, signs);
    }
};

template <int CP, int W, int LANES>
__global__ __launch_bounds__(LANES + 64, LANES >= 448 ? (W <= 8 ? 7 : 5) : 1) void decode_wide_rows_kernel(decode_wide_params p)
{
    extern __shared__ __align__(16) uint32_t lds_words[];
    constexpr int D = 64 * CP;
    int *stat = reinterpret_cast<int *>(lds_words + row_slots(W) * row_bytes(W) / 4);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t slots = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds_words;
    if (wave == LANES / 64) {
        bring_rows<D, W, LANES>(p, slots, stat, lane);
        __syncthreads();
        return;
    }
    const int64_t g0 = p.first_group + (int64_t)blockIdx.x * LANES;
    // the lane's group (lanes behind the last group take that one, and write nothing)
    const int64_t gid = std::min<int64_t>(g0 + tid, p.total_groups - 1);
    const int64_t row = gid / p.groups, g = gid - row * p.groups;

    // q = N(D,K) - 1 - index; an index that is no codeword decodes to zeros
    uint32_t q[W], br = 0, any = 0;
#pragma unroll
    for (int i = 0; i < W; i++) {
        const uint32_t w = index_word(p.index + row * p.index_row_words, p, g, i);
        any |= w;
        q[i] = __builtin_subc(p.last_index[i], w, br, &br);
    }
    const bool valid = !br, one_hot = any == 0;
    // Groups that are no codeword, and those with index 0, (0, ..., 0, K), zeros among them, whose k does not fall until the end,
    // would widen the workgroup's windows: they walk another group of the wave once more, and get their points afterwards.
    const uint64_t walkers = __ballot(valid && !one_hot);
    const int source = valid && !one_hot ? lane : walkers ? __builtin_ctzll(walkers) : 0;
#pragma unroll
    for (int i = 0; i < W; i++) q[i] = walkers ? (uint32_t)__shfl((int)q[i], source, 64) : 0u;

    if (tid < row_slots(W) * kRowPad) lds_words[tid / kRowPad * (row_bytes(W) / 4) + tid % kRowPad] = 0;
    rows_walk<CP, W, LANES> walk{{}, p, slots, stat, tid, wave, walkers != 0};
#pragma unroll
    for (int i = 0; i < W; i++) walk.q[i] = q[i];
    walk.k2 = 2 * p.K; walk.n2 = 0; walk.i = 0; walk.sign = walk.mag = 0; walk.slot = slots; walk.first = 0;
    uint32_t mags[D / 4], signs[D / 32] = {};   // (mags: D = 64 in registers, indexed by what is the same for all lanes, D = 128 in scratch)
    walk.template walk<W>(mags, signs);

    int n2 = walk.n2 >> 2;
    if (valid && one_hot) {
#pragma unroll
        for (int x = 0; x < D / 4; x++) mags[x] = x == D / 4 - 1 ? (uint32_t)p.K << 24 : 0u;
#pragma unroll
        for (int x = 0; x < D / 32; x++) signs[x] = 0;
        n2 = p.K * p.K;
    }
    const float gain = valid ? p.scale[gid] / sqrtf((float)n2) : 0.0f;

    // The wave's groups out, 64 values of each at a time: through LDS (where the rows were, once all waves are done with
    // them), from which 8 lanes take a group's 64 values.
    __syncthreads();
    uint32_t *points = lds_words + wave * 64 * kPointWords;
    const int64_t at = row * p.ldw + g * D;
    const int part = lane % 8;
#pragma unroll 1
    for (int half = 0; half < D / 64; half++) {
#pragma unroll
        for (int x = 0; x < 16; x++) points[lane * kPointWords + x] = D == 128 && half ? mags[D / 4 - 16 + x] : mags[x];
#pragma unroll
        for (int x = 0; x < 2; x++) points[lane * kPointWords + 16 + x] = D == 128 && half ? signs[D / 32 - 2 + x] : signs[x];
#pragma unroll 2
        for (int s0 = 0; s0 < 64; s0 += 8) {
            const int s = s0 + lane / 8;
            const float gs = __shfl(gain, s, 64);
            const int64_t to = ((int64_t)__shfl((int)(at >> 32), s, 64) << 32 | (uint32_t)__shfl((int)at, s, 64)) + half * 64 + 8 * part;
            const uint32_t *point = points + s * kPointWords;
            const uint32_t m[2] = {point[2 * part], point[2 * part + 1]}, negative = point[16 + part / 4] >> (8 * (part & 3));
            float v[8];
#pragma unroll
            for (int x = 0; x < 8; x++) {
                const int mag = (int)(m[x / 4] >> (8 * (x & 3)) & 0xFFu);
                v[x] = gs * (float)((negative >> x & 1u) ? -mag : mag);
            }
            if (g0 + wave * 64 + s >= p.total_groups) continue;
            if (p.out_dtype == PVQ_F32) {
                float *o = reinterpret_cast<float *>(p.W_out) + to;
                *reinterpret_cast<float4 *>(o) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4 *>(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
            } else {
                uint32_t u[4];
#pragma unroll
                for (int x = 0; x < 4; x++) {
                    if (p.out_dtype == PVQ_F16) {
                        u[x] = __builtin_bit_cast(uint32_t, __halves2half2(__float2half_rn(v[2 * x]), __float2half_rn(v[2 * x + 1])));
                    } else {
                        const f32x2_t pair = {v[2 * x], v[2 * x + 1]};
                        u[x] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2_t));
                    }
                }
                *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(p.W_out) + to) = make_uint4(u[0], u[1], u[2], u[3]);
            }
        }
    }
}

// ---- many pulses: a lane per group, the tables in device memory ----------------------------------------------
// (rows of thresholds take up to 128 KB)
// Bytes of LDS per lane for the decoded point, rounded up to an odd number of words, so that the lanes' rows spread over the
// banks.  BYTES (K <= 255): a byte per magnitude and a bit per sign; else int16 values, with which 18 waves and not 32 fit a
// unit (393216 groups of 64, K = 180: 93 us with bytes, 136).
template <bool BYTES>
__host__ __device__ constexpr int decode_point_bytes(int D) { return 4 * ((BYTES ? D / 4 + D / 32 : D / 2) | 1); }

// The walk of one lane.  A coordinate takes three dependent trips to the tables, of which the L1 and L2 hold the few lines
// of a row that are in use: the guess of q's bucket, the four keys behind it, and the threshold found.  Equal keys
// (about one comparison in a million, and the all-zero groups) show as a borrow of the subtraction, after which the
// threshold before is taken.  Bound by its chain of about 140 instructions a coordinate and three trips.
template <int CP, int W, bool BYTES>
struct lane_walk : lane_q<W> {
    using lane_q<W>::q;
    static constexpr int D = 64 * CP;
    const decode_wide_params &p;
    unsigned char *mine;
    int k, n2, i;
    uint32_t sign_byte;

    // one coordinate; every q of the wave lies below 2^(32 WP)
    template <int WP>
    __device__ inline void step()
    {
        const uint32_t row = (uint32_t)(D - 1 - i);
        uint32_t j = lane_q<W>::place_by_guess(p, row, this->template key_of_q<WP>(), k);
        uint32_t t[(WP + 3) / 4 * 4];
        lane_q<W>::template read_threshold<WP>(p, row, j, t);
        this->template subtract<WP>(p, row, j, t);
        const int C = (int)(j >> 1), m = k - C;
        k = C;
        n2 += __mul24(m, m);
        if constexpr (BYTES) {
            mine[i] = (unsigned char)m;
            sign_byte = ((i & 7) ? sign_byte : 0u) | ((~j & 1u) << (i & 7));
            if ((i & 7) == 7) mine[D + (i >> 3)] = (unsigned char)sign_byte;
        } else {
            reinterpret_cast<int16_t *>(mine)[i] = (int16_t)(j & 1u ? m : -m);
        }
        i++;
    }

    // q shrinks as it goes: the walk runs in as many words as the wave's largest q needs
    template <int WP>
    __device__ inline void walk()
    {
        while (i < D && (WP == 1 || __any(q[WP - 1] != 0))) step<WP>();
        if constexpr (WP > 1) walk<WP - 1>();
    }
};

// A wave is a workgroup, with decode_point_bytes of LDS per lane.
template <int CP, int W, bool BYTES>
__global__ __launch_bounds__(64) void decode_wide_kernel(decode_wide_params p)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int D = 64 * CP, LB = decode_point_bytes<BYTES>(D);
    const int lane = threadIdx.x;
    const int64_t g0 = (int64_t)blockIdx.x * 64;
    const int count = (int)std::min<int64_t>(64, p.total_groups - g0);
    int64_t out_row = g0 / p.groups, out_g = g0 - out_row * p.groups;

    // the lane's group (lanes behind the last group take that one, unused)
    const uint32_t ahead = (uint32_t)out_g + (uint32_t)std::min(lane, count - 1);
    const int64_t mine = g0 + std::min(lane, count - 1);
    const int64_t row = out_row + ahead / (uint32_t)p.groups, g = ahead % (uint32_t)p.groups;
    lane_walk<CP, W, BYTES> walk{{}, p, lds_raw + (size_t)lane * LB, p.K, 0, 0, 0u};
    // q = N(D,K) - 1 - index; an index that is no codeword decodes to zeros
    uint32_t br = 0;
#pragma unroll
    for (int i = 0; i < W; i++) walk.q[i] = __builtin_subc(p.last_index[i], index_word(p.index + row * p.index_row_words, p, g, i), br, &br);
    const bool valid = !br;
    if (!valid) {
#pragma unroll
        for (int i = 0; i < W; i++) walk.q[i] = 0;
    }
    walk.template walk<W>();
    const float gain = valid ? p.scale[mine] / sqrtf((float)walk.n2) : 0.0f;

    // the groups out, one after the other: consecutive lanes, consecutive values
    int64_t at = out_row * p.ldw + out_g * D + CP * lane;
    const unsigned char *pt = lds_raw;
    for (int s = 0; s < count; s++) {
        const float gs = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(gain), s));
        float v[CP];
#pragma unroll
        for (int j = 0; j < CP; j++) {
            const int at_j = CP * lane + j;
            if constexpr (BYTES) v[j] = gs * (float)((pt[D + (at_j >> 3)] >> (at_j & 7) & 1) ? -(int)pt[at_j] : (int)pt[at_j]);
            else v[j] = gs * (float)reinterpret_cast<const int16_t *>(pt)[at_j];
        }
        store_values<CP>(p, at, v);
        pt += LB;
        at += D;
        if (++out_g == p.groups) { out_g = 0; at += p.ldw - p.groups * D; }
    }
}

// ---- few groups: a wave per group --------------------------------------------------------------------

// The walk of one wave.  q lies across the lanes, a word each; float64 approximations of 64 neighbouring thresholds of
// the row (32 possible values of the pulses left) lie across them too, the highest in lane 0, and the thresholds
// themselves in LDS.  A coordinate is one comparison of approximations, the first lane that passes it, one read of that
// threshold by words, and a subtraction whose borrows run through a scalar addition.  Rows are fetched four coordinates
// in advance, straight into LDS, at the place that k has then: k only falls, by one or two a coordinate, so the window
// nearly always still holds the coordinate.
// A walk is one chain of dependent instructions (8 clocks each, 52 for a read of LDS), so the chain of one coordinate on
// the next is all that counts: about twenty instructions and one read of LDS, hence the few instructions written out;
// everything else about a coordinate is done while the next one's read is on its way.  D = 128, K = 187, one row of 8192
// values / 16 of them: 23 / 30 us, where a lane per group takes 95 (and took 208 when each magnitude was one trip).
constexpr int kWavesFew = 2;          // of a workgroup

template <int CP, int W>
struct wave_walk {
    static constexpr int D = 64 * CP, kAhead = 4;
    static constexpr int kLoads = W / 4 + 1;                       // of a window, 1 KiB each: its thresholds, its approximations
    static constexpr int kWindow = 1024 * kLoads;
    const decode_wide_params &p;
    const int lane;
    const uint32_t ring;              // LDS address of kAhead windows
    uint32_t q;                       // lane x: word x
    int k, n2, i;
    int y[CP];                        // the lane's coordinates: CP * lane + j
    int j, base[kAhead];              // place of the coordinate before in its row; first threshold of a window
    // LDS addresses: the lane's approximation in window 0; its word of the threshold that lane l of a window stands for
    // is from - 4 W l (lanes without a word read a zero)
    uint32_t near_from, from[kAhead];
    int entry;

    // Thresholds b .. b + 63 of a row (a row has 64 at least) and their approximations, 16 bytes a lane and load.  The
    // loads have no result in registers, and the compiler does not see that they write LDS: step waits for them by their
    // number, where the compiler, which knows no windows, would wait for the ones just issued as well.  What is read from
    // a window afterwards are ordinary loads, so that every register has the compiler's own wait before its first use.
    template <int u>
    __device__ __forceinline__ void fetch(int row, int b)
    {
        base[u] = b;
        const uint32_t at = (uint32_t)(row * p.row_len + b);
        const uint32_t t = at * (uint32_t)(4 * W) + 16u * (uint32_t)lane, n = at * 8u + 16u * (uint32_t)lane;
        const uint32_t to = ring + u * kWindow;
        // (the instruction's offset counts on both sides)
#define PVQ_TO_LDS "s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
        if constexpr (W == 4)
            asm volatile(PVQ_TO_LDS : : "s"(to), "v"(t), "s"(p.tab_t) : "memory", "m0");
        else if constexpr (W == 8)
            asm volatile(PVQ_TO_LDS "\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024" : : "s"(to), "v"(t), "s"(p.tab_t) : "memory", "m0");
        else if constexpr (W == 12)
            asm volatile(PVQ_TO_LDS "\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024\n\tglobal_load_lds_dwordx4 %1, %2 offset:2048"
                         : : "s"(to), "v"(t), "s"(p.tab_t) : "memory", "m0");
        else
            asm volatile(PVQ_TO_LDS "\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024\n\tglobal_load_lds_dwordx4 %1, %2 offset:2048"
                         "\n\tglobal_load_lds_dwordx4 %1, %2 offset:3072" : : "s"(to), "v"(t), "s"(p.tab_t) : "memory", "m0");
        asm volatile(PVQ_TO_LDS : : "s"(to + 1024 * (W / 4)), "v"(n), "s"(p.tab_near) : "memory", "m0");
#undef PVQ_TO_LDS
    }

    template <typename T>
    __device__ __forceinline__ static T from_lds(uint32_t at) { return *reinterpret_cast<const __attribute__((address_space(3))) T *>(at); }

    // The coordinate's place in its row, all words compared, window by window from the one for the present k down (ends:
    // T_0 = 0): for windows that lie too high.
    __device__ __forceinline__ static int search(const uint32_t *trow, uint32_t q, int lane, int k)
    {
        for (int b = max(2 * k + 1 - 63, 0);; b = max(b - 64, 0)) {
            bool less = false, equal = true;                       // threshold against q, from the highest word down
#pragma unroll 1
            for (int x = W - 1; x >= 0; x--) {
                const uint32_t qx = (uint32_t)__builtin_amdgcn_readlane((int)q, x), tx = trow[(uint32_t)((b + lane) * W + x)];
                less = less || (equal && tx < qx);
                equal = equal && tx == qx;
            }
            const uint64_t found = __ballot(less || equal);
            if (found) return b + 63 - __builtin_clzll(found);
            if (b == 0) return 0;                                  // (cannot be: T_0 = 0)
        }
    }

    // q -= t over the lanes.  A word borrows from the next where it is smaller (generate), or equal and borrowed from
    // (propagate): the borrows are what the carries of propagate + 2 generate change.  Returns them.
    __device__ __forceinline__ static uint32_t subtract(uint32_t &q, uint32_t t)
    {
        const uint32_t generate = (uint32_t)__builtin_amdgcn_uicmp(q, t, 36), propagate = (uint32_t)__builtin_amdgcn_uicmp(q, t, 32);
        const uint32_t borrows = (propagate + 2u * generate) ^ propagate;
        asm("v_subb_co_u32_e64 %0, vcc, %1, %2, %3" : "=v"(q) : "v"(q), "v"(t), "s"((uint64_t)borrows) : "vcc");
        return borrows;
    }

    // what the coordinate before, at place j of its row, leaves to be done; u is its window, which takes the row four on
    template <int u>
    __device__ __forceinline__ void finish()
    {
        const int C = j >> 1, m = k - C;
        k = C;
        n2 += m * m;
        y[u % CP] = lane == (i - 1) / CP ? ((j & 1) ? m : -m) : y[u % CP];   // (i - 1 = u modulo 4; none for i = 0, whose m is 0)
        fetch<u>(max(D - kAhead - i, 0), max(2 * k - 62, 0));      // (past the last row: row 0, not used)
    }

    template <int u>
    __device__ __forceinline__ void step()
    {
        // this window has arrived once only the loads of the two fetched behind it are on their way (in order)
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"((kAhead - 2) * kLoads) : "memory");
        const double near = from_lds<double>(near_from + u * kWindow);
        __builtin_amdgcn_sched_barrier(0);
        // q's approximation (pvq_wide_double), from its highest word that is not zero and the one below it (lane 63 holds
        // 0; for q = 0 the highest word is "lane 32", which holds 0)
        int lead, first;
        asm("s_flbit_i32_b32 %0, %1" : "=s"(lead) : "s"((uint32_t)__builtin_amdgcn_uicmp(q, 0u, 33)));
        const int at = 31 - lead;
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)q, at), lo = (uint32_t)__builtin_amdgcn_readlane((int)q, at - 1);
        const double nq = __builtin_amdgcn_ldexp(__builtin_fma((double)hi, 4294967296.0, (double)lo), 32 * at - 32);
        uint64_t found = __ballot(near <= nq);
        asm("s_ff1_i32_b64 %0, %1" : "=s"(first) : "s"(found));    // (-1 for none: what is read then is not used)
        uint32_t t = from_lds<uint32_t>(from[u] + (uint32_t)__mul24(first, entry));
        __builtin_amdgcn_sched_barrier(0);
        finish<(u + kAhead - 1) % kAhead>();
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t q0 = q;
        uint32_t borrows = subtract(q, t);
        if (__builtin_expect(((borrows & (1u << W)) | ((uint32_t)first & 0x80000000u)) != 0, 0)) {
            // a threshold above q of the same approximation: the one behind it in the window
            while (found != 0 && (borrows >> W & 1u)) {
                found &= found - 1;
                first = found ? __builtin_ctzll(found) : 0;
                t = from_lds<uint32_t>(from[u] + (uint32_t)__mul24(first, entry));
                q = q0;
                borrows = subtract(q, t);
            }
            if (found == 0) {
                const uint32_t *trow = p.tab_t + (uint32_t)((D - 1 - i) * p.row_len * W);
                q = q0;
                j = __builtin_amdgcn_readfirstlane(search(trow, q, lane, k));
                t = lane < W ? trow[(uint32_t)(j * W + lane)] : 0u;
                subtract(q, t);
                first = base[u] + 63 - j;
            }
        }
        j = base[u] + 63 - first;
        i++;
    }
};

template <int CP, int W>
__global__ __launch_bounds__(64 * kWavesFew) void decode_wide_wave_kernel(decode_wide_params p)
{
    using walk_t = wave_walk<CP, W>;
    constexpr int D = 64 * CP, kRing = walk_t::kAhead * walk_t::kWindow;
    extern __shared__ __align__(16) unsigned char lds_raw[];       // the waves' windows, and a zero
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t gid = (int64_t)blockIdx.x * kWavesFew + wave;
    if (gid >= p.total_groups) return;
    const int64_t row = gid / p.groups, g = gid - row * p.groups;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds_raw;
    walk_t walk{p, lane, lds0 + wave * kRing};
    walk.k = p.K; walk.n2 = 0; walk.i = 0; walk.j = 2 * p.K;       // (before the first coordinate: one of magnitude 0)
#pragma unroll
    for (int j = 0; j < CP; j++) walk.y[j] = 0;
    walk.near_from = lds0 + wave * kRing + 1024 * (W / 4) + 8 * (63 - lane);
    walk.entry = lane < W ? -4 * W : 0;
#pragma unroll
    for (int u = 0; u < walk_t::kAhead; u++)
        walk.from[u] = lds0 + (lane < W ? wave * kRing + u * walk_t::kWindow + 4 * lane + 63 * 4 * W : kWavesFew * kRing);
    asm volatile("ds_write_b32 %0, %1" : : "v"(lds0 + kWavesFew * kRing), "v"(0u) : "memory");
    const int b0 = max(2 * p.K - 62, 0);
    walk.template fetch<0>(D - 1, b0);
    walk.template fetch<1>(D - 2, b0);
    walk.template fetch<2>(D - 3, b0);
    // q = N(D,K) - 1 - index; an index that is no codeword decodes to zeros
    walk.q = 0;
#pragma unroll
    for (int x = 0; x < W; x++) walk.q = lane == x ? p.last_index[x] : walk.q;
    const uint32_t borrows = walk_t::subtract(walk.q, lane < W ? index_word(p.index + row * p.index_row_words, p, g, lane) : 0u);
    const bool valid = !((borrows >> W) & 1u);
    if (valid) {
#pragma unroll 1
        while (walk.i < D) {
            walk.template step<0>();
            walk.template step<1>();
            walk.template step<2>();
            walk.template step<3>();
        }
        walk.template finish<3>();
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");             // (the workgroup's LDS is not given back before the last loads into it)
    const float gain = valid ? p.scale[gid] / sqrtf((float)walk.n2) : 0.0f;
    float v[CP];
#pragma unroll
    for (int j = 0; j < CP; j++) v[j] = gain * (float)walk.y[j];
    store_values<CP>(p, row * p.ldw + g * D + CP * lane, v);
}

int gcd_int(int a, int b) { return b ? gcd_int(b, a % b) : a; }

}  // namespace

hipError_t pvq_wide_launch_encode(const pvq_ctx *c, const pvq_encode_args &a, int dtype, hipStream_t s)
{
    encode_wide_params p;
    p.X = a.W; p.ldx = a.ldw; p.groups = a.groups; p.index_row_words = a.index_row_words;
    p.K = c->K; p.bits = c->index_bits; p.ls = a.ls_amplitude;
    p.tab_t = c->tab_u; p.row_len = pvq_wide_row(c->K);
    for (int i = 0; i < 16; i++) p.last_index[i] = c->last_index[i];
    p.index_out = a.index_out; p.scale_out = reinterpret_cast<float *>(a.scale_out); p.pulses_out = a.pulses_out;
    p.cols = a.cols;
    // tiles of whole words and whole waves, four groups each
    p.tile_groups = std::max(4, 32 / gcd_int(c->index_bits, 32));
    p.tiles_per_row = (int)((a.groups + p.tile_groups - 1) / p.tile_groups);
    if (a.rows * p.tiles_per_row > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int waves = std::min(p.tile_groups / 4, 8);
    const size_t lds = (size_t)(p.tile_groups * c->index_bits / 32) * 4;
    const dim3 grid((unsigned)(a.rows * p.tiles_per_row)), blk(64u * waves);
#define PVQ_WIDE_ENC(T, CP, W) hipLaunchKernelGGL((encode_wide16_kernel<T, CP, W>), grid, blk, lds, s, p)
#define PVQ_WIDE_ENC_W(T, D64)                                                                                  \
    switch (c->words) {                                                                                         \
    case 4: if (D64) PVQ_WIDE_ENC(T, 4, 4); else PVQ_WIDE_ENC(T, 8, 4); break;                                  \
    case 8: if (D64) PVQ_WIDE_ENC(T, 4, 8); else PVQ_WIDE_ENC(T, 8, 8); break;                                  \
    case 12: if (D64) PVQ_WIDE_ENC(T, 4, 12); else PVQ_WIDE_ENC(T, 8, 12); break;                               \
    default: if (D64) PVQ_WIDE_ENC(T, 4, 16); else PVQ_WIDE_ENC(T, 8, 16); break;                               \
    }
    const bool d64 = c->D == 64;
    if (dtype == PVQ_F32) { PVQ_WIDE_ENC_W(PVQ_F32, d64) } else { PVQ_WIDE_ENC_W(PVQ_BF16, d64) }
#undef PVQ_WIDE_ENC_W
#undef PVQ_WIDE_ENC
    return hipGetLastError();
}

hipError_t pvq_wide_launch_rotate_encode(const pvq_ctx *c, const pvq_encode_args &a, int dtype, int block,
                                         const uint8_t *signs, hipStream_t s)
{
    rotate_encode_params p;
    int log2n = 0;
    while ((1 << log2n) < block) log2n++;
    const int L = std::min(1024, std::max(256, block / 8));
    const int chunk = 8 * L;
    p.X = a.W; p.ldx = a.ldw; p.cols = a.cols; p.log2n = log2n; p.signs = signs;
    p.chunks_per_row = (int)((a.cols + chunk - 1) / chunk);
    p.scale = (float)(1.0 / std::sqrt((double)block));
    p.e.X = nullptr; p.e.ldx = 0; p.e.groups = a.groups; p.e.index_row_words = a.index_row_words;
    p.e.K = c->K; p.e.bits = c->index_bits; p.e.ls = a.ls_amplitude;
    p.e.tile_groups = L / 16; p.e.tiles_per_row = p.chunks_per_row;
    p.e.tab_t = c->tab_u; p.e.row_len = pvq_wide_row(c->K);
    for (int i = 0; i < 16; i++) p.e.last_index[i] = c->last_index[i];
    p.e.index_out = a.index_out; p.e.scale_out = reinterpret_cast<float *>(a.scale_out);
    p.e.pulses_out = nullptr; p.e.cols = a.cols;
    if (a.rows * p.chunks_per_row > 0x7FFFFFFF) return hipErrorInvalidValue;
    size_t lds = (size_t)(L / 16) * c->index_bits / 8 + 16;
    if (log2n > 9) lds += (size_t)(chunk + chunk / 32 + 1) * sizeof(float);
    const dim3 grid((unsigned)(a.rows * p.chunks_per_row)), blk((unsigned)L);
#define PVQ_RE(T, W, N) hipLaunchKernelGGL((rotate_encode16_kernel<T, W, N>), grid, blk, lds, s, p)
#define PVQ_RE_N(T, W)                             \
    switch (log2n) {                               \
    case 13: PVQ_RE(T, W, 13); break;              \
    case 12: PVQ_RE(T, W, 12); break;              \
    case 11: PVQ_RE(T, W, 11); break;              \
    case 10: PVQ_RE(T, W, 10); break;              \
    default: PVQ_RE(T, W, 9); break;               \
    }
#define PVQ_RE_W(T)                                \
    switch (c->words) {                            \
    case 4: PVQ_RE_N(T, 4) break;                  \
    case 8: PVQ_RE_N(T, 8) break;                  \
    default: PVQ_RE_N(T, 12) break;                \
    }
    if (dtype == PVQ_F32) { PVQ_RE_W(PVQ_F32) } else { PVQ_RE_W(PVQ_BF16) }
#undef PVQ_RE_W
#undef PVQ_RE_N
#undef PVQ_RE
    return hipGetLastError();
}

// Up to this many groups a wave per group decodes.  Its time grows with the groups once the SIMDs' issue slots are full, in
// steps, by the width of the integers (and for many pulses by the windows a coordinate is looked for in); a lane per group
// takes the one walk of a wave whatever their number, until there are several waves per SIMD.  us, a wave per group, and lanes
// (the last column):
//                        2048   2176   2560   2816   3072   3200   3584   3840   4096   4352   4608    lanes
//   D = 128, K = 28      29     36     36     44     44     44     44     44     44     51     51      45      (integers of 4 words)
//            K = 84      30     37     37     46     46     56     58                                  50      (8)
//            K = 120     33     51     56     63     66     67     73                                  50      (12)
//            K = 187     33     51     56     63     66     67     73                                  52      (12)
//            K = 255     56     60     67     68     71     82     85                                  67      (16)
//   D = 64,  K = 40      16     19     19     23     23     23     23     23     23     27     27      23      (4)
//            K = 96      16     20     20     25     25     30     31                                  26      (8)
//            K = 127     16     20     20     25     25     30     31     35     37     39     40      31      (8)
//            K = 143     16     20     20     25     25     30     31     35     37     39     40      39      (8)
//            K = 150     16     20     20     25     25     30     31     35     37     39     40      42      (8; 4800 groups 42 / 42)
//            K = 160     5120 groups: 43 / 46                                                                  (8; lanes: device memory)
//            K = 220     2048 24, 3520 40, 4096 43, 4608 50 / lanes 47 to 48                                   (12; the same)
//            K = 255     2048 30, 3520 45, 4096 50, 4608 57 / 48                                               (12; the same)
static int64_t few_groups(const pvq_ctx *c)
{
    if (c->words == 4) return 4096;
    if (c->D == 128) return c->words == 8 ? 3072 : c->K > 255 ? 3584 : c->words == 12 ? 2048 : 2560;
    if (c->words == 8) return c->K <= 112 ? 3072 : c->K <= 135 ? 3584 : c->K <= 143 ? 4352 : c->K <= 150 ? 4800 : 5120;
    return c->K <= 230 ? 4608 : 3584;
}

// Beyond that, whether the rows of the tables go through LDS.  They do while a magnitude fits a byte; but with more than about
// twice as many pulses as coordinates many places lie outside a window of 256, and then all of them are as well read from device
// memory: with many pulses always, with fewer once a unit has more groups than its two workgroups of 512 take at once (where device memory
// has its next step in turn).  us, LDS / device memory:
//                    8192 groups   65536      131072     163840     196608     262144     294912     393216     524288     1048576
//   D = 64, K = 96     27 / 45    31 / 48    36 / 50    46 / 52    46 / 53    48 / 80    70 / 82    71 / 88    89 / 102  162 / 190
//           K = 112    28 / 46    34 / 49    40 / 51    50 / 53    52 / 54    52 / 80    78 / 83    81 / 89    95 / 104  173 / 194
//           K = 120    30 / 46    37 / 49    43 / 51    54 / 53    55 / 54    56 / 80    85 / 83    88 / 90   102 / 105  184 / 195
//           K = 127    33 / 46    40 / 48    46 / 51    57 / 53    59 / 54    60 / 80    91 / 82    93 / 90   108 / 106  195 / 197
//           K = 135    35 / 46    43 / 48    51 / 51    61 / 53    63 / 54    64 / 81   100 / 83   103 / 91   117 / 107  213 / 198
//           K = 150    41 / 46    50 / 49    57 / 51    69 / 53    70 / 55    71 / 81   113 / 84   115 / 91   132 / 107  244 / 203
//           K = 160    49 / 46                63 / 52                          78 / 81              126 / 91   147 / 108  282 / 200   (LDS: every wave
//           K = 200    58 / 47                75 / 57                          96 / 91              157 / 105  182 / 122  351 / 226    requesting rows)
//   D = 128, K = 187 8192 groups 53 / 95, 262144 91 / 164, 524288 209 / 325; K = 255 70 / 97, 132 / 279, 267 / 528.
static bool rows_in_lds(const pvq_ctx *c, int64_t groups)
{
    if (c->D == 128) return c->K <= 255;
    return c->K <= 120 || (c->K <= 150 && groups <= 256 * 1024);
}

// Lanes of a workgroup whose rows of the tables go through LDS: the fewest, from 128 on, with which the groups take one place
// on each of the 256 units, up to 512.  (64 lanes, a wave that loads its rows alone: 8192 groups of 128 in 80 us, with 128
// lanes 70; 256 at most: 262144 groups in 151 us, with 512 lanes, two workgroups to a unit, 109.)
// With integers of up to 8 words three workgroups of 512 and the wave that brings their rows fit a unit, 27 waves where it has room for 28 or
// 32; what comes in the place of one that is done does not always find room for nine waves (or leaves five waves' room unused).  Workgroups of 448 lanes have
// eight waves, of which three or four fit any time.  From where workgroups follow one another, us, 512 / 448 lanes:
//                      393216     458752     524288     655360     786432     1048576    1572864 groups
//   D = 64, K = 40     63 / 69    76 / 69    77 / 81    93 / 94   117 / 106  154 / 145  234 / 199
//           K = 96     72 / 75    86 / 76   101 / 89   112 / 104  144 / 119  181 / 162  274 / 224
//           K = 112    80 / 82   104 / 85   119 / 97   125 / 112  164 / 129  208 / 175  303 / 243
//   D = 128, K = 28    99 / 115  129 / 116  131 / 141  159 / 166  185 / 189  260 / 257  374 / 349      (integers of 4 words)
//            K = 84   115 / 131  151 / 132  153 / 163  209 / 190  252 / 221  324 / 299  459 / 411      (8)
static int rows_lanes(const pvq_ctx *c, int64_t groups)
{
    if (c->words == 8 ? groups > (c->D == 64 ? 768 : 1024) * 512 : c->words == 4 && c->D == 64 && groups > 1280 * 512) return 448;
    int lanes = 128;
    while (lanes < 512 && groups > (int64_t)256 * lanes) lanes *= 2;
    return lanes;
}

template <int CP, int W, int LANES>
static hipError_t launch_rows(const decode_wide_params &p, size_t lds, hipStream_t s)
{
    if constexpr (LANES == 448 ? W == 8 || (CP == 1 && W == 4) : CP == 2 || W <= 8) {  // (as wide as the integers of rows_in_lds are)
        if (lds > 64 * 1024) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(decode_wide_rows_kernel<CP, W, LANES>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        // With integers of 16 words a workgroup reads 17 KB a coordinate, from L2 as long as the workgroups of a die are at about the same one.
        // Those that come in the place of others are not, so the 512 that have a place at once are a launch, unless the last would have
        // few (D = 128, K = 255, us, in one / in launches of 512: 458752 groups 310 / 263, 524288 312 / 267, 786432 460 / 403, 1048576 579 / 538,
        // but 393216 222 / 239, 655360 349 / 368, 917504 478 / 511; with 12 words 524288 209 / 184, but 917504 327 / 360, and in one no slower than any
        // form before).
        const int64_t workgroups = (p.total_groups + LANES - 1) / LANES;
        const int64_t of_launch = W == 16 && (workgroups - 1) % 512 >= 256 ? 512 : workgroups;
        for (int64_t at = 0; at < workgroups; at += of_launch) {
            decode_wide_params q = p;
            q.first_group = at * LANES;
            hipLaunchKernelGGL((decode_wide_rows_kernel<CP, W, LANES>), dim3((unsigned)std::min(of_launch, workgroups - at)), dim3(LANES + 64), lds, s, q);
        }
        return hipSuccess;
    } else {
        return hipErrorInvalidValue;
    }
}

// Groups of 64 that the machine's LDS holds at once as int16 values, 18 waves a unit.  Up to there those take less time to keep
// (8192 groups, K = 180: 46 us, as bytes 48); beyond, waves wait for a place (393216: 136, as bytes 93).
constexpr int64_t kGroupsAtOnce16 = 256 * 64 * (int64_t)(160 * 1024 / ((64 * decode_point_bytes<false>(64) + 1279) / 1280 * 1280));

template <int CP, int W>
static hipError_t launch_lanes(const decode_wide_params &p, hipStream_t s)
{
    const dim3 grid((unsigned)((p.total_groups + 63) / 64)), blk(64);
    if constexpr (CP == 1 && (W == 8 || W == 12)) {
        if (p.K <= 255 && p.total_groups > kGroupsAtOnce16) {
            hipLaunchKernelGGL((decode_wide_kernel<CP, W, true>), grid, blk, (size_t)64 * decode_point_bytes<true>(64 * CP), s, p);
            return hipSuccess;
        }
    }
    if constexpr (CP == 2 ? W == 16 : W >= 8) {
        hipLaunchKernelGGL((decode_wide_kernel<CP, W, false>), grid, blk, (size_t)64 * decode_point_bytes<false>(64 * CP), s, p);
        return hipSuccess;
    } else {
        return hipErrorInvalidValue;
    }
}

#define PVQ_WIDE_DEC_W(CP)                                  \
    switch (c->words) {                                     \
    case 4: PVQ_WIDE_DEC(CP, 4); break;                     \
    case 8: PVQ_WIDE_DEC(CP, 8); break;                     \
    case 12: PVQ_WIDE_DEC(CP, 12); break;                   \
    default: PVQ_WIDE_DEC(CP, 16); break;                   \
    }
#define PVQ_WIDE_DEC_DW if (c->D == 128) { PVQ_WIDE_DEC_W(2) } else { PVQ_WIDE_DEC_W(1) }

hipError_t pvq_wide_launch_decode(const pvq_ctx *c, const pvq_decode_args &a, int out_dtype, hipStream_t s)
{
    decode_wide_params p;
    p.index = a.index; p.scale = reinterpret_cast<const float *>(a.scale);
    p.groups = a.groups; p.total_groups = a.rows * a.groups; p.index_row_words = a.index_row_words; p.ldw = a.ldw;
    p.K = c->K; p.bits = c->index_bits; p.out_dtype = out_dtype;
    p.row_len = pvq_wide_row(c->K); p.key_len = pvq_wide_key_row(c->K); p.buckets = pvq_wide_buckets(c->words);
    p.tab_t = c->tab_u; p.tab_key = c->tab_key; p.tab_near = c->tab_near; p.tab_guess = c->tab_guess;
    p.W_out = a.W_out; p.first_group = 0;
    for (int i = 0; i < 16; i++) p.last_index[i] = c->last_index[i];
    if ((p.total_groups + 63) / 64 > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int64_t total = p.total_groups;
    if (total <= few_groups(c)) {
        const size_t lds = (size_t)kWavesFew * 4 * 1024 * (c->words / 4 + 1) + 16;
#define PVQ_WIDE_DEC(CP, W) \
    hipLaunchKernelGGL((decode_wide_wave_kernel<CP, W>), dim3((unsigned)((total + kWavesFew - 1) / kWavesFew)), dim3(64 * kWavesFew), lds, s, p)
        PVQ_WIDE_DEC_DW
#undef PVQ_WIDE_DEC
    } else if (!rows_in_lds(c, total)) {
        hipError_t e = hipSuccess;
#define PVQ_WIDE_DEC(CP, W) e = launch_lanes<CP, W>(p, s)
        PVQ_WIDE_DEC_DW
#undef PVQ_WIDE_DEC
        if (e != hipSuccess) return e;
    } else {
        const int lanes = rows_lanes(c, total);
        const size_t lds = decode_rows_lds(c->words, lanes);
        hipError_t e = hipSuccess;
#define PVQ_WIDE_DEC(CP, W)                                                        \
    switch (lanes) {                                                               \
    case 128: e = launch_rows<CP, W, 128>(p, lds, s); break;                       \
    case 256: e = launch_rows<CP, W, 256>(p, lds, s); break;                       \
    case 448: e = launch_rows<CP, W, 448>(p, lds, s); break;                       \
    default: e = launch_rows<CP, W, 512>(p, lds, s); break;                        \
    }
        PVQ_WIDE_DEC_DW
#undef PVQ_WIDE_DEC
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}
