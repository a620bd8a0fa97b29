// Correcting the quantisation error group after group (Sec. 3.3 Step 6), rows of W in place.
//
// For every row, groups g = 0 .. G-1 in order: the group's current values w_g are quantised as in Steps 3
// and 4 (point y, amplitude s), q = (s / sqrt(sum y^2)) y, e = w_g - q, and the columns behind the group
// take up the error:  t U_gg = e by substitution, then w_c <- w_c - t_0 U[gD][c] - ... - t_{D-1} U[gD+D-1][c],
// with U the upper triangular factor of the inverse Hessian (U^T U = H^-1).  float32; every "- t_i U" is
// one fused multiply-add applied in the order i = 0, 1, ... to the running value, group after group: the
// order is part of the definition, because later roundings are decided from these values.  On return W
// holds, for every group, the values that were quantised: encoding it gives the corrected code.
//
// Rows are independent, groups of a row strictly sequential, and U is the same for every row.  Columns are taken in panels
// of 128, one or two panels a launch on the caller's stream (correct_step_kernel), whose workgroups have one of two roles:
//     panel   (the first workgroups, 32 or 16 rows each) for each of the launch's panels, the multiply-adds of the launch before's
//             panels onto its columns (and of the launch's own first panel onto its second), then its groups one after the
//             other, a row across 8 or 16 lanes.  Leaves the panel's t values (rows x 128) in a work buffer.  One wave a SIMD,
//             which issues an instruction in four to five clocks whether it depends on the one before or not, so its time is
//             the number of its instructions: with one panel a launch 4.1 us in front (first reads 2, matrix instructions 1.7),
//             1.2 for the panel's part of U, 10.5 for 16 groups of 8 (2.4, 0.5 and 10.5 with 16 rows); with two 44 us for both.
//     update  (all others) the launch before's panels onto all columns behind the launch's own: 128 or 256 multiply-adds per
//             element, in the same order, W read and written once a launch.
// Bound: float32 matrix instructions (155 TFLOP/s in registers with any number of waves), and they keep other waves of their SIMD from
// the vector unit while they run (a wave of them beside a wave of vector instructions takes the sum of both times, whatever
// the priorities; beside bfloat16 ones it is the longer of both).  So the chain of panels costs the updates what it issues, and there is
// little to gain from more waves.  What counts is that no wave waits for its own stores, that a launch's updates start and end
// together, and fewer launches and passes over W.
// The two roles touch different columns; the updates read the t values of the launch before's panels while the panel role writes
// its own, so two panels a launch take four work buffers, one panel two.  Two panels a launch halve the passes over W and the launches'
// starts; the chain pays for it with longer fronts, which shows where there are few rows (64 x 2048 268 / 281 us).  The panel
// workgroups come first in the grid and raise their waves' priority.  A workgroup has the LDS of the role that needs more: 64 KB with two
// panels, two workgroups to a unit; with one 36.9 KB in groups of 8, 39.9 in groups of 16, four to a unit; 45.1 in groups of 32, three.
// Both roles' multiply-adds run on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four products to an
// element one by one, k ascending, each a fused multiply-add (measured bit for bit against fmaf over random, cancelling,
// tied, subnormal and non-finite operands).
// 8192 x 8192 in groups of 8 5.07 ms, 28672 x 8192 17.8, 8192 x 4096 1.52, 4096 x 4096 1.05, 1024 x 8192 1.51; one panel a launch, for which the smallest
// work buffer has room, 5.56, 19.7, 1.61, 1.10, 1.57.  Before, with one panel a launch, tasks of 64 columns and 128 to 1024 rows and waves
// that waited for their stores after every 16 rows, 6.10, 21.2, 1.74, 1.10, 1.55 (so with that work buffer 7 to 10 million values in groups of 8 take
// up to 1.5 % longer now); with tiles of 128 x 128 whose workgroups moved in step 6.6 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "pvq_exact_dev.h"
#include "pvq_internal.h"

namespace {

using namespace pvq_exact_dev;

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kPanelCols = 128;   // columns per panel
constexpr int kWaves = 4;         // waves of a workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kTileCols = 64;     // columns of an update's task
constexpr int kItemRows = 16;     // rows that a wave of it takes at a time
constexpr int kStepRows = kItemRows * kWaves;
constexpr int kUpdateFloats = kPanelCols * kTileCols;

// t values of a panel as the matrix instructions' operands: per 16 rows (fewer at the end) pieces of four values, of which a
// lane takes one for four instructions in a row: piece (i, k4) of a row holds columns 16 i + 4 s + k4, s = 0 .. 3, and the rows'
// pieces lie side by side, so that a read of 16 rows is 1 KiB in a row.
struct t_rows {
    int64_t at;      // piece (0, 0) of the row
    int step;        // from a piece to the next one of the row
    __device__ t_rows(int64_t row, int64_t rows)
    {
        const int64_t block = row & ~(int64_t)15;
        step = 4 * (int)std::min<int64_t>(16, rows - block);
        at = block * kPanelCols + 4 * (row - block);
    }
    __device__ const f32x4 *piece(const float *T, int i, int k4) const { return reinterpret_cast<const f32x4 *>(T + at + (4 * i + k4) * step); }
    __device__ float *column(float *T, int k) const { return T + at + (4 * (k >> 4) + (k & 3)) * step + (k >> 2 & 3); }
};

struct correct_shape {
    int64_t ldw, rows, cols, ldu;
    int K, ls;
};

// How the updates are shared out: the rows' steps of kStepRows are in 2^log2_chunks chunks of `steps` each, the first `longer` of them one more;
// a chunk's steps times the blocks of kTileCols columns go to its shares, `each` or, the first `rest` shares, one more (of a chunk that is
// no longer, or is).
struct update_split {
    uint32_t log2_chunks, steps, longer, each[2], rest[2];
};

// The buffers of t values (rows x 128 floats each) that a launch uses: those of the launch before's panels, and its own behind them.
template <int PANELS> struct t_buffers {
    float *of[2 * PANELS];
};

// ---- a row's group across L neighbouring lanes, C = D / L coordinates a lane --------------------------------
template <int D> struct split {
    static constexpr int L = D == 8 ? 8 : 16, C = D / L;
    static constexpr int kRowsOfWave = 64 / L, kMost = kWaves * kRowsOfWave;         // rows of a panel workgroup, at most
    static constexpr int kGroups = kPanelCols / D;
    // LDS of the panel role: D x D blocks of U on and above the panel's diagonal, before that t values and sums on their way
    // to and from the matrix cores' layout (kXPitch: an operand's values lie on different banks)
    static constexpr int kBlocks = kGroups * (kGroups + 1) / 2;
    // The first kNear groups behind a group are updated whether they are there or not (their instructions fill the waits of the
    // substitution's chain), which reads up to kPast blocks behind the last; the divisors lie there, 4 words per column.
    static constexpr int kNear = D == 8 ? 7 : D == 16 ? 3 : 0, kPast = kNear > 0 ? kNear : 1;
    static constexpr int kDivisors = kBlocks * D * D;
    static constexpr int kFloats = kDivisors + (4 * kPanelCols > kPast * D * D ? 4 * kPanelCols : kPast * D * D);
    static constexpr int kXPitch = kPanelCols + 4;
};
template <int D, int PANELS> constexpr int lds_floats() { return std::max(PANELS * kUpdateFloats, split<D>::kFloats); }

template <int CTRL, int BANKS = 0xF>
__device__ inline int dpp(int old, int v) { return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xF, BANKS, false); }
template <int CTRL>
__device__ inline float dpp_add(float v) { return v + __int_as_float(dpp<CTRL>(0, __float_as_int(v))); }

// Sum over the L lanes of a row, adjacent pairs level by level, in every lane.
template <int L>
__device__ inline float lanes_sum(float v)
{
    v = dpp_add<0xB1>(v);                       // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);                       // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);                      // row_half_mirror: the other quad, all of whose lanes hold its sum
    if constexpr (L == 16) v = dpp_add<0x140>(v);   // row_mirror
    return v;
}

// A column's divisor: for diagonals from 2^-20 to 2^20 and quotients from 2^-70 to 2^70; others get y = NaN, which every quotient then is.
__device__ inline divisor column_divisor(float b)
{
    divisor d = divisor_of(b, reciprocal(b));
    if (!magnitude_in(b, 0x1p-20f, 0x1p20f)) d.y = __builtin_nanf("");
    return d;
}

// v of the lane j ^ X of the row
template <int X>
__device__ inline int lane_xor(int v)
{
    if constexpr (X == 0) return v;
    else if constexpr (X == 1) return dpp<0xB1>(0, v);
    else if constexpr (X == 2) return dpp<0x4E>(0, v);
    else if constexpr (X == 3) return dpp<0x1B>(0, v);
    else if constexpr (X < 8) return lane_xor<7 - X>(dpp<0x141>(0, v));
    else if constexpr (X < 12) return lane_xor<X - 8>(dpp<0x128>(0, v));   // row_ror:8
    else return lane_xor<15 - X>(dpp<0x140>(0, v));
}

// v of lane N of the row, in all L lanes
template <int L, int N>
__device__ inline float lane_broadcast(float v)
{
    const int i = __float_as_int(v), low = __builtin_amdgcn_mov_dpp(i, 0x150 + N, 0xF, 0xF, true);   // row_newbcast
    return __int_as_float(L == 16 ? low : dpp<0x150 + (L == 16 ? 0 : 8) + N, 0xC>(low, i));          // (one for either half)
}

// A bit of `behind` per coordinate of lanes j ^ X, X = 1 .. L - 1, set if it does not come before coordinate c of this lane in
// the order of keys (largest first, lower coordinate first on ties): key < th, th being mine, and one more where bit b of j does
// not say that the other lane is the lower one.  Keys are not negative, so the difference has the answer in its sign.  (The
// other lane's key is the minuend: the reversed subtraction v_subrev_u32 with a DPP operand, which the compiler makes of the opposite,
// permutes its other operand here.)
template <int L, int C, int X>
__device__ inline void mark_behind(const int (&key)[C], const int (&th)[C][4], uint32_t (&behind)[C])
{
    if constexpr (X < L) {
        constexpr int b = X < 2 ? 0 : X < 4 ? 1 : X < 8 ? 2 : 3;
#pragma unroll
        for (int o = 0; o < C; o++) {
            const int other = lane_xor<X>(key[o]);
#pragma unroll
            for (int c = 0; c < C; c++) behind[c] = __builtin_amdgcn_alignbit(behind[c], (uint32_t)(other - th[c][b]), 31);
        }
        mark_behind<L, C, X + 1>(key, th, behind);
    }
}

// The quantiser of Sec. 2.5 (as in pvq_quantize_dev.h) with the group's coordinates C j .. C j + C - 1 in lane j of its row: the
// same sums in the same order, the coordinates that hold the first places in the order of deviations found by comparing all
// of them.  ss: the sum of squares, y: the signed point (zeros of either sign).
//   PLAIN: for groups whose ss lies between 2^-90 and 2^90, which have a direction and whose norms are far from either end of the
// type.
template <int D, bool PLAIN>
__device__ inline void quantize_lanes(const float (&w)[split<D>::C], int j, int K, float &ss, float (&y)[split<D>::C])
{
    constexpr int L = split<D>::L, C = split<D>::C;
    float a1 = fabsf(w[0]), s2 = w[0] * w[0];
    if constexpr (C == 2) { a1 = a1 + fabsf(w[1]); s2 = s2 + w[1] * w[1]; }
    const float l1 = lanes_sum<L>(a1), Kf = (float)K;
    ss = lanes_sum<L>(s2);
    float g;
    bool degenerate = false;
    if constexpr (PLAIN) {
        g = small_over(Kf, l1);
    } else {
        g = Kf / l1;
        degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(g < INFINITY);
    }
    float t[C], yf[C];
#pragma unroll
    for (int c = 0; c < C; c++) {
        t[c] = fabsf(w[c]) * g;
        yf[c] = rintf(t[c]);
    }
    // small integers: exact in any order;  > 0: pulses to add, < 0: pulses to take away
    const float m = Kf - lanes_sum<L>(C == 2 ? yf[0] + yf[C - 1] : yf[0]);
    const float unit = m < 0.0f ? -1.0f : 1.0f;
    const int need = (int)fabsf(m);
    // deviations; the `need` largest are positive, and positive floats order like their bits
    int key[C], th[C][4];
#pragma unroll
    for (int c = 0; c < C; c++) {
        key[c] = std::max(__float_as_int((t[c] - yf[c]) * unit), 0);
#pragma unroll
        for (int v = 0; v < 4; v++) th[c][v] = key[c] + (~(j >> v) & 1);
    }
    uint32_t behind[C];
    behind[0] = 0;
    if constexpr (C == 2) { behind[0] = key[0] >= key[C - 1] ? 1u : 0u; behind[C - 1] = 1u - behind[0]; }
    mark_behind<L, C, 1>(key, th, behind);
#pragma unroll
    for (int c = 0; c < C; c++) {
        // unit where fewer than `need` are in front
        const int moved = (D - 1 - need - (int)__builtin_popcount(behind[c])) >> 31 & __float_as_int(unit);
        float mag = yf[c] + __int_as_float(moved);
        // (a weight of -0 has the point's +0, which shows in the sign of its error; PLAIN refuses errors that stay zero)
        if constexpr (PLAIN) {
            y[c] = copysignf(mag, w[c]);
        } else {
            if (degenerate) mag = C * j + c == D - 1 ? Kf : 0.0f;
            y[c] = w[c] < 0.0f && !degenerate ? -mag : mag;
        }
    }
}

// t U_GG = e, coordinate after coordinate: t_I is final once t_0 .. t_{I-1} have been taken off e_I.  e: the lane's
// coordinates; u: rows of the block in the lane's columns, zero on and below the diagonal; d: its diagonal there.  tb gets all of
// t, mine the lane's own.  PLAIN: a lane's e stays what it is behind its own place, since it loses products with zeros, so the
// last quotients are the lane's own t; right if they all lie between 2^-70 and 2^70 (a zero would lose its sign).
// next(I): work with t_0 .. t_I that the waits of the chain have time for.
template <int D, bool PLAIN, int I, typename Next>
__device__ inline void substitute(float (&e)[split<D>::C], const float (&u)[split<D>::C][D], const divisor (&d)[split<D>::C],
                                  int j, float (&tb)[D], float (&mine)[split<D>::C], const Next &next)
{
    constexpr int L = split<D>::L, C = split<D>::C;
    if constexpr (I < D) {
        const float q = PLAIN ? divide(e[I % C], d[I % C]) : e[I % C] / d[I % C].b;
        if constexpr (PLAIN) mine[I % C] = q;
        else mine[I % C] = j == I / C ? q : mine[I % C];
        if constexpr (I > 0) next(I - 1);
        tb[I] = lane_broadcast<L, I / C>(q);
#pragma unroll
        for (int c = 0; c < C; c++) e[c] = __builtin_fmaf(-tb[I], u[c][I], e[c]);
        substitute<D, PLAIN, I + 1>(e, u, d, j, tb, mine, next);
        if constexpr (I + 1 == D) next(I);
    }
}

// A group from its values w: quantiser, amplitude, error, substitution; tb and mine as above.  Returns whether the group is one
// that PLAIN is right for.
template <int D, bool LS, bool PLAIN, typename Next>
__device__ inline bool solve_group(const float (&w)[split<D>::C], const float (&u)[split<D>::C][D], const divisor (&d)[split<D>::C],
                                   int j, int K, float (&tb)[D], float (&mine)[split<D>::C], const Next &next)
{
    constexpr int L = split<D>::L, C = split<D>::C;
    float y[C], ss;
    quantize_lanes<D, PLAIN>(w, j, K, ss, y);
    float sq = 0.0f, dot = 0.0f;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const float s = y[c] * y[c], p = y[c] * w[c];
        sq = c == 0 ? s : sq + s;                               // integers
        dot = c == 0 ? p : dot + p;
    }
    sq = lanes_sum<L>(sq);
    float gain;
    if constexpr (PLAIN) {
        const divisor root = root_divisor(sq);
        gain = divide(LS ? divide(lanes_sum<L>(dot), root) : root_of(ss), root);
    } else {
        const float root = sqrtf(sq);
        gain = (LS ? lanes_sum<L>(dot) / root : sqrtf(ss)) / root;
    }
    float e[C];
#pragma unroll
    for (int c = 0; c < C; c++) { e[c] = w[c] - gain * y[c]; mine[c] = 0.0f; }
    substitute<D, PLAIN, 0>(e, u, d, j, tb, mine, next);
    bool ordinary = magnitude_in(ss, 0x1p-90f, 0x1p90f);
#pragma unroll
    for (int c = 0; c < C; c++) ordinary = ordinary && magnitude_in(mine[c], 0x1p-70f, 0x1p70f);
    return ordinary;
}

// Panel role.  A workgroup takes ROWS rows, a wave 8 (D = 8) or 4 of them: lane (row, j) holds coordinate(s) j of
// every group of the panel, and the waves do not wait for each other once the panel's part of U is in LDS.
//   First the multiply-adds of the `before` panels in front whose updates have not reached this panel's columns, on the matrix cores:
// a wave takes 32 columns, the results change hands through LDS.
//   Then group after group: the quantiser across the lanes of a row, amplitude, error, substitution, and the t values,
// which the substitution has brought to all lanes of the row, onto the groups behind (rows of U ascending).  The next group
// is always w[0]: one body for all groups, which stays in the instruction cache.
template <int D, bool LS, int ROWS, int PANELS>
__device__ inline void panel_role(float *__restrict__ W, const float *__restrict__ U, const t_buffers<PANELS> &T, const correct_shape &a,
                                  int panel, int own, int width, float *lds)
{
    using S = split<D>;
    constexpr int L = S::L, C = S::C, NG = S::kGroups, RB = ROWS / 16;
    int tid = threadIdx.x;
    if constexpr (PANELS > 1) asm volatile("" : "+v"(tid));     // (else what follows from it is kept over both panels)
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & (L - 1);
    const int64_t p0 = (int64_t)panel * kPanelCols;
    const int before = PANELS == 1 ? (panel > 0 ? 1 : 0) : panel < PANELS ? panel : own;      // panels in front whose updates it lacks
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int rloc = wave * S::kRowsOfWave + lane / L;
    const bool in = rloc < ROWS && row0 + rloc < a.rows;
    // lanes beyond the rows work on the last row again; they store nothing
    const int64_t row = std::min<int64_t>(row0 + rloc, a.rows - 1);
    float *wrow = W + row * a.ldw + p0 + C * j;
    const int ngroups = width / D;
    const float *Up = U + p0 * a.ldu + p0;                      // row p0 + k, column p0 + c of the factor
    const float diagonal = Up[std::min<int64_t>(tid, width - 1) * (a.ldu + 1)];

    // U on and above the panel's diagonal, on its way from the start: 64 columns of four rows make a piece, of which the panel's
    // right half has 32 and its left half 16; a lane's four values lie side by side in LDS.
    constexpr int kRight = kPanelCols / 4 / kWaves, kMyPieces = kRight + kPanelCols / 8 / kWaves;
    const bool right_half = width > 64;
    float up[kMyPieces][4];
    auto first_row = [&](int x) { return 4 * (wave + kWaves * (x < kRight ? x : x - kRight)); };
    auto fetch_panel = [&]() {
#pragma unroll
        for (int x = 0; x < kMyPieces; x++) {
            // (of a panel that has no right half the left one's, which is not used)
            const float *p = Up + (first_row(x) & (right_half ? 127 : 63)) * a.ldu + (x < kRight && right_half ? 64 : 0);
#pragma unroll
            for (int i = 0; i < 4; i++) up[x][i] = p[i * a.ldu + (uint32_t)lane];
        }
    };
    // Block (G, G + rel) is number G NG - G (G - 1) / 2 + rel, its element (i, C j + c) at ((i / 4 C + c) L + j) 4 + i % 4, so that a
    // lane reads four rows of its column at a time; the diagonal itself apart, as divisors, with zeros in its place and below.
    // EARLY: the pieces that lie behind what the sums need on their way from the matrix cores.
    const int col = lane % D, in_block = (lane / D) * D * D + (col % C * L + col / C) * 4;
    auto store_panel = [&](auto early) {
#pragma unroll
        for (int x = 0; x < kMyPieces; x++) {
            const int least = 4 * kWaves * (x < kRight ? x : x - kRight) / D;   // the piece's group is not below it
            const bool behind = (least * NG - least * (least - 1) / 2) * D * D >= ROWS * S::kXPitch;
            if (behind == (decltype(early)::value) && (x >= kRight || right_half)) {
                const int k = first_row(x), G = k / D, c = x < kRight ? 64 : 0;
                float *to = lds + ((G * NG - G * (G - 1) / 2 - G + c / D) * D * D + (k % D) * (C * L)) + in_block;
                float4 v = make_float4(up[x][0], up[x][1], up[x][2], up[x][3]);
                if (4 * kWaves * (x < kRight ? x : x - kRight) < c) {
                    *reinterpret_cast<float4 *>(to) = v;        // (right of the diagonal as a whole)
                } else if (c + lane >= G * D) {
                    const int below = c + lane - k;             // rows of the piece above the diagonal
                    v.x = below > 0 ? v.x : 0.0f; v.y = below > 1 ? v.y : 0.0f; v.z = below > 2 ? v.z : 0.0f; v.w = below > 3 ? v.w : 0.0f;
                    *reinterpret_cast<float4 *>(to) = v;
                }
            }
        }
    };
    float *divisors = lds + S::kDivisors;
    static_assert(ROWS * S::kXPitch <= S::kDivisors, "divisors lie behind the transposition");
    auto store_divisors = [&]() {
        if (tid < width) {
            const divisor d = column_divisor(diagonal);
            *reinterpret_cast<float4 *>(divisors + 4 * tid) = make_float4(d.b, d.y, d.yl, 0.0f);
        }
    };
    // (lanes beyond the rows of the workgroup have none)
    const bool chain = wave * S::kRowsOfWave < ROWS;
    float w[NG][C];
    if (before > 0) {
        const int c16 = lane & 15, k4 = lane >> 4;              // an operand's row or column, and its place in k
        const bool cols_in = 32 * wave < width;
        f32x4 acc[RB][2];
        constexpr int kAhead = 8;                               // operands of so many instructions are on their way while as many are used
        float uv[2][kAhead][2];
        // (a wave without columns reads the first ones)
        const float *ub = U + (p0 - before * kPanelCols + k4) * a.ldu + p0 + (cols_in ? 32 * wave : 0) + c16;
        auto fetch = [&](float (&v)[kAhead][2]) {
#pragma unroll
            for (int s = 0; s < kAhead; s++) { v[s][0] = ub[0]; v[s][1] = ub[16]; ub += 4 * a.ldu; }
        };
        f32x4 tq[2][RB][kAhead / 4];
        auto fetch_t = [&](const float *Tb, int h) {
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                const t_rows t(std::min<int64_t>(row0 + 16 * rb + c16, a.rows - 1), a.rows);
#pragma unroll
                for (int i = 0; i < kAhead / 4; i++) tq[h & 1][rb][i] = *t.piece(Tb, kAhead / 4 * h + i, k4);
            }
        };
        fetch(uv[0]);
        fetch_t(T.of[PANELS == 1 ? 0 : own - before], 0);
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const float *p = W + std::min<int64_t>(row0 + 16 * rb + c16, a.rows - 1) * a.ldw + p0 + (cols_in ? 32 * wave : 0) + 4 * k4;
            acc[rb][0] = *reinterpret_cast<const f32x4 *>(p);
            acc[rb][1] = *reinterpret_cast<const f32x4 *>(p + 16);
        }
        constexpr int kSteps = kPanelCols / 4 / kAhead;
        static_assert(kSteps % 2 == 0, "the next panel's first operands go where its own are");
        fetch_panel();
#pragma unroll 1
        for (int b = PANELS > 1 ? before : 1; b > 0; b--) {
            const float *Tb = T.of[PANELS == 1 ? 0 : own - b];
#pragma unroll
            for (int h = 0; h < kSteps; h++) {
                if (h + 1 < kSteps) { fetch(uv[(h + 1) & 1]); fetch_t(Tb, h + 1); }
                else if (PANELS > 1 && b > 1) { fetch(uv[0]); fetch_t(T.of[own - b + 1], 0); }
                if (ROWS == 16 && h == 1 && (PANELS == 1 || b == 1)) { store_panel(std::true_type{}); store_divisors(); }
#pragma unroll
                for (int s = 0; s < kAhead; s++)
#pragma unroll
                    for (int rb = 0; rb < RB; rb++)
#pragma unroll
                        for (int x = 0; x < 2; x++)
                            acc[rb][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[h & 1][s][x], tq[h & 1][rb][s / 4][s % 4], acc[rb][x], 0, 0, 0);
            }
        }
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int h = 0; h < 2; h++)
                if (cols_in) *reinterpret_cast<f32x4 *>(lds + (16 * rb + c16) * S::kXPitch + 32 * wave + 16 * h + 4 * k4) = acc[rb][h];
        __syncthreads();
#pragma unroll
        for (int g = 0; g < NG; g++)
#pragma unroll
            for (int c = 0; c < C; c++) w[g][c] = chain ? lds[rloc * S::kXPitch + (g < ngroups ? g : 0) * D + C * j + c] : 0.0f;
        __syncthreads();
    } else {
        fetch_panel();
        store_divisors();
        store_panel(std::true_type{});
#pragma unroll
        for (int g = 0; g < NG; g++)
#pragma unroll
            for (int c = 0; c < C; c++) w[g][c] = wrow[(g < ngroups ? g : 0) * D + c];
    }

    store_panel(std::false_type{});
    if (ROWS > 16 && before > 0) { store_panel(std::true_type{}); store_divisors(); }   // (there are no registers for it in front)
    __syncthreads();

    // What the next panel reads of U comes to this die's L2 meanwhile: its rows in the next panel's columns and the next panel's
    // own, 2 x 128 rows of four 128-byte lines, a lane each (rows lie far apart, so that a first touch is a page's first touch
    // too: 64 rows 17.7 us a panel, 18.6 without).
    constexpr int kTouches = 16 / kWaves;
    float touched[kTouches] = {};
    if (p0 + 2 * kPanelCols <= a.cols) {
#pragma unroll
        for (int x = 0; x < kTouches; x++) touched[x] = Up[(int64_t)(tid / 4 + 16 * kWaves * x) * a.ldu + kPanelCols + tid % 4 * 32];
    }
    float *Tcur = T.of[PANELS == 1 ? 1 : own];
    const t_rows trow(row, a.rows);                             // t values, negated
    const float *ublk = lds + j * 4;                            // block (G, G), the lane's column
    bool plain = true;
    auto arrived = [&]() {
#pragma unroll
        for (int x = 0; x < kTouches; x++) asm volatile("" : : "v"(touched[x]));
    };
    if (!chain) { arrived(); return; }
#pragma unroll 1
    for (int G = 0; G < ngroups; G++) {
        float wg[C], u[C][D], mine[C], tb[D];
        divisor d[C];
#pragma unroll
        for (int c = 0; c < C; c++) {
            wg[c] = w[0][c];
#pragma unroll
            for (int i = 0; i < D; i += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(ublk + (i / 4 * C + c) * L * 4);
                u[c][i] = v.x; u[c][i + 1] = v.y; u[c][i + 2] = v.z; u[c][i + 3] = v.w;
            }
            const float4 v = *reinterpret_cast<const float4 *>(divisors + 4 * (G * D + C * j + c));
            d[c].b = v.x; d[c].y = v.y; d[c].yl = v.z;
        }
        // onto the groups behind: w[rel] less the products with the block's rows, ascending
        auto behind = [&](int rel, int c) {
            float v = w[rel][c];
#pragma unroll
            for (int i = 0; i < D; i += 4) {
                const float4 q = *reinterpret_cast<const float4 *>(ublk + rel * D * D + (i / 4 * C + c) * L * 4);
                v = __builtin_fmaf(-tb[i], q.x, v); v = __builtin_fmaf(-tb[i + 1], q.y, v);
                v = __builtin_fmaf(-tb[i + 2], q.z, v); v = __builtin_fmaf(-tb[i + 3], q.w, v);
            }
            return v;
        };
        // the first ones beside the substitution
        float near[S::kPast][C];
        f32x4 q[S::kPast][C][D / 4];
#pragma unroll
        for (int n = 0; n < S::kNear; n++)
#pragma unroll
            for (int c = 0; c < C; c++)
#pragma unroll
                for (int i = 0; i < D; i += 4) q[n][c][i / 4] = *reinterpret_cast<const f32x4 *>(ublk + (n + 1) * D * D + (i / 4 * C + c) * L * 4);
        auto next = [&](int i) {
#pragma unroll
            for (int n = 0; n < S::kNear; n++)
#pragma unroll
                for (int c = 0; c < C; c++) near[n][c] = __builtin_fmaf(-tb[i], q[n][c][i / 4][i % 4], i == 0 ? w[n + 1][c] : near[n][c]);
        };
        // A group without a direction, with zeros in its error, or with values near either end of the type, is rare, and the wave
        // takes its groups again with the operations that serve every argument; not so in a row of such groups, where the last
        // one tells (a third of the rows zero, 1024 x 4096: 970 us where each is taken twice, now 800; none zero 680 either way).
        bool right = false;
        if (plain) right = __all(solve_group<D, LS, true>(wg, u, d, j, a.K, tb, mine, next));
#pragma unroll
        for (int n = 0; n < S::kNear; n++)
#pragma unroll
            for (int c = 0; c < C; c++) asm volatile("" : "+v"(near[n][c]));   // (here, not behind the branch)
        plain = right;
        if (!right) plain = __all(solve_group<D, LS, false>(wg, u, d, j, a.K, tb, mine, next));
        // what was quantised stays in W
        if (in) {
#pragma unroll
            for (int c = 0; c < C; c++) { wrow[c] = wg[c]; *trow.column(Tcur, G * D + C * j + c) = -mine[c]; }
        }
        // the groups behind move up by one; those that are further off four at a time, as many of them as there are
#pragma unroll
        for (int rel = 1; rel <= S::kNear; rel++)
#pragma unroll
            for (int c = 0; c < C; c++) w[rel - 1][c] = near[rel - 1][c];
#pragma unroll
        for (int r4 = S::kNear + 1; r4 < NG; r4 += 4) {
            if (G + r4 < ngroups) {
#pragma unroll
                for (int rel = r4; rel < r4 + 4 && rel < NG; rel++)
#pragma unroll
                    for (int c = 0; c < C; c++) w[rel - 1][c] = behind(rel, c);
            }
        }
        ublk += (NG - G) * D * D;
        wrow += D;
    }
    arrived();
}

// Update role.  Rows [row0, row1), columns [col0, col0 + 64): W[r][c] <- W[r][c] - t[r][0] U[c0][c] - ... (128 or 256 of them), one
// multiply-add after the other, t = the t values of the panels from column c0 on, on the matrix cores: v_mfma_f32_16x16x4_f32 adds its
// four products one by one, k ascending, each a fused multiply-add (bit for bit, subnormals, infinities and NaN included).
// The workgroup has its part of U in LDS, after which its waves do not wait for each other: a wave takes 16 rows at a time.  Their W is
// requested an item ahead and t values (as operands, t_rows) eight pieces ahead, into the registers that have just been used, and no store is
// under a condition: memory operations complete in order, so a wait for a load that may or may not have stores behind it would
// wait for the stores too (update alone, 8192 rows x 3968 columns: 87 us so, now 76).  Items of 32 rows, an operand of U for eight
// instructions, take longer (8192 x 8192 5.02 / 5.17 ms).
// IN_ORDER: the instructions stay as they are written.  Not where a wave mostly has one item, with one panel a launch of up to 2048 rows in
// groups of 8 (1024 x 8192 1582 / 1568 us, 1280 x 8192 1719 / 1697; 3000 x 4096 1009 / 1040).
template <int PANELS, bool IN_ORDER>
__device__ inline void update_role(float *__restrict__ W, const float *__restrict__ U, const t_buffers<PANELS> &T, const correct_shape &a,
                                   int panel, int64_t col0, int64_t row0, int64_t row1, float *lds)
{
    constexpr int kDeep = PANELS * kPanelCols;
    constexpr int kPieces = kDeep / 16;           // float4 of t values of a lane for a row, each for four instructions in a row
    constexpr int kRing = kPanelCols / 16;
    const int64_t c0 = (int64_t)panel * kPanelCols;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, k4 = lane >> 4;
    // U as operands: the four blocks of 16 columns side by side, so that an instruction's four are one read
    float uq[kDeep * 16 / kThreads][4];
    {
        const float *up = U + (c0 + (tid >> 4)) * a.ldu + col0 + (tid & 15);
#pragma unroll
        for (int x = 0; x < kDeep * 16 / kThreads; x++) {
#pragma unroll
            for (int q = 0; q < 4; q++) uq[x][q] = up[16 * q];
            up += kThreads / 16 * a.ldu;
        }
    }
    // The instruction's rows are columns of W, so that a lane's four results are neighbours: row c16 of the item's, columns
    // 16 cb + 4 k4 .. + 3.  A row that is not there is the last one once more, which gets the same values.
    f32x4 w[4], t[kRing];
    auto place = [&](int64_t r) { return W + (r + std::min<int64_t>(c16, a.rows - 1 - r)) * a.ldw + col0 + 4 * k4; };
    auto fetch_w = [&](int64_t r) {
        const float *p = place(r);
#pragma unroll
        for (int cb = 0; cb < 4; cb++) w[cb] = *reinterpret_cast<const f32x4 *>(p + 16 * cb);
    };
    auto fetch_piece = [&](int64_t r, int i) {
        const int n = (int)std::min<int64_t>(kItemRows, a.rows - r);      // (t_rows, whose block is the item)
        t[i % kRing] = *reinterpret_cast<const f32x4 *>(T.of[i / kRing] + r * kPanelCols + 16 * n * (i % kRing) +
                                                        (uint32_t)(4 * std::min(c16, n - 1) + 4 * n * k4));
    };
    int64_t r = row0 + kItemRows * wave;
    int items = r < row1 ? (int)((row1 - r + kStepRows - 1) / (kStepRows)) : 0;
    if (items > 0) {
#pragma unroll
        for (int i = 0; i < kRing; i++) fetch_piece(r, i);
        fetch_w(r);
    }
#pragma unroll
    for (int x = 0; x < kDeep * 16 / kThreads; x++)
        *reinterpret_cast<f32x4 *>(lds + (tid + x * kThreads) * 4) = f32x4{uq[x][0], uq[x][1], uq[x][2], uq[x][3]};
    __syncthreads();
    int at = lane;                                                         // ([4 s + k4][c16])
    auto item = [&](auto more) {
        constexpr bool kMore = decltype(more)::value;
        asm volatile("" : "+v"(at));              // (the operands are the same for all rows, and more than there are registers)
        const f32x4 *us = reinterpret_cast<const f32x4 *>(lds) + at;
        const int64_t next = r + kStepRows;
        f32x4 acc[4];
#pragma unroll
        for (int cb = 0; cb < 4; cb++) acc[cb] = w[cb];
        if constexpr (kMore) fetch_w(next);
        f32x4 uv[2];
        uv[0] = us[0];
#pragma unroll
        for (int s = 0; s < kDeep / 4; s++) {
            if (s + 1 < kDeep / 4) uv[(s + 1) & 1] = us[(s + 1) * 64];
#pragma unroll
            for (int cb = 0; cb < 4; cb++) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[s & 1][cb], t[s / 4 % kRing][s % 4], acc[cb], 0, 0, 0);
            if (s % 4 == 3) {
                const int i = s / 4 + kRing;
                if (i < kPieces) fetch_piece(r, i);
                else if constexpr (kMore) fetch_piece(next, i - kPieces);
            }
            if constexpr (IN_ORDER) __builtin_amdgcn_sched_barrier(0);
        }
        float *p = place(r);
#pragma unroll
        for (int cb = 0; cb < 4; cb++) *reinterpret_cast<f32x4 *>(p + 16 * cb) = acc[cb];
        r = next;
    };
    for (; items > 1; items--) item(std::true_type{});
    if (items > 0) item(std::false_type{});
}

// The PANELS panels from number `panel` on (128 columns each, 64 at the end), and the panels in front of them, as many, onto the columns
// behind.  The grid is panel_wgs + chunks * shares workgroups, the latter none for panel 0: the updates' rows are in up to eight chunks, which
// neighbouring workgroups, on different dies, take in turn, so that with eight a chunk's t values are read from one L2 (with fewer, from one of
// two or more); a chunk's steps of 64 rows times 64 columns are shared out evenly.
// (at most 128 registers per lane with one panel, four workgroups per compute unit, three for groups of 32, whose blocks take more LDS)
template <int D, bool LS, int ROWS, int PANELS>
__global__ __launch_bounds__(kThreads, PANELS > 1 ? 2 : D == 32 ? 3 : 4) void correct_step_kernel(float *__restrict__ W, const float *__restrict__ U,
                                                                 t_buffers<PANELS> T, correct_shape a, int panel, int panel_wgs, update_split parts, int late)
{
    __shared__ __align__(16) float lds[lds_floats<D, PANELS>()];
    if ((int)blockIdx.x < panel_wgs) {
        // the chain's waves go first where they share a SIMD with update waves, which have plenty of others to fill in
        __builtin_amdgcn_s_setprio(2);
#pragma unroll 1
        for (int x = 0; x < PANELS; x++) {
            const int64_t left = a.cols - (int64_t)(panel + x) * kPanelCols;
            if (left <= 0) break;
            if (x > 0) {
                // the panel before has left its t values, and nobody needs its LDS any more
                __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
                __syncthreads();
            }
            panel_role<D, LS, ROWS, PANELS>(W, U, T, a, panel + x, PANELS + x, (int)std::min<int64_t>(kPanelCols, left), lds);
        }
    } else {
        // With few rows the chain is what a launch waits for, and its first reads stand in line with those of all tasks (1024 rows of
        // 8192: its front 4 us alone, 12 to 15 beside them); the tasks, 15 to 27 us in all, let it go first by `late` times 0.43 us.
        for (int x = 0; x < late; x++) __builtin_amdgcn_s_sleep(16);
        const uint32_t wg = blockIdx.x - panel_wgs, share = wg >> parts.log2_chunks, chunk = wg - (share << parts.log2_chunks);
        const bool more = chunk < parts.longer;
        const uint32_t steps = parts.steps + (more ? 1u : 0u), first = chunk * parts.steps + std::min(chunk, parts.longer);
        const uint32_t each = parts.each[more], rest = parts.rest[more];
        uint32_t at = share * each + std::min(share, rest);
        const uint32_t end = at + each + (share < rest ? 1u : 0u);
        while (at < end) {
            const uint32_t tile = at / steps, from = at - tile * steps, to = std::min(steps, from + end - at);
            update_role<PANELS, PANELS != 1 || D != 8 || ROWS != 16>(W, U, T, a, panel - PANELS, (int64_t)(panel + PANELS) * kPanelCols + (int64_t)tile * kTileCols,
                                (int64_t)(first + from) * kStepRows, std::min<int64_t>((int64_t)(first + to) * kStepRows, a.rows), lds);
            at += to - from;
            if (at < end) __syncthreads();
        }
    }
}

template <int D, int ROWS, int PANELS>
void launch_step(float *W, const float *U, float *work, const correct_shape &a, int panel, hipStream_t s)
{
    t_buffers<PANELS> T;                           // 2 PANELS buffers, used in turn
    for (int x = 0; x < 2 * PANELS; x++) T.of[x] = work + (panel + PANELS + x) % (2 * PANELS) * a.rows * kPanelCols;
    const int64_t behind = a.cols - (int64_t)(panel + PANELS) * kPanelCols;
    const int col_tiles = panel > 0 && behind > 0 ? (int)(behind / kTileCols) : 0;
    const int panel_wgs = (int)((a.rows + ROWS - 1) / ROWS);
    // Update workgroups.  Where every unit has as many panel workgroups as the others, one beside them: they all start with the launch,
    // and whatever the columns are they end together; with one panel a launch also where all panel workgroups have a place at once.
    // Elsewhere some units are ahead, and smaller shares let them take more.  (Shares 256 / 1024 / 2048 / 4096, us.  Two panels a launch:
    // 8192 x 8192 5020 / 5370 / - / 5940, 16384 x 4096 2850 / 2820 / 2900 / 2990, 32768 x 4096 5590 / 5660 / 5710 / 5810, but 8200 x 8192 5980 / 5600 / 5490 / 5690,
    // 20000 x 4096 5200 / 3660 / 3630 / 3690, in groups of 16 10000 x 4096 2740 / 2000 / 2010 / -; 3000 x 8192 2750 / 2650 / - / 2750, 1024 x 8192 1640 / 1550 / - /
    // 1480.  One panel: 8200 x 8192 5870 / 6000 / 5830 / 5870, 16384 x 4096 3020 / 3150 / 3020 / 3070, in groups of 32 7168 x 4096 1490 / 1540 / 1500 / -; 2048 x 8192
    // - / 2170 / 2080 / 2140, in groups of 16 - / 2000 / 1910 / 1980.  Where a unit does not hold them all the last panel workgroups have update
    // workgroups in front of them: one panel 40000 x 4096 10900 / 7650 / 7460 / 7650, in groups of 32 14336 x 4096 4130 / 2810 / 2740 / -.)
    constexpr uint32_t kUnits = 256, kPlaces = (D == 32 ? 3 : 4) * kUnits;
    const uint32_t steps = (uint32_t)((a.rows + kStepRows - 1) / kStepRows), chain = (uint32_t)panel_wgs;
    const bool even = 16 * ((chain + kUnits - 1) / kUnits * kUnits - chain) <= chain;
    const bool beside = chain >= kUnits && (PANELS > 1 ? even : chain <= kPlaces || (even && chain <= 4 * kUnits));
    const uint32_t most = beside ? kUnits : chain > kUnits ? 8 * kUnits : a.rows > 2048 ? 4 * kUnits : (PANELS > 1 ? 16 : 8) * kUnits;
    update_split parts;
    // As many chunks as take about the same number of steps: a die whose chunks have one step in two more than the others' keeps
    // the launch waiting (768 rows, 12 steps, of 8192: in eight chunks 1507 us, in four 1451; 1280 rows in eight 1756, in four 1638; 320 rows
    // in four 1317, in one 1290).
    parts.log2_chunks = 3;
    auto rows_of_chunks = [&]() { return (int64_t)(steps + (1u << parts.log2_chunks) - 1 >> parts.log2_chunks << parts.log2_chunks) * kStepRows; };
    while (parts.log2_chunks > 0 && 16 * (rows_of_chunks() - a.rows) > a.rows) parts.log2_chunks--;
    const uint32_t chunks = 1u << parts.log2_chunks;
    parts.steps = steps / chunks;
    parts.longer = steps % chunks;
    const uint32_t shares = (uint32_t)std::min<uint64_t>(most / chunks, (uint64_t)(parts.steps + (parts.longer ? 1 : 0)) * col_tiles);
    for (uint32_t more = 0; more < 2; more++) {
        const uint32_t all = (parts.steps + more) * (uint32_t)col_tiles;      // (fewer than 2^32: the matrix has 4096 values for each, 16 KiB)
        parts.each[more] = shares ? all / shares : 0;
        parts.rest[more] = shares ? all % shares : 0;
    }
    // How long the updates wait, in 0.43 us: with one panel a launch until the rest of its chain is about what they take, so less with more
    // of them.  (0 / 4 / 7 / 10 / 12, us, in groups of 8: 256 x 8192 1200 / 1160 / 1160 / 1170 / 1150, 512 x 4096 613 / 608 / - / 599 / 591, 768 x 4096 675 / 662 /
    // 655 / 646 / 643, 1024 x 8192 1600 / 1590 / 1580 / 1580 / -, 1280 x 8192 1720 / 1710 / 1710 / 1730 / -, 2048 x 8192 2100 / 2080 / 2100 / 2160 / -; of 16 768 x 4096 530 /
    // 513 / 504 / 497 / -, 1024 x 6144 906 / 890 / 899 / 919 / -, 2048 x 6144 1210 / 1240 / 1270 / 1320 / -.  Two panels: 1024 x 4096 756 to 714, 2048 x 4096 869 to 830.
    // More than 2048 rows: none, 4096 x 4096 1090 either way.)
    int late = 0;
    if (a.rows <= 2048) {
        const int64_t n = a.rows * a.cols;
        if (PANELS > 1) late = 8;
        else if (D == 8) late = n <= 5 << 20 ? 12 : n <= 8 << 20 ? 10 : 4;
        else late = n < 4 << 20 ? 10 : n < 6 << 20 ? 8 : n <= 8 << 20 ? 4 : 0;
    }
    auto kernel = a.ls ? &correct_step_kernel<D, true, ROWS, PANELS> : &correct_step_kernel<D, false, ROWS, PANELS>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)panel_wgs + chunks * shares), dim3(kThreads), 0, s,
                       W, U, T, a, panel, panel_wgs, parts, late);
}

template <int D, int PANELS>
hipError_t launch_panels(float *W, const float *U, float *work, const correct_shape &a, hipStream_t s)
{
    const int panels = (int)((a.cols + kPanelCols - 1) / kPanelCols);
    for (int p = 0; p < panels; p += PANELS) {
        // With few rows, which do not fill the units either way, a panel workgroup takes 16: half the matrix instructions in front
        // (64 x 2048 17.8 to 16.6 us a panel, 2048 x 4096 26.0 to 25.2; 4096 x 4096 34.1 to 35.0).
        if (a.rows <= 2048) launch_step<D, 16, PANELS>(W, U, work, a, p, s);
        else launch_step<D, split<D>::kMost, PANELS>(W, U, work, a, p, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int PANELS>
hipError_t launch_panels(int D, float *W, const float *U, float *work, const correct_shape &a, hipStream_t s)
{
    switch (D) {
    case 8: return launch_panels<8, PANELS>(W, U, work, a, s);
    case 16: return launch_panels<16, PANELS>(W, U, work, a, s);
    default: return launch_panels<32, PANELS>(W, U, work, a, s);
    }
}

// W: rows x cols float32 (cols a multiple of 64), U: cols x cols, work: `buffers` (two or four) of rows x 128 floats.
// Two panels a launch where the updates are what there is to wait for; with few rows, or up to 2048 of a narrow matrix, it is the chain,
// whose fronts get longer, and so it is where the panel workgroups are more than the two for every unit that have a place at once, and the
// columns few (one / two panels in groups of 8, 512 x 8192 1343 / 1378 us, 768 x 6144 1020 / 1039, 768 x 8192 1451 / 1451,
// 1024 x 2048 294 / 311, 1024 x 4096 670 / 667, 1280 x 2560 397 / 406, 1280 x 3072 497 / 497, 1536 x 2048 318 / 321, 2048 x 2048 338 / 330,
// 8192 x 704 138 / 128; in groups of 16 1024 x 4096 531 / 522, 768 x 8192 1218 / 1163, in groups of 32 547 / 540, 1273 / 1196;
// 16384 x 1024 318 / 306, 16400 x 1024 324 / 402, 16400 x 3072 1812 / 1900, 20000 x 3072 2164 / 2247, 16400 x 4096 3056 / 3031, 20000 x 4096 3708 / 3629; 32768 x 1536
// 997 / 1071, 32768 x 2048 1724 / 1667, 40000 x 2048 2104 / 2061, 65536 x 3072 7176 / 6620; in groups of 16, 16 rows a workgroup, 8192 x 1024 203 / 188, 8200 x 2048
// 560 / 592, 10000 x 4096 2011 / 2009, 20000 x 2048 1129 / 1177, 20000 x 4096 3801 / 3717).
hipError_t launch_correct(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                          int64_t ldu, float *work, int buffers, hipStream_t s)
{
    correct_shape a;
    a.ldw = ldw; a.rows = rows; a.cols = cols; a.ldu = ldu; a.K = c->K; a.ls = c->amplitude == PVQ_AMP_LS ? 1 : 0;
    const int64_t most_rows = c->D == 8 ? split<8>::kMost : split<16>::kMost, chain = (rows + most_rows - 1) / most_rows;
    const bool at_once = chain <= 512 || cols >= (chain > 960 && c->D == 8 ? 2048 : 4096);
    const bool two = buffers == 4 && (rows > 2048 ? at_once : rows > 512 && (rows - 512) * cols >= 1 << 21);
    return two ? launch_panels<2>(c->D, W, U, work, a, s) : launch_panels<1>(c->D, W, U, work, a, s);
}

// Work buffers of the entry point that allocates nothing: the t values of two panels for up to kStaticRows rows
// (twice 128 floats per row), 8 MiB on every GPU that loads the library, until the process ends; of four for up to half the rows.
constexpr int64_t kStaticRows = 8192;
static __device__ __align__(256) float scratch[2 * kStaticRows * kPanelCols];

// The array's address on each device (in host code the array's name is only a stand-in for it), asked
// for once per device with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
float *g_scratch_ptr[kMaxDevices] = {};

hipError_t scratch_on_current_device(float **ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

hipError_t pvq_launch_correct(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                              int64_t ldu, float *work, hipStream_t s)
{
    return launch_correct(c, W, rows, cols, ldw, U, ldu, work, 2, s);
}

hipError_t pvq_launch_correct_two_panels(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                                         int64_t ldu, float *work, hipStream_t s)
{
    return launch_correct(c, W, rows, cols, ldw, U, ldu, work, 4, s);
}

int64_t pvq_correct_static_max_rows(void) { return kStaticRows; }

// The same launches with the library's own work buffers.
hipError_t pvq_launch_correct_static(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw,
                                     const float *U, int64_t ldu, hipStream_t s)
{
    if (rows > kStaticRows) return hipErrorInvalidValue;   // (the entry point has refused it already)
    float *work = nullptr;
    const hipError_t e = scratch_on_current_device(&work);
    if (e != hipSuccess) return e;
    return launch_correct(c, W, rows, cols, ldw, U, ldu, work, 2 * rows <= kStaticRows ? 4 : 2, s);
}
