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
// of 128, a launch per panel on the caller's stream (correct_step_kernel), whose workgroups have one of two roles:
//     panel   (the first workgroups, 32 or 16 rows each) panel p - 1's 128 multiply-adds per element onto the panel's columns,
//             which is all that panel p waits for, then the panel's groups one after the other, a row across 8 or 16
//             lanes.  Leaves the panel's t values (rows x 128) in a work buffer.  Bound by the latency of one chain:
//             23 us for 16 groups of 8.
//     update  (all others) panel p - 1's 128 multiply-adds per element, in the same order, for the columns behind panel p:
//             tiles of 128 rows x 128 columns, W read and written once per panel.  Bound: float32 matrix instructions
//             (143 TFLOP/s in registers) and HBM together, 100 TFLOP/s at 63 x 64 tiles.
// The two roles touch different columns, and the update reads panel p - 1's t values while the panel role writes
// panel p's, which is why there are two work buffers used in turn.  The panel workgroups come first in the grid
// and raise their waves' priority, so they are placed before the flood of update tiles and run beside it: the
// chain of panels (each needs the one before) stays off the critical path as long as a launch has enough update
// tiles to outlast it; with few rows the chain is what remains.  A workgroup has the LDS of the role that needs more: 36.9 KB
// in groups of 8 (the update's), 39.9 in groups of 16 (the panel's), four workgroups to a compute unit; 53.2 in groups of
// 32, three.
// Both roles' 128 multiply-adds per element run on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four products to an
// element one by one, k ascending, each a fused multiply-add (measured bit for bit against fmaf over random, cancelling,
// tied, subnormal and non-finite operands).
// Before, with the update on the vector ALU (64 TFLOP/s) and 64 rows of a panel a lane each on four waves that took its
// groups in turn (37 to 46 us a panel and 10 to 15 for a launch in front of it with its update): 8192 x 8192 9.5 ms, now
// 6.7; 1024 x 4096 1.6 ms, now 0.92; 1024 x 8192 3.3, now 2.07; 28672 x 8192 29.5, now 21.2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "pvq_internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kPanelCols = 128;   // columns per panel
constexpr int kWaves = 4;         // waves of a workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kTile = 128;        // rows and columns of an update tile
constexpr int kStage = 32;        // rows of U (and t values per row) that an update tile holds in LDS at a time
// words from a row of t values, or of U, in LDS to the next: the 64 values of an operand lie on different banks
constexpr int kTPitch = kStage + 4, kUPitch = kTile + 16;
constexpr int kUpdateFloats = kTile * kTPitch + kStage * kUPitch;

struct correct_shape {
    int64_t ldw, rows, cols, ldu;
    int K, ls;
};

// ---- a row's group across L neighbouring lanes, C = D / L coordinates a lane --------------------------------
template <int D> struct split {
    static constexpr int L = D == 8 ? 8 : 16, C = D / L;
    static constexpr int kRowsOfWave = 64 / L, kRows = kWaves * kRowsOfWave;   // of a workgroup
    static constexpr int kGroups = kPanelCols / D;
    // LDS of the panel role: D x D blocks of U on and above the panel's diagonal, before that t values and sums on their way
    // to and from the matrix cores' layout (kXPitch: an operand's values lie on different banks)
    static constexpr int kBlocks = kGroups * (kGroups + 1) / 2;
    static constexpr int kFloats = (kBlocks + 3) * D * D;      // (a trailing update reads up to three blocks past the last)
    static constexpr int kXPitch = kPanelCols + 4;
    static_assert(kRows * kXPitch <= kFloats, "the transposition fits");
};
template <int D> constexpr int lds_floats() { return kUpdateFloats > split<D>::kFloats ? kUpdateFloats : split<D>::kFloats; }

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
    const int i = __float_as_int(v);
    if constexpr (L == 16) return __int_as_float(dpp<0x150 + N>(0, i));                        // row_newbcast
    else return __int_as_float(dpp<0x150 + 8 + N, 0xC>(dpp<0x150 + N>(0, i), i));              // one for either half
}

// How many coordinates of lanes j ^ X, X = 1 .. L - 1, come before coordinate c of this lane in the order of keys (largest
// first, lower coordinate first on ties): key > mine, or >= where the other lane is the lower one (th: mine, less one
// where bit b of j says so).
template <int L, int C, int X>
__device__ inline void count_before(const int (&key)[C], const int (&th)[C][4], int (&before)[C])
{
    if constexpr (X < L) {
        constexpr int b = X < 2 ? 0 : X < 4 ? 1 : X < 8 ? 2 : 3;
#pragma unroll
        for (int o = 0; o < C; o++) {
            const int other = lane_xor<X>(key[o]);
#pragma unroll
            for (int c = 0; c < C; c++) before[c] += other > th[c][b] ? 1 : 0;
        }
        count_before<L, C, X + 1>(key, th, before);
    }
}

// The quantiser of Sec. 2.5 (as in pvq_quantize_dev.h) with the group's coordinates C j .. C j + C - 1 in lane j of its row: the
// same sums in the same order, the coordinates' places in the order of deviations counted by comparisons.  Returns the
// sum of squares; y gets the signed point.
template <int D>
__device__ inline float quantize_lanes(const float (&w)[split<D>::C], int j, int K, int (&y)[split<D>::C])
{
    constexpr int L = split<D>::L, C = split<D>::C;
    float a1 = fabsf(w[0]), s2 = w[0] * w[0];
    if constexpr (C == 2) { a1 = a1 + fabsf(w[1]); s2 = s2 + w[1] * w[1]; }
    const float l1 = lanes_sum<L>(a1), ss = lanes_sum<L>(s2);
    const float g = (float)K / l1;
    const bool degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(g < INFINITY);
    float t[C], yf[C];
    float S = 0.0f;
#pragma unroll
    for (int c = 0; c < C; c++) {
        t[c] = fabsf(w[c]) * g;
        yf[c] = rintf(t[c]);
        S += yf[c];                           // small integers: exact in any order
    }
    S = lanes_sum<L>(S);
    const float m = (float)K - S;             // > 0: pulses to add, < 0: pulses to take away
    const float unit = m < 0.0f ? -1.0f : 1.0f;
    // deviations as integers that order like them (zeros have one sign: t - yf is +0 there)
    int key[C], th[C][4];
#pragma unroll
    for (int c = 0; c < C; c++) {
        const float d = t[c] - yf[c];
        const int b = __float_as_int(m < 0.0f ? -d : d);
        key[c] = b ^ ((b >> 31) & 0x7FFFFFFF);
#pragma unroll
        for (int v = 0; v < 4; v++) th[c][v] = key[c] - ((j >> v) & 1);
    }
    int before[C];
#pragma unroll
    for (int c = 0; c < C; c++) before[c] = 0;
    if constexpr (C == 2) {
        const int first = key[0] >= key[1] ? 1 : 0;
        before[1] = first; before[0] = 1 - first;
    }
    count_before<L, C, 1>(key, th, before);
    const int need = (int)fabsf(m);
#pragma unroll
    for (int c = 0; c < C; c++) {
        int mag = (int)(yf[c] + (before[c] < need ? unit : 0.0f));
        if (degenerate) mag = C * j + c == D - 1 ? K : 0;
        y[c] = (w[c] < 0.0f && !degenerate) ? -mag : mag;
    }
    return ss;
}

// t U_GG = e, coordinate after coordinate: t_I is final once t_0 .. t_{I-1} have been taken off e_I.  e: the lane's
// coordinates; u: rows of the block in the lane's columns, ud: its diagonal there.  tb gets all of t, mine the lane's own.
template <int D, int I>
__device__ inline void substitute(float (&e)[split<D>::C], const float (&u)[split<D>::C][D], const float (&ud)[split<D>::C],
                                  int j, float (&tb)[D], float (&mine)[split<D>::C])
{
    constexpr int L = split<D>::L, C = split<D>::C;
    if constexpr (I < D) {
        const float q = e[I % C] / ud[I % C];
        mine[I % C] = j == I / C ? q : mine[I % C];
        tb[I] = lane_broadcast<L, I / C>(q);
#pragma unroll
        for (int c = 0; c < C; c++) e[c] = __builtin_fmaf(-tb[I], u[c][I], e[c]);
        substitute<D, I + 1>(e, u, ud, j, tb, mine);
    }
}

// Panel role.  A workgroup takes split<D>::kRows rows, a wave 8 (D = 8) or 4 of them: lane (row, j) holds coordinate(s) j of
// every group of the panel, and the waves do not wait for each other once the panel's part of U is in LDS.
//   First the panel before's 128 multiply-adds per element onto this panel's columns, on the matrix cores: a wave takes 32
// columns, the results change hands through LDS.
//   Then group after group: the quantiser across the lanes of a row, amplitude, error, substitution, and the t values,
// which the substitution has brought to all lanes of the row, onto the groups behind (rows of U ascending).  The next group
// is always w[0]: one body for all groups, which stays in the instruction cache.
template <int D>
__device__ inline void panel_role(float *__restrict__ W, const float *__restrict__ U, const float *__restrict__ Tprev,
                                  float *__restrict__ Tcur, const correct_shape &a, int64_t p0, int width, float *lds)
{
    using S = split<D>;
    constexpr int L = S::L, C = S::C, NG = S::kGroups, RB = S::kRows / 16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & (L - 1);
    const int64_t row0 = (int64_t)blockIdx.x * S::kRows;
    const int rloc = wave * S::kRowsOfWave + lane / L;
    const bool in = row0 + rloc < a.rows;
    // lanes beyond the rows work on the last row again; they store nothing
    const int64_t row = std::min<int64_t>(row0 + rloc, a.rows - 1);
    float *wrow = W + row * a.ldw + p0 + C * j;
    const int ngroups = width / D;
    const float *Up = U + p0 * a.ldu + p0;                      // row p0 + k, column p0 + c of the factor

    float w[NG][C];
    if (p0 > 0) {
        // t values of the workgroup's rows
#pragma unroll
        for (int x = 0; x < S::kRows * kPanelCols / 4 / kThreads; x++) {
            const int e = threadIdx.x + x * kThreads, rr = e / (kPanelCols / 4), c4 = (e % (kPanelCols / 4)) * 4;
            *reinterpret_cast<float4 *>(lds + rr * S::kXPitch + c4) =
                *reinterpret_cast<const float4 *>(Tprev + std::min<int64_t>(row0 + rr, a.rows - 1) * kPanelCols + c4);
        }
        const int c16 = lane & 15, k4 = lane >> 4;              // an operand's row or column, and its place in k
        const bool cols_in = 32 * wave < width;
        f32x4 acc[RB][2];
        constexpr int kAhead = 16;                              // operands of so many instructions on their way at a time
        float uv[kAhead][2];
        const float *ub = U + (p0 - kPanelCols + k4) * a.ldu + p0 + 32 * wave + c16;
        auto fetch = [&]() {
#pragma unroll
            for (int s = 0; s < kAhead; s++) { uv[s][0] = ub[0]; uv[s][1] = ub[16]; ub += 4 * a.ldu; }
        };
        if (cols_in) {
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                const float *p = W + std::min<int64_t>(row0 + 16 * rb + c16, a.rows - 1) * a.ldw + p0 + 32 * wave + 4 * k4;
                acc[rb][0] = *reinterpret_cast<const f32x4 *>(p);
                acc[rb][1] = *reinterpret_cast<const f32x4 *>(p + 16);
            }
            fetch();
        }
        __syncthreads();
        if (cols_in) {
#pragma unroll 1
            for (int s0 = 0; s0 < kPanelCols / 4; s0 += kAhead) {
                if (s0) fetch();
#pragma unroll
                for (int s = 0; s < kAhead; s++)
#pragma unroll
                    for (int rb = 0; rb < RB; rb++) {
                        const float tv = lds[(16 * rb + c16) * S::kXPitch + 4 * (s0 + s) + k4];
#pragma unroll
                        for (int h = 0; h < 2; h++) acc[rb][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[s][h], tv, acc[rb][h], 0, 0, 0);
                    }
            }
        }
        __syncthreads();
        if (cols_in) {
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int h = 0; h < 2; h++) *reinterpret_cast<f32x4 *>(lds + (16 * rb + c16) * S::kXPitch + 32 * wave + 16 * h + 4 * k4) = acc[rb][h];
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < NG; g++)
#pragma unroll
            for (int c = 0; c < C; c++) w[g][c] = lds[rloc * S::kXPitch + (g < ngroups ? g : 0) * D + C * j + c];
        __syncthreads();
    } else {
#pragma unroll
        for (int g = 0; g < NG; g++)
#pragma unroll
            for (int c = 0; c < C; c++) w[g][c] = wrow[(g < ngroups ? g : 0) * D + c];
    }

    // U on and above the panel's diagonal: block (G, G + rel) is number G NG - G (G - 1) / 2 + rel, its element (i, C j + c) at
    // ((i / 4 C + c) L + j) 4 + i % 4, so that a lane reads four rows of its column at a time
    constexpr int kQuads = kPanelCols * kPanelCols / 4;         // float4 of the panel's square
    for (int e = threadIdx.x; e < kQuads; e += kThreads) {
        const int k = e / (kPanelCols / 4), c4 = (e % (kPanelCols / 4)) * 4;
        const int G = k / D, g = c4 / D, i = k % D, col = c4 % D;
        if (g >= G && k < width && c4 < width) {
            const float4 v = *reinterpret_cast<const float4 *>(Up + (int64_t)k * a.ldu + c4);
            float *b = lds + (G * NG - G * (G - 1) / 2 + g - G) * D * D + i % 4;
            const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; q++) b[((i / 4 * C + (col + q) % C) * L + (col + q) / C) * 4] = vv[q];
        }
    }
    __syncthreads();

    float *trow = Tcur + row * kPanelCols + C * j;              // t values, negated
    const float *ublk = lds + j * 4;                            // block (G, G), the lane's column
    const int own = C * j;
#pragma unroll 1
    for (int G = 0; G < ngroups; G++) {
        float (&wg)[C] = w[0];
        // what is quantised, and stays in W
        if (in) {
#pragma unroll
            for (int c = 0; c < C; c++) wrow[c] = wg[c];
        }
        float u[C][D], ud[C];
#pragma unroll
        for (int c = 0; c < C; c++) {
#pragma unroll
            for (int i = 0; i < D; i += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(ublk + (i / 4 * C + c) * L * 4);
                u[c][i] = v.x; u[c][i + 1] = v.y; u[c][i + 2] = v.z; u[c][i + 3] = v.w;
            }
            ud[c] = ublk[((own + c) / 4 * C + c) * L * 4 + (own + c) % 4];
        }
        int y[C];
        const float ss = quantize_lanes<D>(wg, j, a.K, y);
        float sq = 0.0f, dot = 0.0f;
#pragma unroll
        for (int c = 0; c < C; c++) {
            const float yc = (float)y[c];
            sq += yc * yc;                                      // integers
            const float p = yc * wg[c];
            dot = c == 0 ? p : dot + p;
        }
        const float root = sqrtf(lanes_sum<L>(sq));
        const float s = a.ls ? lanes_sum<L>(dot) / root : sqrtf(ss);
        const float gain = s / root;
        float e[C], mine[C], tb[D];
#pragma unroll
        for (int c = 0; c < C; c++) { e[c] = wg[c] - gain * (float)y[c]; mine[c] = 0.0f; }
        substitute<D, 0>(e, u, ud, j, tb, mine);
        if (in) {
#pragma unroll
            for (int c = 0; c < C; c++) trow[c] = -mine[c];
        }
        // onto the groups behind, which move up by one; four at a time, as many of them as there are
#pragma unroll
        for (int r4 = 0; r4 < NG; r4 += 4) {
            if (G + r4 + (r4 == 0) < ngroups) {
#pragma unroll
                for (int rel = r4 == 0 ? 1 : r4; rel < r4 + 4 && rel < NG; rel++)
#pragma unroll
                    for (int c = 0; c < C; c++) {
                        float v = w[rel][c];
#pragma unroll
                        for (int i = 0; i < D; i += 4) {
                            const float4 q = *reinterpret_cast<const float4 *>(ublk + rel * D * D + (i / 4 * C + c) * L * 4);
                            v = __builtin_fmaf(-tb[i], q.x, v); v = __builtin_fmaf(-tb[i + 1], q.y, v);
                            v = __builtin_fmaf(-tb[i + 2], q.z, v); v = __builtin_fmaf(-tb[i + 3], q.w, v);
                        }
                        w[rel - 1][c] = v;
                    }
            }
        }
        ublk += (NG - G) * D * D;
        wrow += D;
        trow += D;
    }
}

// Update role.  Tile (row tile, column tile) of the columns [c1, cols): W[r][c] <- W[r][c] - t[r][0] U[c0][c] - ...
// - t[r][127] U[c0 + 127][c], one multiply-add after the other, t = the t values of the panel at column c0, on the matrix
// cores: v_mfma_f32_16x16x4_f32 adds its four products one by one, k ascending, each a fused multiply-add (bit for bit,
// subnormals, infinities and NaN included).  A wave takes 64 x 64 of the tile, a stage = 32 rows of U and 32 t values per row
// in LDS.  Neighbouring workgroups share the tile of U.
__device__ inline void update_role(float *__restrict__ W, const float *__restrict__ U, const float *__restrict__ T,
                                   const correct_shape &a, int64_t c0, int64_t c1, int row_tile, int col_tile, float *lds)
{
    float *Ts = lds;                              // [row of the tile][k], kTPitch words a row
    float *Us = lds + kTile * kTPitch;            // [k][column of the tile], kUPitch words a row
    const int64_t row0 = (int64_t)row_tile * kTile, col0 = c1 + (int64_t)col_tile * kTile;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;      // the wave's 64 rows and 64 columns
    const int c16 = lane & 15, k4 = lane >> 4;
    const bool mine = row0 + 64 * wr < a.rows && col0 + 64 * wc < a.cols;   // (columns come in whole 64s)
    // The instruction's rows are columns of the tile, so that a lane's four results are neighbours: row 16 rb + c16 of the
    // wave's, columns 16 cb + 4 k4 .. + 3.
    f32x4 acc[4][4];
    float *wt = W + (row0 + 64 * wr + c16) * a.ldw + col0 + 64 * wc + 4 * k4;
    const int rows_left = (int)std::min<int64_t>(64, a.rows - (row0 + 64 * wr)) - c16;   // row 16 rb of the lane is there if below this
    if (mine) {
#pragma unroll
        for (int rb = 0; rb < 4; rb++) {
            // (for a row that is not there the wave's last one, whose distance may be negative)
            const float *p = wt + std::min(16 * rb, rows_left - 1) * a.ldw;
#pragma unroll
            for (int cb = 0; cb < 4; cb++) acc[rb][cb] = *reinterpret_cast<const f32x4 *>(p + 16 * cb);
        }
    }
    // the lane's places in a stage's tiles: row tid / 8 and every 32nd one behind it of t, row tid / 32 and every eighth one
    // behind it of U (one pointer that moves on: a pointer per load would take the registers of the sums)
    const bool u_in = col0 + (tid & 31) * 4 < a.cols;
    const float *up = U + (c0 + (tid >> 5)) * a.ldu + col0 + (tid & 31) * 4;
    const float *tp = T + row0 * kPanelCols + (tid & 7) * 4;
    const int t_last = (int)std::min<int64_t>(kTile, a.rows - row0) - 1;
    uint32_t t_at[4];
#pragma unroll
    for (int x = 0; x < 4; x++) t_at[x] = (uint32_t)std::min((tid >> 3) + 32 * x, t_last) * kPanelCols;
#pragma unroll 1
    for (int st = 0; st < kPanelCols / kStage; st++) {
        f32x4 tq[4], uq[4];
#pragma unroll
        for (int x = 0; x < 4; x++) tq[x] = *reinterpret_cast<const f32x4 *>(tp + t_at[x]);
        if (u_in) {
#pragma unroll
            for (int x = 0; x < 4; x++) { uq[x] = *reinterpret_cast<const f32x4 *>(up); up += 8 * a.ldu; }
        } else {
#pragma unroll
            for (int x = 0; x < 4; x++) uq[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        tp += kStage;
        if (st) __syncthreads();                  // the tiles of the stage before are no longer read
#pragma unroll
        for (int x = 0; x < 4; x++) {
            *reinterpret_cast<f32x4 *>(Ts + ((tid >> 3) + 32 * x) * kTPitch + (tid & 7) * 4) = tq[x];
            *reinterpret_cast<f32x4 *>(Us + ((tid >> 5) + 8 * x) * kUPitch + (tid & 31) * 4) = uq[x];
        }
        __syncthreads();
        if (mine) {
#pragma unroll 2
            for (int s = 0; s < kStage / 4; s++) {
                float tv[4], uv[4];
#pragma unroll
                for (int x = 0; x < 4; x++) {
                    tv[x] = Ts[(64 * wr + 16 * x + c16) * kTPitch + 4 * s + k4];
                    uv[x] = Us[(4 * s + k4) * kUPitch + 64 * wc + 16 * x + c16];
                }
#pragma unroll
                for (int rb = 0; rb < 4; rb++)
#pragma unroll
                    for (int cb = 0; cb < 4; cb++) acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[cb], tv[rb], acc[rb][cb], 0, 0, 0);
            }
        }
    }
    if (mine) {
#pragma unroll
        for (int rb = 0; rb < 4; rb++)
            if (16 * rb < rows_left) {
#pragma unroll
                for (int cb = 0; cb < 4; cb++) *reinterpret_cast<f32x4 *>(wt + 16 * rb * a.ldw + 16 * cb) = acc[rb][cb];
            }
    }
}

// The panel at column p0 (its own 128 or 64 columns, and in front of them the panel before's update of those), and the
// panel before's update of the columns from p0 + 128 on.  Tprev: the t values of the panel before (unused for
// p0 = 0), Tcur: where this panel's go.  The grid is panel_wgs + row_tiles * (column tiles behind the panel) workgroups,
// the latter none for p0 = 0.
// (at most 128 registers per lane, four workgroups per compute unit; three for groups of 32, whose blocks take more LDS)
template <int D>
__global__ __launch_bounds__(kThreads, D == 32 ? 3 : 4) void correct_step_kernel(float *__restrict__ W, const float *__restrict__ U,
                                                                 const float *__restrict__ Tprev, float *__restrict__ Tcur,
                                                                 correct_shape a, int64_t p0, int width, int panel_wgs, int row_tiles)
{
    __shared__ __align__(16) float lds[lds_floats<D>()];
    if ((int)blockIdx.x < panel_wgs) {
        // the chain's waves go first where they share a SIMD with update waves, which have plenty of others to fill in
        __builtin_amdgcn_s_setprio(2);
        panel_role<D>(W, U, Tprev, Tcur, a, p0, width, lds);
    } else {
        const int tile = (int)blockIdx.x - panel_wgs;
        update_role(W, U, Tprev, a, p0 - kPanelCols, p0 + kPanelCols, tile % row_tiles, tile / row_tiles, lds);
    }
}

template <int D>
void launch_step(float *W, const float *U, const float *Tprev, float *Tcur, const correct_shape &a, int64_t p0, int width,
                 int row_tiles, int col_tiles, hipStream_t s)
{
    const int panel_wgs = (int)((a.rows + split<D>::kRows - 1) / split<D>::kRows);
    hipLaunchKernelGGL((correct_step_kernel<D>), dim3((unsigned)(panel_wgs + row_tiles * col_tiles)), dim3(kThreads), 0, s,
                       W, U, Tprev, Tcur, a, p0, width, panel_wgs, row_tiles);
}

// W: rows x cols float32 (cols a multiple of 64), U: cols x cols, work: two buffers of rows x 128 floats.
hipError_t launch_correct(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                          int64_t ldu, float *work, hipStream_t s)
{
    correct_shape a;
    a.ldw = ldw; a.rows = rows; a.cols = cols; a.ldu = ldu; a.K = c->K; a.ls = c->amplitude == PVQ_AMP_LS ? 1 : 0;
    const int row_tiles = (int)((rows + kTile - 1) / kTile);
    int p = 0;
    for (int64_t p0 = 0; p0 < cols; p0 += kPanelCols, p++) {
        const int width = (int)std::min<int64_t>(kPanelCols, cols - p0);   // 128, or 64 at the end
        const int64_t behind = cols - (p0 + kPanelCols);
        const int col_tiles = p0 > 0 && behind > 0 ? (int)((behind + kTile - 1) / kTile) : 0;
        float *Tcur = work + (int64_t)(p & 1) * rows * kPanelCols, *Tprev = work + (int64_t)((p & 1) ^ 1) * rows * kPanelCols;
        switch (c->D) {
        case 8: launch_step<8>(W, U, Tprev, Tcur, a, p0, width, row_tiles, col_tiles, s); break;
        case 16: launch_step<16>(W, U, Tprev, Tcur, a, p0, width, row_tiles, col_tiles, s); break;
        default: launch_step<32>(W, U, Tprev, Tcur, a, p0, width, row_tiles, col_tiles, s); break;
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Work buffers of the entry point that allocates nothing: the t values of two panels for up to kStaticRows rows
// (twice 128 floats per row), 8 MiB on every GPU that loads the library, until the process ends.
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
    return launch_correct(c, W, rows, cols, ldw, U, ldu, work, s);
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
    return launch_correct(c, W, rows, cols, ldw, U, ldu, work, s);
}
