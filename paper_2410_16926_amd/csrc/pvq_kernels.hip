// gfx950 kernels of libpvq: the generic encoder (every group size and index width that has no kernel of its
// own); the matching decoders are in pvq_walk.hip.
//
// Work mapping (wave64): one lane owns one group of D weights from load to store, so the group's float32 sums are plain
// register trees with a fixed order.  A team of up to four waves takes whole rows, 64 groups a wave at a time; a workgroup
// has one team or several, which share its tables, and as many workgroups run as the machine holds at once.
//   * The index (App. B.2) is N(D,K) - 1 less one number per coordinate: with U(d,k) = N(d,0) + ... + N(d,k) and C pulses
//     left behind a coordinate that has d coordinates after it, 2 U(d,C-1), and N(d,C) more if it is positive (what is left
//     at the last coordinate: 1 if positive).  These are the thresholds that the decoders compare with.  A workgroup makes
//     their table in LDS from the size table, coordinates next to one another, so that a read's address is one
//     multiply-add from the coordinate before and the coordinate an offset in the instruction.
//   * A wave assembles its 64 indices, 2 b whole words, in words of its own in LDS with ds_or and writes them out.
//   * The row's sum and the amplitude codes are the ones of the encoder for groups of 8 (pvq_quantize_dev.h).
// Bound by instructions, vector and scalar alike: 435 and 97 a group of 16 (16-bit weights, 48 bits, float32 amplitudes).
// Launches in a row: 8192 x 8192 of 16-bit weights, 2-bit codes, groups of 16, 48-bit indices: 52 us; groups of 32, 96 bits: 70 us;
// 3001 x 11008 float32 weights, least-squares amplitudes in 4-bit codes, groups of 16, 52 bits: 32 us; 7001 x 1000
// in groups of 8: 11.7 us.  Before, with the places of the repair marked by masks on the scalar unit (513 and 189): 60, 82, 38, 12.5; with a
// workgroup per row that copied the size table, four reads of it per coordinate, a
// bisection for the code and words assembled by a whole workgroup between barriers: 101, 148, 63, 26.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pvq_internal.h"
#include "pvq_quantize_dev.h"

namespace {

using namespace pvq_quantize_dev;

template <int W> struct wide;
template <> struct wide<1> { using type = uint32_t; };
template <> struct wide<2> { using type = uint64_t; };
template <> struct wide<4> { using type = unsigned __int128; };

constexpr int kMaxLanes = 1024;      // of a workgroup
constexpr int kMaxK = 127;           // of a context with groups of up to 32 (pulses are int8)

struct encode_launch {
    const uint32_t *tab_u;  // [D][K+2] entries of W words
    const float *edges;     // 2^scale_bits (last = +inf)
    int K, index_bits, scale_bits;
    int team;               // lanes that take a row: 64, 128 or 256
    int working;            // teams of a workgroup that take rows; the others help with the table only
};

// LDS, from byte 0: thresholds [2K+2][D-1] of W words, the edges' tree, each wave's words of an index tile, and per team
// two rows' wave sums (used in turn, so that one barrier a row is enough) and the row's sums of squares (every wave reads its own)
struct encode_lds {
    uint32_t tree, stage, stage_words, sums, sum_words, rows, row_words, total;      // starts and total in bytes
};
__host__ __device__ inline encode_lds lds_of(int D, int W, const encode_launch &f, int G, int lanes)
{
    encode_lds l;
    const bool codes = f.scale_bits > 0;
    const uint32_t teams = (uint32_t)(lanes / f.team);
    l.tree = ((uint32_t)(2 * f.K + 2) * (D - 1) * W * 4 + 15) / 16 * 16;
    l.stage = l.tree + (codes ? kEdgeNodes * 16 : 0);
    l.stage_words = 2 * f.index_bits + W;
    l.sums = l.stage + (uint32_t)(lanes / kWave) * l.stage_words * 4;
    l.sum_words = codes ? (uint32_t)(G + kWave * kWave - 1) / (kWave * kWave) * kWave : 0;
    l.rows = (l.sums + 2 * teams * l.sum_words * 4 + 15) / 16 * 16;
    l.row_words = codes ? (uint32_t)(G + 3) / 4 * 4 : 0;
    l.total = l.rows + teams * l.row_words * 4;
    return l;
}

// ---------------------------------------------------------------------------------------------
// encode
// ---------------------------------------------------------------------------------------------

// Waves that a SIMD's registers are divided among (with the repair before: groups of 16, 3001 x 11008: 39 us, with 4 43, with 6, which
// spill, 49; groups of 32, 8192 x 8192, 2-bit codes: 84 us, with 3 118, with 5, which spill, 130).  With these a lane of groups of 16 from
// float32 or with least-squares amplitudes has 2 to 7 values in scratch memory, of groups of 32 9 to 24.
constexpr int waves_per_simd(int D) { return D == 8 ? 7 : D == 16 ? 5 : 4; }

// A group as it comes from memory
template <int D, typename TIn> struct raw_group {
    static constexpr int N = D * (int)sizeof(TIn) / 16;
    uint32_t q[4 * N];
    __device__ void load(const TIn *__restrict__ p)
    {
#pragma unroll
        for (int i = 0; i < N; i++) {
            const uint4 v = reinterpret_cast<const uint4 *>(p)[i];
            q[4 * i] = v.x; q[4 * i + 1] = v.y; q[4 * i + 2] = v.z; q[4 * i + 3] = v.w;
        }
    }
    __device__ void get(float (&w)[D]) const
    {
        if constexpr (sizeof(TIn) == 4) {
#pragma unroll
            for (int i = 0; i < D; i++) w[i] = __uint_as_float(q[i]);
        } else {
#pragma unroll
            for (int i = 0; i < D; i += 2) {
                w[i] = __uint_as_float(q[i / 2] << 16);
                w[i + 1] = __uint_as_float(q[i / 2] & 0xFFFF0000u);
            }
        }
    }
};

// The point of Sec. 2.5: |w| K / ||w||_1, rounded, and pulses moved at the largest deviations.  Signed point in y (zeros of
// either sign); a group without a direction gets zeros (its point is (0, ..., 0, K)).
template <int D>
__device__ inline void project_group(const float (&w)[D], float K, float &ss_out, bool &ordinary, bool &degenerate, float (&y)[D])
{
    float tmp[D];
#pragma unroll
    for (int i = 0; i < D; i++) tmp[i] = fabsf(w[i]);
    const float l1 = tree_sum<D>(tmp);
#pragma unroll
    for (int i = 0; i < D; i++) tmp[i] = w[i] * w[i];
    ss_out = tree_sum<D>(tmp);

    const float g = K / l1;
    float t[D], pulses = K;
#pragma unroll
    for (int i = 0; i < D; i++) t[i] = w[i] * g;
    degenerate = false;
    ordinary = __all(ordinary_norm(l1));
    if (!ordinary) {
        degenerate = !(l1 > 0.0f) || !(l1 < INFINITY) || !(g < INFINITY);
        pulses = degenerate ? 0.0f : K;
#pragma unroll
        for (int i = 0; i < D; i++) t[i] = degenerate ? 0.0f : t[i];
    }
#pragma unroll
    for (int i = 0; i < D; i++) { y[i] = rintf(t[i]); tmp[i] = fabsf(y[i]); }
    // pulses to add (> 0) or to take away (< 0)   (small integers: exact in any order)
    const float m = pulses - tree_sum<D>(tmp);
    const float unit = m < 0.0f ? -1.0f : 1.0f;
    // places in the order of deviations (negated where pulses have to go)
    constexpr int kLog2D = D == 8 ? 3 : D == 16 ? 4 : 5;
    const float order = m < 0.0f ? -order_scale<kLog2D>() : order_scale<kLog2D>();
    uint32_t key[D];
#pragma unroll
    for (int i = 0; i < D; i++) key[i] = order_of<kLog2D>(fabsf(t[i]) - fabsf(y[i]), order, i);
    adjust_first_places<D>(key, fabsf(m), unit, y);
}

// The index of the point.  table: LDS address of the thresholds, last: N(D,K) - 1.
template <int D, int W>
__device__ inline typename wide<W>::type rank_point(const float (&y)[D], bool degenerate, float K,
                                                    uint32_t table, typename wide<W>::type last)
{
    using T = typename wide<W>::type;
    constexpr int kStep = (D - 1) * W * 4;       // bytes between a coordinate's thresholds
    T c = last;
    float at = __builtin_fmaf(K, bytes(2 * kStep), __uint_as_float(table));
#pragma unroll
    for (int i = 0; i < D - 1; i++) {
        at = __builtin_fmaf(fabsf(y[i]), -bytes(2 * kStep), at);
        const float positive = __builtin_amdgcn_fmed3f(y[i], 0.0f, 1.0f);
        const uint32_t address = __float_as_uint(__builtin_fmaf(positive, bytes(kStep), at));
        c -= *reinterpret_cast<const __attribute__((address_space(3))) T *>(address + i * W * 4);
    }
    c -= y[D - 1] > 0.0f || degenerate ? 1 : 0;
    return c;
}

// Least-squares amplitude (Sec. 3.3 Step 4) for the point y: (y . w) / ||y||_2, products rounded one by one and summed over
// adjacent pairs, level by level.
template <int D>
__device__ inline float ls_amplitude(const float (&w)[D], const float (&y)[D], bool ordinary, bool degenerate, float K)
{
    float p[D], n[D];
#pragma unroll
    for (int i = 0; i < D; i++) {
        p[i] = y[i] * w[i];
        n[i] = y[i] * y[i];                   // small integers
    }
    if (!ordinary) {
        // zeros of the point are positive (the sign of a sum of zeros is theirs)
#pragma unroll
        for (int i = 0; i < D; i++) p[i] = degenerate ? (i < D - 1 ? 0.0f : K) * w[i] : p[i];
        n[D - 1] = degenerate ? K * K : n[D - 1];
    }
    return over_root(tree_sum<D>(p), tree_sum<D>(n), ordinary);
}

// OR a `bits`-wide value into a wave's words at bit 32 * (word of `at`) + sh (one word behind it too, with nothing)
template <int W>
__device__ inline void stage_field(uint32_t *at, uint32_t sh, typename wide<W>::type v)
{
    atomicOr(at, (uint32_t)v << sh);
#pragma unroll
    for (int i = 1; i <= W; i++) {
        const uint64_t two = (uint64_t)(uint32_t)(v >> (32 * (i - 1))) | (i < W ? (uint64_t)(uint32_t)(v >> (32 * (i % W))) << 32 : 0);
        atomicOr(at + i, (uint32_t)(two >> (32 - sh)));
    }
}

// LS: least-squares amplitudes (Sec. 3.3 Step 4) instead of norms.
template <int D, int W, typename TIn, bool LS>
__global__ __launch_bounds__(kMaxLanes, waves_per_simd(D)) void encode_kernel(encode_launch f, pvq_encode_args a)
{
    using T = typename wide<W>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lanes = blockDim.x, b = f.index_bits, sb = f.scale_bits;
    const int G = (int)a.groups;
    const float K = (float)f.K;
    const encode_lds l = lds_of(D, W, f, G, lanes);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = f.team / kWave, team = wave / waves, first = wave % waves;     // waves of a team, and the wave's place there
    const int teams = lanes / f.team;

    float4 *tree = reinterpret_cast<float4 *>(smem + l.tree);
    uint32_t *stage = reinterpret_cast<uint32_t *>(smem + l.stage) + wave * l.stage_words;
    float *sums = reinterpret_cast<float *>(smem + l.sums) + team * 2 * l.sum_words;
    float *ss_row = reinterpret_cast<float *>(smem + l.rows) + team * l.row_words;
    const uint32_t table = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char *)smem);

    const int tiles = (G + kWave - 1) / kWave;
    const TIn *source = reinterpret_cast<const TIn *>(a.W);
    // (a lane past the row's end takes the last group again, and writes nothing)
    auto group_at = [&](int64_t row, int t) { return source + row * a.ldw + (int64_t)min(t * kWave + lane, G - 1) * D; };
    const int64_t step = (int64_t)gridDim.x * f.working;
    int64_t row = team < f.working ? (int64_t)blockIdx.x * f.working + team : (int64_t)1 << 40;      // (no row has that number)

    // groups of 32 are loaded where they are used: there are no registers for a second one (16-bit weights, 96-bit indices,
    // 8192 x 8192: 105 us with one, 88)
    constexpr bool kAhead = D < 32;
    raw_group<D, TIn> next;
    if (kAhead && first < tiles) next.load(group_at(min(row, a.rows - 1), first));

    // thresholds from the size table, whose rows are shifted by one entry so that U(-1) is stored; neighbouring lanes read
    // neighbouring entries of a row (64 x 512, D = 8, K = 127: 4.2 us, an entry of another row to every lane 5.0)
    const T *tab_u = reinterpret_cast<const T *>(f.tab_u);
    const uint32_t per = (uint32_t)f.K + 1;
#pragma unroll 1
    for (uint32_t e = (uint32_t)tid; e < per * (D - 1); e += (uint32_t)lanes) {
        const uint32_t i = e / per, C = e % per;
        const T *u = tab_u + (D - 1 - i) * (per + 1) + C;                  // u[0] = U(D-1-i, C-1)
        const T u0 = u[0], u1 = u[1];
        T *t = reinterpret_cast<T *>(smem) + 2 * C * (D - 1) + i;
        t[0] = u0 + u0;
        t[D - 1] = u0 + u1;
    }
    if (sb > 0) fill_edge_tree(tree, f.edges, sb, tid, lanes);
    for (int i = tid; i < (int)(lanes / kWave * l.stage_words); i += lanes) reinterpret_cast<uint32_t *>(smem + l.stage)[i] = 0;
    for (int i = tid; i < (int)(2 * teams * l.sum_words); i += lanes) reinterpret_cast<float *>(smem + l.sums)[i] = 0.0f;
    __syncthreads();
    // U(D-1,K) + U(D-1,K-1) = N(D,K)
    const T last = reinterpret_cast<const T *>(smem)[(2 * f.K + 1) * (D - 1)] - 1;

    const uint32_t sh = (uint32_t)(lane * b) & 31;
    uint32_t *const at = stage + ((uint32_t)(lane * b) >> 5);
    uint32_t turn = 0;
    for (int64_t base = (int64_t)blockIdx.x * f.working; base < a.rows; base += step, row += step) {
        const bool live = row < a.rows;          // (a team without a row waits at the barrier)
        for (int t = first; live && t < tiles; t += waves) {
            const int g = t * kWave + lane;
            const bool in = g < G;
            float w[D], y[D], ss;
            if constexpr (!kAhead) next.load(group_at(row, t));
            next.get(w);
            if constexpr (kAhead) {
                // the tile behind, or the next row's first (of the last row once more)
                const bool more = t + waves < tiles;
                next.load(group_at(more ? row : min(row + step, a.rows - 1), more ? t + waves : first));
            }
            bool ordinary, degenerate;
            project_group<D>(w, K, ss, ordinary, degenerate, y);
            const T c = rank_point<D, W>(y, degenerate, K, table, last);
            stage_field<W>(at, sh, in ? c : 0);
            // the amplitude: the norm, or the least-squares one, whose square then stands for
            // the sum of squares in the codes (Sec. 3.3 Steps 4 and 5)
            float amp;
            if constexpr (LS) { amp = ls_amplitude<D>(w, y, ordinary, degenerate, K); ss = amp * amp; }
            else amp = root_of_squares(ss, ordinary);
            if (in) {
                if (sb > 0) ss_row[g] = ss;
                else reinterpret_cast<float *>(a.scale_out)[row * G + g] = amp;
            }
            if (a.pulses_out && in) {
                int8_t *p = a.pulses_out + row * a.cols + (int64_t)g * D;
                if (degenerate) y[D - 1] = K;
#pragma unroll
                for (int i = 0; i < D; i += 8) {
                    uint32_t lo = 0, hi = 0;
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        lo |= ((uint32_t)(int)y[i + j] & 0xFFu) << (8 * j);
                        hi |= ((uint32_t)(int)y[i + 4 + j] & 0xFFu) << (8 * j);
                    }
                    *reinterpret_cast<uint2 *>(p + i) = make_uint2(lo, hi);
                }
            }
            if (sb > 0) {
                // pairwise sum over the wave's 64 groups (absent groups add +0.0, which is exact)
                const float v = wave_pair_sum(in ? ss : 0.0f);
                if (lane == kWave - 1) sums[turn + t] = v;
            }
            // the tile's words, cleared for the next (a wave's LDS instructions are carried out in order)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint32_t *irow = a.index_out + row * a.index_row_words + (int64_t)t * 2 * b;
            const int nw = (int)min((int64_t)2 * b, a.index_row_words - (int64_t)t * 2 * b);
            for (int i = lane; i < nw; i += kWave) {
                irow[i] = stage[i];
                stage[i] = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        // Row normaliser (code mode only): sum of the groups' sums of squares, adjacent pairs
        // level by level, an odd last element moving up unchanged (as if zeros followed).
        if (sb > 0) {
            __syncthreads();
            if (live) {
                float part[4];                       // of 4096 groups each (rows of more than 16384 do not fit)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    part[i] = 0.0f;
                    if (i * kWave < tiles)
                        part[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_pair_sum(sums[turn + i * kWave + lane])), kWave - 1));
                }
                const float rowss = (part[0] + part[1]) + (part[2] + part[3]);
                if (first == 0 && lane == 0) a.rownorm_out[row] = rowss;
                write_codes<1>(sb, ss_row, rowss, tree, reinterpret_cast<uint32_t *>(a.scale_out) + row * a.scale_row_words, G,
                            first, waves, lane);
            }
            turn = l.sum_words - turn;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------

constexpr size_t kMaxLds = 64 * 1024;

// What a row may take: a size table, index words of 256 groups, and with amplitude codes the row's sums of squares and what
// their sum takes level by level.  (A row within it has at most 9362 groups, and encode_kernel's LDS is less than
// 136 KB with one team of 256 lanes: twice the size table, the rest below the 8 KB of the two largest index widths.)
size_t encode_row_bytes(const pvq_ctx *c, size_t G)
{
    size_t lds = (size_t)c->D * (c->K + 2) * c->words * 4 + (size_t)8 * c->index_bits * 4 + 64 * 4 + 256 * 4;
    if (c->scale_bits > 0) lds += (G + (G + 1) / 2 + (G + 3) / 4 + 4) * 4;
    return lds;
}

template <int D, int W, typename TIn, bool LS>
hipError_t launch_encode_kernel(const pvq_ctx *c, const pvq_encode_args &a, hipStream_t s)
{
    encode_launch f;
    f.tab_u = c->tab_u; f.edges = c->edges;
    f.K = c->K; f.index_bits = c->index_bits; f.scale_bits = c->scale_bits;
    f.team = a.groups <= kWave ? kWave : a.groups <= 2 * kWave ? 2 * kWave : 4 * kWave;
    // Lanes of a workgroup: the fewest with which the most waves fit a unit's LDS beside one another.
    constexpr int kWavesMost = 4 * waves_per_simd(D);
    int lanes = 0, waves = 0;
    for (int n = 256; n <= kMaxLanes; n *= 2) {
        const uint32_t lds = (lds_of(D, W, f, (int)a.groups, n).total + 1279) / 1280 * 1280;
        const int fit = std::min<int>(160 * 1024 / lds * (n / kWave), kWavesMost / (n / kWave) * (n / kWave));
        if (fit > waves) { waves = fit; lanes = n; }
    }
    if (lanes == 0) return hipErrorInvalidValue;      // (the caller has asked pvq_encode_fits)
    const uint32_t lds = lds_of(D, W, f, (int)a.groups, lanes).total;
    const auto kernel = &encode_kernel<D, W, TIn, LS>;
    if (lds > kMaxLds) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // Neighbouring rows go to the teams of a workgroup (28672 x 512, D = 16, K = 5: 35 us, rows a grid apart 38), but few rows
    // go to as many units as there are (256 x 4096, D = 32, K = 105: 11.4 us, to the teams of as few as hold them 15.5).
    f.working = (int)std::min<int64_t>(lanes / f.team, (a.rows + 255) / 256);
    const unsigned grid = (unsigned)std::min<int64_t>((a.rows + f.working - 1) / f.working, 256 * (waves / (lanes / kWave)));
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(lanes), lds, s, f, a);
    return hipGetLastError();
}

template <int D, int W>
hipError_t launch_encode_dw(const pvq_ctx *c, const pvq_encode_args &a, int dtype, hipStream_t s)
{
    if (a.ls_amplitude)
        return dtype == PVQ_F32 ? launch_encode_kernel<D, W, float, true>(c, a, s) : launch_encode_kernel<D, W, uint16_t, true>(c, a, s);
    return dtype == PVQ_F32 ? launch_encode_kernel<D, W, float, false>(c, a, s) : launch_encode_kernel<D, W, uint16_t, false>(c, a, s);
}

}  // namespace

bool pvq_encode_fits(const pvq_ctx *c, const pvq_encode_args &a) { return encode_row_bytes(c, (size_t)a.groups) <= kMaxLds; }

hipError_t pvq_launch_encode(const pvq_ctx *c, const pvq_encode_args &a, int dtype, hipStream_t s)
{
    if (c->D == 8) {
        if (c->words == 1) return launch_encode_dw<8, 1>(c, a, dtype, s);
        return launch_encode_dw<8, 2>(c, a, dtype, s);
    }
    if (c->D == 16) {
        if (c->words == 1) return launch_encode_dw<16, 1>(c, a, dtype, s);
        if (c->words == 2) return launch_encode_dw<16, 2>(c, a, dtype, s);
        return launch_encode_dw<16, 4>(c, a, dtype, s);
    }
    if (c->words == 1) return launch_encode_dw<32, 1>(c, a, dtype, s);
    if (c->words == 2) return launch_encode_dw<32, 2>(c, a, dtype, s);
    return launch_encode_dw<32, 4>(c, a, dtype, s);
}

// ---------------------------------------------------------------------------------------------
// y = 0 for a product over zero columns (a kernel rather than a memset, so that a caller may
// capture the call into a graph)
// ---------------------------------------------------------------------------------------------

namespace {
__global__ void fill_zero_kernel(float *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}
}  // namespace

hipError_t pvq_launch_fill_zero(float *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}
