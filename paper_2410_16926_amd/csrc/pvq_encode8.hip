// Encoder specialised for D = 8 with 24-bit indices (the 3 bits/weight setting).
//
// Same arithmetic, in the same order, as the generic encoder (pvq_kernels.hip) — results are bit for
// bit the same — but organised for throughput, which vector instructions bound:
//   * one lane per group, workgroups of 256 lanes that take whole rows, 256 groups at a time, as many workgroups as
//     the machine holds at once; the next tile's weights are on their way while one is worked on;
//   * the pulse-count repair (Sec. 2.5) adjusts the coordinates that hold the |sum - K| first places in the
//     order of deviations, which a network of three-operand minima, medians and maxima finds (adjust_first_places8).  This
//     equals the one-at-a-time repair because no coordinate is ever adjusted twice (for finite input the
//     |sum - K| largest deviations are all positive, an adjusted coordinate drops below -1/2);
//   * the index (App. B.2) is a sum of seven table entries, one per coordinate, from a table of per-coordinate offsets
//     indexed by (coordinate, pulses left, signed value), whose addresses come out of one multiply-add each
//     (encode_group8);
//   * four neighbouring lanes assemble their 24-bit indices into three dwords with DPP moves and write
//     them straight to global memory; amplitude codes are OR-reduced across lanes the same way;
//   * the row normaliser's pairwise sum is a wave butterfly followed by a small tree over wave sums
//     (adding +0.0 for absent groups is exact, so padding a row to a power of two does not change
//     the pair-level sum);
//   * an amplitude code takes one 16-byte read for two of its bits, and a lane makes those of up to four groups (write_codes).
// Bound by instructions, whichever unit they go to: 8 waves a SIMD issue one in about 2.7 clocks.  (Alone, with 8 waves a SIMD,
// additions, multiplications, float32 multiply-adds and exclusive ors take 2.6 clocks a wave, comparisons, shifts, minima and
// maxima, conversions, byte permutations and lane moves 4.3 to 4.8, v_rcp 8.9.)  28672 x 8192 bf16 weights, 2-bit codes: 234 vector,
// 46 scalar and 10 LDS instructions a group, 152 us (launches in a row); with the places of the repair marked by masks on the
// scalar unit, a code a lane and general quotients 242, 129 and 11, 185 us; with integer addresses, marks of all rounds as masks
// and a bisection for the code 284 vector ones and 211 us.  With clamped differences for comparisons in the repair and short quotients for
// the codes, another 6 %: 160 / 151 us on one card, 14336 x 4096 with 8-bit codes 48.1 / 45.3 (before that 55 and 81).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "pvq_hadamard_dev.h"
#include "pvq_internal.h"
#include "pvq_quantize_dev.h"

namespace {

using namespace pvq_quantize_dev;

constexpr int D = 8;

// The offset table in LDS: [7][kMaxK + 1][2 kMaxK + 1] words (coordinate, pulses left, value + kMaxK), whatever K is
// (15 or 16 with 24-bit indices), so that the rows' distances are known here.
constexpr int kMaxK = PVQ_ENC8_MAX_K;
constexpr int kStepValue = 4, kStepPulse = 4 * (2 * kMaxK + 1), kStepCoordinate = kStepPulse * (kMaxK + 1);   // bytes
constexpr int kTableWords = (PVQ_ENC8_WORDS + 3) & ~3;

struct enc8_launch {
    const uint32_t *offs;
    const float *edges;     // 2^scale_bits entries, last = +inf (or nullptr)
    int K, scale_bits;
};

// Sum over adjacent pairs, level by level (fixed order, float32).
__device__ inline float tree8(float (&v)[D])
{
#pragma unroll
    for (int s = 1; s < D; s *= 2)
#pragma unroll
        for (int i = 0; i < D; i += 2 * s) v[i] = v[i] + v[i + s];
    return v[0];
}

// A group as it comes from memory: 8 float32 or bf16 values.
template <typename TIn> struct raw8;
template <> struct raw8<float> {
    float4 q0, q1;
    __device__ void load(const float *__restrict__ p)
    {
        q0 = *reinterpret_cast<const float4 *>(p); q1 = *reinterpret_cast<const float4 *>(p + 4);
    }
    __device__ void flip(uint2 bits)
    {
        float *v[D] = {&q0.x, &q0.y, &q0.z, &q0.w, &q1.x, &q1.y, &q1.z, &q1.w};
#pragma unroll
        for (int j = 0; j < D; j++) *v[j] = pvq_hadamard_dev::with_sign(*v[j], bits, j);
    }
    __device__ void get(float (&w)[D]) const
    {
        w[0] = q0.x; w[1] = q0.y; w[2] = q0.z; w[3] = q0.w; w[4] = q1.x; w[5] = q1.y; w[6] = q1.z; w[7] = q1.w;
    }
};
template <> struct raw8<uint16_t> {
    uint4 q;
    __device__ void load(const uint16_t *__restrict__ p) { q = *reinterpret_cast<const uint4 *>(p); }
    __device__ void flip(uint2 bits)
    {
        q.x = pvq_hadamard_dev::with_signs(q.x, bits, 0); q.y = pvq_hadamard_dev::with_signs(q.y, bits, 1);
        q.z = pvq_hadamard_dev::with_signs(q.z, bits, 2); q.w = pvq_hadamard_dev::with_signs(q.w, bits, 3);
    }
    __device__ void get(float (&w)[D]) const
    {
        const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            w[2 * j] = __uint_as_float(u[j] << 16);
            w[2 * j + 1] = __uint_as_float(u[j] & 0xFFFF0000u);
        }
    }
};

// One group: returns its 24-bit index, the sum of squares, and the signed point in y (float, zeros of either sign).
// table: LDS address of offs[0][0][0].  POINT: y of a group without a direction is set too (else its y is unspecified).
// ordinary: whether all groups of the wave have an ordinary norm.
template <bool POINT>
__device__ inline uint32_t encode_group8(const float (&w)[D], float K, uint32_t table, float &ss_out, bool &ordinary, bool &degenerate, float (&y)[D])
{
    float tmp[D];
#pragma unroll
    for (int i = 0; i < D; i++) tmp[i] = fabsf(w[i]);
    const float l1 = tree8(tmp);
#pragma unroll
    for (int i = 0; i < D; i++) tmp[i] = w[i] * w[i];
    ss_out = tree8(tmp);

    const float g = over_norm(K, l1, ordinary, degenerate);
    float t[D], mag[D], pulses = K;
#pragma unroll
    for (int i = 0; i < D; i++) t[i] = w[i] * g;
    // a group without a direction gets zeros, whose index comes out as that of (0, ..., 0, K): 0
    if (!ordinary) {
        pulses = degenerate ? 0.0f : K;
#pragma unroll
        for (int i = 0; i < D; i++) t[i] = degenerate ? 0.0f : t[i];
    }
    // from here on t is finite and within [-K(1+eps), K(1+eps)], so that the addresses below lie inside the table
    float S[D];
#pragma unroll
    for (int i = 0; i < D; i++) { mag[i] = rintf(fabsf(t[i])); S[i] = mag[i]; }
    // pulses to add (> 0) or to take away (< 0)   (small integers: exact in any order)
    const float m = pulses - tree8(S);
    const float unit = m < 0.0f ? -1.0f : 1.0f;
    // places in the order of deviations: how far a magnitude is below its projected value (above it where pulses have to go)
    const float order = m < 0.0f ? -order_scale<3>() : order_scale<3>();
    uint32_t key[D];
#pragma unroll
    for (int i = 0; i < D; i++) key[i] = order_of<3>(fabsf(t[i]) - mag[i], order, i);
    adjust_first_places8(key, fabsf(m), unit, mag);
    // (-0.0 never carries a pulse: a coordinate whose projection is zero is not among the ones raised)
#pragma unroll
    for (int i = 0; i < D; i++) y[i] = copysignf(mag[i], w[i]);
    // offs[i][k][y]: what coordinate i adds to the index with k pulses left (App. B.2); 0 for y = 0
    uint32_t part[D - 1];
    float at = __uint_as_float(table) + K * bytes(kStepPulse) + bytes(kMaxK * kStepValue);   // offs[0][K][0]
#pragma unroll
    for (int i = 0; i < D - 1; i++) {
        const uint32_t address = __float_as_uint(__builtin_fmaf(y[i], bytes(kStepValue), at));
        part[i] = *reinterpret_cast<const __attribute__((address_space(3))) uint32_t *>(address + i * kStepCoordinate);
        at = __builtin_fmaf(mag[i], -bytes(kStepPulse), at);
    }
    // the last coordinate takes what is left: +k is first, -k second
    uint32_t c = y[D - 1] < 0.0f ? 1u : 0u;
#pragma unroll
    for (int i = 0; i < D - 1; i++) c += part[i];
    if constexpr (POINT) {
        if (degenerate) y[D - 1] = K;
    }
    return c;
}

// Least-squares amplitude (Sec. 3.3 Step 4) for the point in y: (y . w) / ||y||_2, products rounded one by one and summed over
// adjacent pairs, level by level.
__device__ inline float ls_amplitude8(const float (&w)[D], const float (&y)[D], bool ordinary, bool degenerate)
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
        for (int i = 0; i < D - 1; i++) p[i] = degenerate ? 0.0f * w[i] : p[i];
    }
    return over_root(tree8(p), tree8(n), ordinary);
}

// four neighbouring 24-bit indices -> three dwords: lane j of a quad (j < 3) builds dword j from its own index and the
// next lane's
__device__ inline uint32_t index_word(uint32_t c, int quad_pos)
{
    const uint32_t cn = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xF9, 0xF, 0xF, false);
    const uint32_t lo = c | (cn << 24), hi = cn >> 8;
    return __builtin_amdgcn_alignbit(hi, lo, 8 * quad_pos);
}

// The row's sum of squares from its wave sums (at most 64, zero padded; the pairwise tree goes on), in a scalar register.
__device__ inline float row_sum(const float *wsum, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_pair_sum(wsum[lane])), kWave - 1));
}

// v as a number that the compiler does not know: what is computed from it is computed where it is used and not kept over the loops
// in front.  The kernels have 64 registers for eight waves a SIMD, and what is only looked at once a row or a chunk (a lane's groups
// when it writes codes, its pointers into weights and signs) had 2 to 10 values of the rotating kernels for 16-bit sources, and
// 2 to 4 of the encoder for float32 sources, in scratch memory: 1500 x 6144 bf16 in blocks of 2048, 2-bit codes, 17.1 us, now 15.2;
// 14336 x 4096 float32, 2-bit codes, 47.6, now 44.4.  (Kernels that have registers for it keep it: the encoder of bf16, 8-bit
// codes, 47.0, with it 47.5.)
template <typename T>
__device__ inline T anew(T v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// LDS of both kernels, from byte 0: the offset table, the edges' tree, two rows' wave sums (used in turn, so that one
// barrier a row is enough), the row's sums of squares (CODES; every wave reads its own).
struct enc8_lds {
    float4 *tree;
    float *wsum, *ss_row;
    uint32_t table;
};
template <int CODES>
__device__ inline enc8_lds fill_lds(uint32_t *smem, const enc8_launch &f, int lanes)
{
    enc8_lds l;
    l.tree = reinterpret_cast<float4 *>(smem + kTableWords);
    l.wsum = reinterpret_cast<float *>(l.tree + kEdgeNodes);
    l.ss_row = l.wsum + 2 * 64;
    l.table = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t *)smem);
    for (int i = threadIdx.x; i < kTableWords / 4; i += lanes) reinterpret_cast<uint4 *>(smem)[i] = reinterpret_cast<const uint4 *>(f.offs)[i];
    if constexpr (CODES) fill_edge_tree(l.tree, f.edges, f.scale_bits, threadIdx.x, lanes);
    for (int i = threadIdx.x; i < 2 * 64; i += lanes) l.wsum[i] = 0.0f;
    return l;
}
// its words in front of the row's sums of squares
constexpr int kHeadWords = kTableWords + 4 * kEdgeNodes + 2 * 64;

// TIn: float or uint16_t (bf16 bits).  A block of kBlock lanes takes whole rows, kBlock groups at a
// time; several blocks share a compute unit, so one block's barriers hide behind the others' arithmetic.
constexpr int kBlock = 256;
constexpr int kMaxGroups = 4096;   // groups per row this kernel takes (their sums of squares sit in LDS)

// CODES: 0 for float32 amplitudes, else the groups that a lane takes when it writes amplitude codes (write_codes).
// LS: least-squares amplitudes (Sec. 3.3 Step 4) instead of norms.
template <typename TIn, int CODES, bool LS>
__global__ __launch_bounds__(kBlock, 8) void encode8_kernel(enc8_launch f, pvq_encode_args a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const int sb = f.scale_bits;
    const float K = (float)f.K;
    const enc8_lds l = fill_lds<CODES>(smem, f, kBlock);

    const int G = (int)a.groups;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int quad_pos = lane & 3;
    // tiles of a row in which the wave has groups
    const int tiles = (G - wave * kWave + kBlock - 1) / kBlock;
    const TIn *W = reinterpret_cast<const TIn *>(a.W);
    // (a lane past the row's end takes the last group again, and writes nothing)
    auto source = [&](int64_t row, int tix) { return W + row * a.ldw + (int64_t)min(tix * kBlock + (int)threadIdx.x, G - 1) * D; };

    raw8<TIn> next;
    if (tiles > 0) next.load(source(blockIdx.x, 0));
    __syncthreads();
    float *wsum = l.wsum;
    for (int64_t row = blockIdx.x; row < a.rows; row += gridDim.x) {
        uint32_t *irow = a.index_out + row * a.index_row_words;
        for (int tix = 0; tix < tiles; tix++) {
            const int g = tix * kBlock + (int)threadIdx.x;
            const bool in = g < G;
            float w[D], y[D], ss;
            next.get(w);
            // the tile behind, or the next row's first (of the last row once more)
            const bool more = tix + 1 < tiles;
            next.load(source(more ? row : min(row + (int64_t)gridDim.x, a.rows - 1), more ? tix + 1 : 0));
            bool ordinary, degenerate;
            const uint32_t c = encode_group8<LS>(w, K, l.table, ss, ordinary, degenerate, y);
            float amp;
            if constexpr (LS) { amp = ls_amplitude8(w, y, ordinary, degenerate); ss = amp * amp; }
            else amp = root_of_squares(ss, ordinary);
            if (a.pulses_out && in) {
                if (degenerate) y[D - 1] = K;
                uint32_t lo = 0, hi = 0;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    lo |= ((uint32_t)(int)y[j] & 0xFFu) << (8 * j);
                    hi |= ((uint32_t)(int)y[4 + j] & 0xFFu) << (8 * j);
                }
                *reinterpret_cast<uint2 *>(a.pulses_out + row * a.cols + (int64_t)g * D) = make_uint2(lo, hi);
            }
            if (in) {
                if constexpr (CODES) l.ss_row[g] = ss;
                else reinterpret_cast<float *>(a.scale_out)[row * G + g] = amp;
            }
            const uint32_t word = index_word(c, quad_pos);
            if (quad_pos < 3 && in) irow[3 * (g >> 2) + quad_pos] = word;
            if constexpr (CODES) {
                // pairwise sum over the wave's 64 groups (absent groups add +0.0, which is exact)
                const float v = wave_pair_sum(in ? ss : 0.0f);
                if (lane == kWave - 1) wsum[tix * (kBlock / kWave) + wave] = v;
            }
        }
        if constexpr (CODES) {
            __syncthreads();
            const float rowss = row_sum(wsum, lane);
            if (threadIdx.x == 0) a.rownorm_out[row] = rowss;
            write_codes<CODES>(sb, l.ss_row, rowss, l.tree, reinterpret_cast<uint32_t *>(a.scale_out) + row * a.scale_row_words, G, wave, kBlock / kWave,
                               sizeof(TIn) == 4 ? anew(lane) : lane);
            wsum = wsum == l.wsum ? l.wsum + 64 : l.wsum;
        }
    }
}

// Rotation of the rows (Sec. 3.3 Step 1) and encoding of the rotated values in one kernel: the transform's
// stages (pvq_hadamard_dev.h) end with 8 consecutive rotated values per lane, which is one group, so the
// lane goes straight on into the encoder above and the rotated matrix is never written.  A workgroup of L
// lanes takes whole rows, a chunk of 8 L values (whole blocks of the rotation) at a time; everything
// after the rotation is encode8_kernel's (its lanes are groups in row order here too, so the row sum's
// pair levels, the quads that assemble index words and the code words come out the same).  The rotated
// values are float32 (scaled by float32(1 / sqrt(block))), exactly those of the rotation kernel with a
// float32 result.  LOG2N as in pvq_hadamard.hip: 9 for blocks of up to 512 values, 10 .. 13 for that block.
template <typename TIn, int CODES, bool LS, int LOG2N>
__device__ inline void rotate_encode8_body(const enc8_launch &f, const pvq_encode_args &a, int log2n,
                                           const uint8_t *signs, float scale)
{
    using namespace pvq_hadamard_dev;
    extern __shared__ __align__(16) uint32_t smem[];
    const int sb = f.scale_bits;
    const float K = (float)f.K;
    const int L = blockDim.x;
    const int G = (int)a.groups;
    const enc8_lds l = fill_lds<CODES>(smem, f, L);
    float *hbuf = l.ss_row + (CODES ? ((G + 3) & ~3) : 0);       // the rotation's exchange buffer
    __syncthreads();

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quad_pos = lane & 3;
    const int chunks = G / L;                                    // whole chunks: every lane has a group
    const uint32_t from = (uint32_t)(load_lane<LOG2N>(tid) * D); // the 8 values of a chunk that the lane loads
    const int waves = L / kWave;

    float *wsum = l.wsum;
    for (int64_t row = blockIdx.x; row < a.rows; row += gridDim.x) {
        const TIn *xrow = reinterpret_cast<const TIn *>(a.W) + row * a.ldw;
        uint32_t *irow = a.index_out + row * a.index_row_words;
        for (int ch = 0; ch < chunks; ch++) {
            const int g = ch * L + (CODES ? anew(tid) : tid);
            float v[D];
            raw8<TIn> raw;
            const uint32_t at = anew(from);                      // (an offset from a scalar address, not a pointer that moves with the chunks)
            raw.load(xrow + (int64_t)(ch * L) * D + at);
            if (signs) raw.flip(sign_bits(*reinterpret_cast<const uint2 *>(signs + (int64_t)(ch * L) * D + at)));
            raw.get(v);
            // (two workgroups of 1024 lanes fit a unit's LDS; the cross-lane stages from 4 lanes on go through the LDS permute unit for blocks of up to 512 values, where the
            // encoder's arithmetic is what the kernel waits for and that unit is idle; none for larger blocks, whose
            // exchanges through LDS need it)
            constexpr int kPermuted = LOG2N <= 9 ? 4 + 8 + 16 + 32 : 0;
            int stages = log2n;
            if constexpr (LOG2N <= 9) asm volatile("" : "+s"(stages));   // (else the comparisons below stay in scalar registers over the loop)
            hadamard_stages<LOG2N, false, kPermuted>(v, tid, stages, hbuf);
            float w[D], y[D], ss;
#pragma unroll
            for (int j = 0; j < D; j++) w[j] = v[j] * scale;
            bool ordinary, degenerate;
            const uint32_t c = encode_group8<LS>(w, K, l.table, ss, ordinary, degenerate, y);
            float amp;
            if constexpr (LS) { amp = ls_amplitude8(w, y, ordinary, degenerate); ss = amp * amp; }
            else amp = root_of_squares(ss, ordinary);
            if constexpr (CODES) l.ss_row[g] = ss;
            else reinterpret_cast<float *>(a.scale_out)[row * G + g] = amp;
            const uint32_t word = index_word(c, quad_pos);
            if (quad_pos < 3) irow[3 * (g >> 2) + quad_pos] = word;
            if constexpr (CODES) {
                const float s64 = wave_pair_sum(ss);
                if (anew(lane) == kWave - 1) wsum[ch * waves + wave] = s64;
            }
        }
        if constexpr (CODES) {
            __syncthreads();
            const float rowss = row_sum(wsum, anew(lane));
            if (anew(tid) == 0) a.rownorm_out[row] = rowss;
            write_codes<CODES>(sb, l.ss_row, rowss, l.tree, reinterpret_cast<uint32_t *>(a.scale_out) + row * a.scale_row_words, G, wave, waves, anew(lane));
            wsum = wsum == l.wsum ? l.wsum + 64 : l.wsum;
        }
    }
}

// Registers for eight waves a SIMD (64 a lane).  8192 x 8192 bf16, 2-bit codes, blocks of 4096: 79 us, calls in a row (with two barriers an
// exchange, selections in the stages across lanes and divisions for the codes 83); 4000 x 6144 in blocks of 64 28.6.
template <typename TIn, int CODES, bool LS, int LOG2N>
__global__ __launch_bounds__(512, 8) void rotate_encode8_kernel(enc8_launch f, pvq_encode_args a, int log2n,
                                                            const uint8_t *signs, float scale)
{
    rotate_encode8_body<TIn, CODES, LS, LOG2N>(f, a, log2n, signs, scale);
}

// (float32 rows of several blocks: the others have the kernel below)
template <int CODES, bool LS>
__global__ __launch_bounds__(1024, 8) void rotate_encode8_kernel_8192(enc8_launch f, pvq_encode_args a, int log2n,
                                                                      const uint8_t *signs, float scale)
{
    rotate_encode8_body<float, CODES, LS, 13>(f, a, log2n, signs, scale);
}

// The same with sixteen values a lane, for blocks of 64 to 2048 and 8192: a wave holds 1024 values in a row, in two runs of 8 a lane, ten
// stages stay inside it, and what is left for larger blocks is one ownership: two trips through LDS where eight values a lane
// need three for blocks of 8192, and no barriers between waves for blocks of up to 1024.  The last trip ends in the wave's own 1024 values,
// which are 128 groups that it takes in two halves, from LDS.  A chunk is what the workgroup's waves hold (eight of them for blocks of more
// than 1024).
// What bounded blocks of 8192 were the barriers: the tables and the values leave room for two workgroups of 1024 lanes on a unit, so that
// either waits for the other, and a row's end (its sum, its codes, the next row's first values) cost 27 of 99 us.  Now there are three
// workgroups, one barrier fewer a chunk, and 80 registers a lane (six waves a SIMD), in which the next values are on their way while
// groups are encoded.  8192 x 8192 bf16: 2-bit codes 98.6 -> 80.4 us, float32 amplitudes 81.1 -> 70.8.  With few rows it is the
// chunks of a row that a workgroup takes one after the other, of 256 groups before and of up to 1024 now, and their memory's latency.
// CODED: 0 for float32 amplitudes, else the chunks that a row may have.  Their sums of squares stay in registers until the row's end and
// then take the place of values that the wave has read (with LDS of their own a third workgroup would not fit).
constexpr int kHalfBlockLanes = 512;
constexpr int kWaveWords = 1024 + 1024 / 32;                         // of the exchange buffer, padded
template <typename TIn, int CODED, bool LS, int LOG2N>
__global__ __launch_bounds__(kHalfBlockLanes, 6) void rotate_encode8_halves_kernel(enc8_launch f, pvq_encode_args a, const uint8_t *signs, float scale)
{
    using namespace pvq_hadamard_dev;
    extern __shared__ __align__(16) uint32_t smem[];
    const float K = (float)f.K;
    const int waves = LOG2N > 10 ? kHalfBlockLanes / kWave : blockDim.x / kWave;
    const enc8_lds l = fill_lds<CODED>(smem, f, waves * kWave);
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = (int)a.groups, chunks = CODED == 1 ? 1 : G / (2 * kWave * waves);
    const TIn *W = reinterpret_cast<const TIn *>(a.W);

    float *const own = l.ss_row + kWaveWords * wave;                 // the wave's values
    float *const across = l.ss_row + pad((uint32_t)tid);             // values 1024 apart, for the last three stages
    const float *const group = own + pad((uint32_t)(D * lane));

    raw8<TIn> raw[2];
    uint2 s8[2];
    constexpr bool kSignsAhead = sizeof(TIn) == 2 || CODED < 4;      // (else they have no registers)
    auto request_signs = [&](int ch) {
        if (!signs) return;
        const uint32_t from = (uint32_t)(1024 * wave + D * load_lane<13>(anew(lane)));
#pragma unroll
        for (int h = 0; h < 2; h++) s8[h] = *reinterpret_cast<const uint2 *>(signs + (int64_t)ch * (1024 * waves) + 512 * h + from);
    };
    auto request = [&](int64_t row, int ch) {
        const uint32_t from = (uint32_t)(1024 * wave + D * load_lane<13>(anew(lane)));
#pragma unroll
        for (int h = 0; h < 2; h++) raw[h].load(W + row * a.ldw + (int64_t)ch * (1024 * waves) + 512 * h + from);
        if constexpr (kSignsAhead) request_signs(ch);
    };
    request(blockIdx.x, 0);
    __syncthreads();
    float *wsum = l.wsum;
    float kept[CODED ? CODED : 1][2] = {};                                // sums of squares of the row's blocks
    for (int64_t row = blockIdx.x; row < a.rows; row += gridDim.x) {
        uint32_t *irow = a.index_out + row * a.index_row_words;
        for (int ch = 0; ch < chunks; ch++) {
            float v[2][D];
            const int at_lane = anew(lane), place = load_lane<13>(at_lane);
            if constexpr (!kSignsAhead) request_signs(ch);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                if (signs) raw[h].flip(sign_bits(s8[h]));
                raw[h].get(v[h]);
                stages_in_registers(v[h], 3);
                stage_across_lanes<1>(v[h], place);
                stage_across_lanes<2>(v[h], place);
                stage_across_lanes<4, false, true>(v[h], place);
                if constexpr (LOG2N > 6) stage_across_lanes<8>(v[h], place);
                if constexpr (LOG2N > 7) stage_across_rows<16, 4, true>(v[h]);
                if constexpr (LOG2N > 8) stage_across_rows<32, 2, true>(v[h]);
            }
            __builtin_amdgcn_wave_barrier();                         // (the wave has read what lay here)
            // (roles of register and lane bits as exchange_from_rows has them)
            constexpr bool k16 = LOG2N > 7, k32 = LOG2N > 8;
            float *const put = own + pad((uint32_t)((k32 ? at_lane >> 4 & 2 : at_lane << 3 & 256) | (k16 ? at_lane >> 2 & 4 : at_lane << 3 & 128) | (place & 15) << 3));
#pragma unroll
            for (int q = 0; q < D; q++) {
                const float x = v[0][q], y = v[1][q];
                const uint32_t at = pad((uint32_t)((q & 1) | (q & 4) << (k16 ? 5 : 0) | (q & 2) << (k32 ? 7 : 0)));
                put[at] = LOG2N > 9 ? x + y : x;
                put[at + pad(512)] = LOG2N > 9 ? x - y : y;
            }
            if constexpr (LOG2N > 10) {
                __syncthreads();
#pragma unroll
                for (int h = 0; h < 2; h++) {
#pragma unroll
                    for (int q = 0; q < D; q++) v[h][q] = across[pad(512) * h + kWaveWords * q];
                }
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    stages_in_registers(v[h], LOG2N - 10);
#pragma unroll
                    for (int q = 0; q < D; q++) across[pad(512) * h + kWaveWords * q] = v[h][q];
                }
                __syncthreads();
            } else {
                __builtin_amdgcn_wave_barrier();
            }
            // the block behind, or the next row's first (of the last row once more)
            const bool more = ch + 1 < chunks;
            request(more ? row : min(row + (int64_t)gridDim.x, a.rows - 1), more ? ch + 1 : 0);
            float ss_first = 0.0f, ss = 0.0f;
#pragma unroll 1
            for (int h = 0; h < 2; h++) {
                const int run = 2 * (waves * ch + wave) + h, g = run * kWave + lane;
                float w[D], y[D];
#pragma unroll
                for (int j = 0; j < D; j++) w[j] = group[pad(512) * h + j] * scale;
                bool ordinary, degenerate;
                ss_first = ss;
                const uint32_t c = encode_group8<LS>(w, K, l.table, ss, ordinary, degenerate, y);
                float amp;
                if constexpr (LS) { amp = ls_amplitude8(w, y, ordinary, degenerate); ss = amp * amp; }
                else amp = root_of_squares(ss, ordinary);
                if constexpr (!CODED) reinterpret_cast<float *>(a.scale_out)[row * G + g] = amp;
                const uint32_t word = index_word(c, lane & 3);
                if ((lane & 3) < 3) irow[3 * (g >> 2) + (lane & 3)] = word;
                if constexpr (CODED) {
                    const float s64 = wave_pair_sum(ss);
                    if (lane == kWave - 1) wsum[run] = s64;
                }
            }
            if constexpr (CODED) {
#pragma unroll
                for (int b = 0; b < CODED; b++) {
                    kept[b][0] = CODED == 1 || b == ch ? ss_first : kept[b][0];
                    kept[b][1] = CODED == 1 || b == ch ? ss : kept[b][1];
                }
            }
        }
        if constexpr (CODED) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int b = 0; b < CODED; b++) {
                own[2 * kWave * b + lane] = kept[b][0];
                own[2 * kWave * b + kWave + lane] = kept[b][1];
            }
            __syncthreads();
            const float rowss = row_sum(wsum, anew(lane));
            if (anew(tid) == 0) a.rownorm_out[row] = rowss;
#pragma unroll 1
            for (int ch = 0; ch < chunks; ch++) {
                const int run = 2 * (waves * ch + wave);                  // two runs of 64 groups
                write_codes<2>(f.scale_bits, own + 2 * kWave * ch - kWave * run, rowss, l.tree,
                               reinterpret_cast<uint32_t *>(a.scale_out) + row * a.scale_row_words, kWave * (run + 2), run, 1, anew(lane));
            }
            wsum = wsum == l.wsum ? l.wsum + 64 : l.wsum;
        }
    }
}

}  // namespace

// Workgroups of `lanes` lanes and `lds` bytes that the machine holds at once, up to 8 waves on a SIMD: they take the rows in
// turn, so that the tables are copied to LDS once per place and not once per row.
static unsigned resident_grid(int64_t rows, int lanes, size_t lds)
{
    const int64_t by_waves = 32 / (lanes / kWave), by_lds = (int64_t)(160 * 1024 / ((lds + 1279) / 1280 * 1280));
    return (unsigned)std::min<int64_t>(rows, 256 * std::max<int64_t>(1, std::min(by_waves, by_lds)));
}

// lanes of the fused kernel's workgroup for a rotation block: whole blocks, at least 256 lanes
static int rotate8_lanes(int block) { return std::min(1024, std::max(256, block / 8)); }

bool pvq_rotate_encode8_usable(const pvq_ctx *c, const pvq_encode_args &a, int block)
{
    // the encoder's own conditions, and rows of whole chunks (so that every lane of a workgroup has a group
    // in every chunk and the transform's barriers are reached by all)
    return pvq_encode8_usable(c, a) && a.pulses_out == nullptr && a.groups % rotate8_lanes(block) == 0;
}

hipError_t pvq_rotate_encode8_launch(const pvq_ctx *c, const pvq_encode_args &a, int dtype, int block,
                                     const uint8_t *signs, hipStream_t s)
{
    enc8_launch f;
    f.offs = c->enc8_offs; f.edges = c->edges; f.K = c->K; f.scale_bits = c->scale_bits;
    int log2n = 0;
    while ((1 << log2n) < block) log2n++;
    const int L = rotate8_lanes(block);
    const bool codes = c->scale_bits > 0, ls = a.ls_amplitude != 0;
    const float scale = (float)(1.0 / std::sqrt((double)block));
    // Sixteen values a lane (us, eight / sixteen, bf16 and 2-bit codes unless said).  A workgroup has as many waves, up to eight, as
    // divide the row's 1024s.
    //  - Where no workgroup has more than a row or two, for all blocks but of 4096: 64 x 8192 in blocks of 64 8.4 / 6.3, 64 x 28672 20.5 / 13.1,
    //    700 x 4096 in blocks of 256 8.0 / 7.0, 700 x 14336 float32 in blocks of 64 17.6 / 17.2, 768 x 16384 in blocks of 1024 21.1 / 17.4.
    //    (One or two waves, and rows of more than four chunks with codes, have the others.)  Not float32 rows of several blocks of 8192 with codes, whose
    //    signs are not on their way early: 768 x 16384 19.4 / 20.4, 1024 x 16384 26.5 / 24.4.
    //  - With more rows in whole chunks of 8192 values, of which three workgroups fit a unit (fewer waves: 4000 x 6144 in blocks of 64 28.6 / 33.2),
    //    768 rows at a time; with eight values a lane eight workgroups fit, 2048 rows.  Rows of one chunk, by their number:
    //                                        769         1100        1300        1536        2048        2304        3000        3500        4500        8192
    //      block 64, float32             11.6 / 10.8 14.9 / 13.8 16.3 / 17.6 17.1 / 17.9 19.8 / 21.2 21.4 / 23.8 26.5 / 29.4 32.3 / 32.3             75.7 / 80.9
    //            64                      10.7 / 10.1 13.0 / 11.9 14.6 / 15.0 15.5 / 15.4 19.0 / 19.2 20.5 / 22.2 24.8 / 27.8 30.5 / 30.7             63.6 / 66.9
    //            128, float32            12.3 / 11.3 15.7 / 14.4 17.3 / 18.2 17.5 / 18.7 21.5 / 22.1 22.9 / 24.9 28.3 / 31.0 33.8 / 34.1             77.4 / 76.2
    //            128                     11.4 / 10.5 13.7 / 12.8 15.5 / 16.0 16.5 / 16.5 20.0 / 20.1 22.0 / 23.4 27.0 / 29.9 32.3 / 33.0             68.3 / 71.8
    //            256, float32            13.3 / 11.8 16.7 / 15.0 18.3 / 18.8 18.6 / 19.1 22.3 / 22.7 24.5 / 25.4 30.2 / 31.7 35.9 / 34.9             85.0 / 81.8
    //            256                     12.3 / 10.7 14.7 / 12.7 16.4 / 16.1 17.2 / 16.6 20.8 / 20.7 22.7 / 23.7 28.6 / 30.0 33.9 / 33.1             71.7 / 71.8
    //            512                     13.0 / 11.0             17.8 / 16.9 18.5 / 17.3 23.0 / 21.5 25.2 / 24.7 31.2 / 31.7 38.5 / 34.7 44.2 / 44.8 78.5 / 75.6
    //            1024, float32           13.0 / 11.4             18.1 / 19.3 18.4 / 19.7 23.3 / 23.4 26.1 / 26.6 32.4 / 33.4 36.1 / 36.4 46.5 / 46.8 89.6 / 84.6
    //            1024                    12.7 / 11.2             16.7 / 17.1 17.6 / 17.5 22.1 / 21.7 25.1 / 24.9 31.8 / 31.9 35.4 / 34.9 44.9 / 45.1 80.2 / 76.4
    //            2048, float32           12.9 / 11.6             18.3 / 19.7 18.7 / 19.8 23.2 / 23.9 26.1 / 27.6 32.8 / 34.9 37.4 / 38.6 46.6 / 50.6 92.2 / 90.5
    //            2048                    12.9 / 11.0             16.8 / 17.4 17.7 / 17.8 22.2 / 22.0 25.4 / 26.0 32.3 / 33.4 35.7 / 36.9 45.6 / 48.0 81.0 / 82.4
    //    blocks of 8192: 1024 x 8192 15.0 / 11.9, 8192 x 8192 98.6 / 80.4, float32 106.9 / 87.8; 3000 x 24576 102.5 / 89.6.  Rows of several chunks: blocks
    //    of 512 8192 x 16384 168 / 153; of 1024 179 / 156, float32 184 / 162; of 2048 181 / 161, 3000 x 16384 65.8 / 63.1, float32 67.5 / 67.1, but with
    //    float32 amplitudes 3000 x 16384 55.5 / 55.5, 8192 x 16384 146 / 148, float32 163 / 171; of 128 and 256 4000 x 16384 66.1 / 68.6, 70.6 / 71.9.
    //  - Not blocks of 4096, of which four workgroups of eight values a lane fit a unit: 8192 x 8192 80.6 / 79.8, 1536 x 16384 float32 33.8 / 36.0.
    const int units = (int)(a.groups / 128);                         // of 1024 values, a wave's
    int waves = 8;
    while (log2n <= 10 && waves > 1 && units % waves != 0) waves--;
    const bool few = a.rows <= 768, whole = a.groups % 1024 == 0, one = a.groups == 1024, f32 = dtype == PVQ_F32;
    const bool some = a.rows <= 1152;                                // (between 1100 and 1300, see the table)
    bool halves = false;
    if (a.groups % 128 == 0 && waves > 2 && (!codes || units <= 4 * waves)) {
        if (log2n == 13) halves = !(f32 && codes && !one && few);
        else if (log2n == 11) halves = whole && (some || (codes && !one));
        else if (log2n == 10) halves = few || (whole && (some || !one || !f32 || a.rows > 2560));
        else if (log2n == 9) halves = few || whole;
        else if (log2n == 8) halves = few || (one && (some || (!f32 && a.rows <= 2048) || a.rows > 3072));
        else if (log2n == 6 || log2n == 7) halves = few || (one && some);
    }
    const size_t hbuf = log2n > 9 ? (size_t)(8 * L + 8 * L / 32 + 1) : 0;
    const size_t lds = (kHeadWords + (codes ? (size_t)((a.groups + 3) & ~3) : 0) + hbuf) * 4;
    if (halves) {
        const size_t lds_halves = (kHeadWords + waves * kWaveWords) * 4;
        const unsigned places = resident_grid(a.rows, waves * kWave, lds_halves);
#define PVQ_RE8_HALVES_N(T, C, LS_, N) \
    hipLaunchKernelGGL((rotate_encode8_halves_kernel<T, C, LS_, N>), dim3(places), dim3(waves * kWave), lds_halves, s, f, a, signs, scale)
#define PVQ_RE8_HALVES(T, C, LS_)                                                   \
    switch (log2n) {                                                                \
    case 13: PVQ_RE8_HALVES_N(T, C, LS_, 13); break;                                \
    case 11: PVQ_RE8_HALVES_N(T, C, LS_, 11); break;                                \
    case 10: PVQ_RE8_HALVES_N(T, C, LS_, 10); break;                                \
    case 9: PVQ_RE8_HALVES_N(T, C, LS_, 9); break;                                  \
    case 8: PVQ_RE8_HALVES_N(T, C, LS_, 8); break;                                  \
    case 7: PVQ_RE8_HALVES_N(T, C, LS_, 7); break;                                  \
    default: PVQ_RE8_HALVES_N(T, C, LS_, 6); break;                                 \
    }
#define PVQ_RE8_HALVES_C(T, LS_)                                                    \
    do {                                                                            \
        if (!codes) PVQ_RE8_HALVES(T, 0, LS_)                                       \
        else if (units == waves) PVQ_RE8_HALVES(T, 1, LS_)                          \
        else PVQ_RE8_HALVES(T, 4, LS_)                                              \
    } while (0)
        if (dtype == PVQ_F32) { if (ls) PVQ_RE8_HALVES_C(float, true); else PVQ_RE8_HALVES_C(float, false); }
        else { if (ls) PVQ_RE8_HALVES_C(uint16_t, true); else PVQ_RE8_HALVES_C(uint16_t, false); }
#undef PVQ_RE8_HALVES_C
#undef PVQ_RE8_HALVES
#undef PVQ_RE8_HALVES_N
        return hipGetLastError();
    }
    const unsigned grid = resident_grid(a.rows, L, lds);
#define PVQ_RE8_LAUNCH(KERNEL)                                                                                   \
    do {                                                                                                        \
        if (lds > 64 * 1024) {                                                                                  \
            const hipError_t e_ = hipFuncSetAttribute(reinterpret_cast<const void *>(KERNEL),                   \
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);    \
            if (e_ != hipSuccess) return e_;                                                                    \
        }                                                                                                       \
        hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(L), lds, s, f, a, log2n, signs, scale);                     \
    } while (0)
#define PVQ_RE8_N(T, C, LS_)                                                        \
    switch (log2n) {                                                                \
    case 12: PVQ_RE8_LAUNCH((rotate_encode8_kernel<T, C, LS_, 12>)); break;         \
    case 11: PVQ_RE8_LAUNCH((rotate_encode8_kernel<T, C, LS_, 11>)); break;         \
    case 10: PVQ_RE8_LAUNCH((rotate_encode8_kernel<T, C, LS_, 10>)); break;         \
    default: PVQ_RE8_LAUNCH((rotate_encode8_kernel<T, C, LS_, 9>)); break;          \
    }
    if (log2n == 13) {                                               // float32, codes, at most 768 rows of two to four blocks
        static_assert(kMaxGroups <= 4 * 8192 / D, "no row is too long for the kernel above");
        if (dtype != PVQ_F32 || !codes) return hipErrorInvalidValue;
        if (a.groups == 2 * L) { if (ls) PVQ_RE8_LAUNCH((rotate_encode8_kernel_8192<2, true>)); else PVQ_RE8_LAUNCH((rotate_encode8_kernel_8192<2, false>)); }
        else if (a.groups == 3 * L) { if (ls) PVQ_RE8_LAUNCH((rotate_encode8_kernel_8192<1, true>)); else PVQ_RE8_LAUNCH((rotate_encode8_kernel_8192<1, false>)); }
        else { if (ls) PVQ_RE8_LAUNCH((rotate_encode8_kernel_8192<4, true>)); else PVQ_RE8_LAUNCH((rotate_encode8_kernel_8192<4, false>)); }
        return hipGetLastError();
    }
    // (a wave has as many runs of 64 groups as a row has chunks; 11754 x 16384 in blocks of 8192: 301 us with four groups a lane, half the
    // waves without a code to write)
#define PVQ_RE8_C(T, LS_)                                                           \
    do {                                                                            \
        if (!codes) PVQ_RE8_N(T, 0, LS_)                                            \
        else if (a.groups == L || a.groups == 3 * L) PVQ_RE8_N(T, 1, LS_)           \
        else if (a.groups == 2 * L) PVQ_RE8_N(T, 2, LS_)                            \
        else PVQ_RE8_N(T, 4, LS_)                                                   \
    } while (0)
    if (dtype == PVQ_F32) { if (ls) PVQ_RE8_C(float, true); else PVQ_RE8_C(float, false); }
    else { if (ls) PVQ_RE8_C(uint16_t, true); else PVQ_RE8_C(uint16_t, false); }
#undef PVQ_RE8_C
#undef PVQ_RE8_N
#undef PVQ_RE8_LAUNCH
    return hipGetLastError();
}

bool pvq_encode8_usable(const pvq_ctx *c, const pvq_encode_args &a)
{
    // quads of lanes write whole dword triples; a row's sums of squares must fit the LDS buffer
    return c->enc8_offs != nullptr && a.groups % 4 == 0 && a.groups <= kMaxGroups;
}

hipError_t pvq_encode8_launch(const pvq_ctx *c, const pvq_encode_args &a, int dtype, hipStream_t s)
{
    enc8_launch f;
    f.offs = c->enc8_offs; f.edges = c->edges; f.K = c->K; f.scale_bits = c->scale_bits;
    const dim3 block(kBlock);
    const bool codes = c->scale_bits > 0;
    const size_t lds = (kHeadWords + (codes ? (size_t)a.groups : 0)) * 4;
    const unsigned grid = resident_grid(a.rows, kBlock, lds);
#define PVQ_ENC8_CASE(T, C, L) hipLaunchKernelGGL((encode8_kernel<T, C, L>), dim3(grid), dim3(block), lds, s, f, a)
    const bool ls = a.ls_amplitude != 0;
    // (runs of 64 groups that a wave has in a row: one, two, or more)
#define PVQ_ENC8_CODES(T, L)                                                        \
    do {                                                                            \
        if (!codes) PVQ_ENC8_CASE(T, 0, L);                                         \
        else if (a.groups <= kBlock) PVQ_ENC8_CASE(T, 1, L);                        \
        else if (a.groups <= 2 * kBlock) PVQ_ENC8_CASE(T, 2, L);                    \
        else PVQ_ENC8_CASE(T, 4, L);                                                \
    } while (0)
    if (dtype == PVQ_F32) { if (ls) PVQ_ENC8_CODES(float, true); else PVQ_ENC8_CODES(float, false); }
    else { if (ls) PVQ_ENC8_CODES(uint16_t, true); else PVQ_ENC8_CODES(uint16_t, false); }
#undef PVQ_ENC8_CODES
#undef PVQ_ENC8_CASE
    return hipGetLastError();
}
