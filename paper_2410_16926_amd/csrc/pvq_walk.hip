// Decoding coordinate by coordinate (App. B.3) with one table probe per coordinate, for every configuration
// that has no table-driven block decoder: groups of 16 and 32 (the paper's 3.25 bits/weight row is D = 16,
// K = 33, 52-bit indices), and groups of 8 with multi-word indices.  One lane owns one group.
//
// With q = N(D,K) - 1 - index first, a coordinate is the last threshold T_j of its row that is not above q, and q loses it
// (pvq_internal.h).  The thresholds of a row grow geometrically, so q's place among them follows from its magnitude: a
// guess row, indexed by the exponent and the leading fraction bits of q as a float, gives the last threshold below q's
// whole bucket, and only the one behind it is left to compare.  A coordinate is one byte and two neighbouring thresholds
// read from LDS, two subtractions, and the borrow of the second decides between them; App. B.3's search over magnitudes,
// and a binary search over the row (six dependent probes at K = 33), become two LDS reads.
//
// Widths: the integers of a step with d dimensions left are below N(d,K), so the later coordinates run in
// narrower arithmetic: dimensions above DX in W words, above DA in 3W/4, above DB in W/2, the rest in W/4 (for D = 16,
// K = 33: doubles, which hold 52 bits, down to nine dimensions, 32 bits from eight on, N(8,33) < 2^32).  The last two coordinates
// need no table: the thresholds of row 1 are 0, 1, 2, 4, 6, ..., and P(1,k) = {+k, -k}.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <utility>

#include "pvq_internal.h"
#include "pvq_walk.h"

namespace {

constexpr int kMaxThreads = 1024;   // lanes of a workgroup: 256 while the tables are small, 1024 (one copy of the
                                    // tables for sixteen waves) when they are not: two workgroups to a unit, or one where
                                    // the tables take more than half of its LDS (D = 32 from K = 68, D = 16 from 123)
constexpr int kWave = 64;

struct walk_launch {
    pvq_walk_params p;
    const unsigned char *blob;
    const float *sqrtc;
    int index_bits, scale_bits;
};

using namespace pvq_walk;

typedef __attribute__((ext_vector_type(4))) short bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// the sum over the lanes of the same place among R (4 or 8), in every lane: rotations by 4 and 8 inside the rows of 16, then
// across the rows
template <int R>
__device__ inline float sum_over_columns(float v)
{
    if constexpr (R == 4) v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x124, 0xF, 0xF, false));
    v += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x128, 0xF, 0xF, false));
    v += __shfl_xor(v, 16, kWave);
    return v + __shfl_xor(v, 32, kWave);
}

// What a group needs from memory, as it comes: the W + 1 words its index may touch, its amplitude (the float, or the
// word that holds its code).  Fetching does no arithmetic on loaded data and
// has no load under a condition, so the loads stay in flight until the item is taken apart, one item later: a wait placed
// right behind a load also waits for every store issued before it (memory operations complete in order).
template <int W>
struct raw_group {
    uint32_t w[W + 1];
    uint32_t amp;
};

// A part of the index plane that a wave reads from, as a buffer: words behind the plane's end read as 0 (and are not part
// of any field), so that a field's words need no bounds of their own.
struct index_plane {
    __amdgpu_buffer_rsrc_t words;
    __device__ inline index_plane(const pvq_decode_args &a, int64_t row)
    {
        const int64_t bytes = (a.rows - row) * a.index_row_words * 4;
        words = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.index) + row * a.index_row_words, 0,
                                                  (int)(uint32_t)std::min<int64_t>(bytes, 0xFFFFFFFC), 0x00027000);
    }
};

// from: byte of the row in the plane; srow: the row of the scale plane
template <int W>
__device__ inline void fetch_group(const index_plane &plane, uint32_t from, const void *__restrict__ scales, uint32_t scale_from,
                                   int g, int index_bits, int scale_bits, raw_group<W> &r)
{
    const uint32_t at = from + 4u * (__umul24((uint32_t)g, (uint32_t)index_bits) >> 5);     // (rows have at most 2^21 groups)
#pragma unroll
    for (int i = 0; i <= W; i++) r.w[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(plane.words, (int)(at + 4u * i), 0, 0);
    const uint32_t aw = scale_bits == 0 ? (uint32_t)g : __umul24((uint32_t)g, (uint32_t)scale_bits) >> 5;
    r.amp = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const unsigned char *>(scales) + (scale_from + 4u * aw));
}

template <int W>
__device__ inline typename wide<W>::type group_index(const raw_group<W> &r, int g, int bits)
{
    using T = typename wide<W>::type;
    const uint32_t sh = __umul24((uint32_t)g, (uint32_t)bits) & 31;
    uint32_t v[W];
#pragma unroll
    for (int i = 0; i < W; i++) {
        const int left = bits - 32 * i;                            // (the same for all lanes)
        const uint32_t mask = left >= 32 ? 0xFFFFFFFFu : left <= 0 ? 0u : (1u << left) - 1u;
        v[i] = __builtin_amdgcn_alignbit(r.w[i + 1], r.w[i], sh) & mask;
    }
    T c = 0;
#pragma unroll
    for (int i = 0; i < W; i++) c |= (T)v[i] << (32 * i);
    return c;
}

// the group's amplitude; with codes, relative to the square root of the row's normaliser
template <int W>
__device__ inline float group_amp(const raw_group<W> &r, int g, int scale_bits, const float *sqrtc)
{
    if (scale_bits == 0) return __uint_as_float(r.amp);
    return sqrtc[__builtin_amdgcn_ubfe(r.amp, __umul24((uint32_t)g, (uint32_t)scale_bits) & 31u, (uint32_t)scale_bits)];
}

// amp / sqrt(n2) (n2 >= 1), eight instructions against twenty for a square root and a quotient.  r lies below 1 / sqrt(n2)
// (the hardware's approximation, an ulp of error, less 2^-21 of it), and what r is short of it, to first order, is
// positive: the two terms of an infinite amplitude have one sign.  The product with r is rounded once, together with the
// other's; besides that only n2 * r is rounded at full size, half of which shows.  Error at most 1.5 * 2^-24 (1.46 over
// all n2 <= 127^2, 0.39 in the mean), against 1.96 and 0.47 for a rounded square root and a rounded quotient.
__device__ inline float norm_gain(float amp, float n2)
{
    const float r = __builtin_amdgcn_rsqf(n2) * 0x1.fffffp-1f;
    const float rest = (0.5f * r) * fmaf(-(n2 * r), r, 1.0f);
    return fmaf(amp, r, amp * rest);
}

// The lanes of a pair (T = 2) or quad: chunk[j] of lane i goes to chunk[i] of lane j.  i: the lane's place.
template <int CTRL>
__device__ inline void exchange_chunks(u32x4 &a, u32x4 &b, bool upper)
{
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const uint32_t from_a = (uint32_t)__builtin_amdgcn_mov_dpp((int)a[e], CTRL, 0xF, 0xF, true);
        const uint32_t from_b = (uint32_t)__builtin_amdgcn_mov_dpp((int)b[e], CTRL, 0xF, 0xF, true);
        a[e] = upper ? from_b : a[e];
        b[e] = upper ? b[e] : from_a;
    }
}
template <int T>
__device__ inline void transpose_chunks(u32x4 (&c)[T], int i)
{
    if constexpr (T == 2) exchange_chunks<0xB1>(c[0], c[1], i & 1);          // the pair's other lane
    if constexpr (T == 4) {
        exchange_chunks<0xB1>(c[0], c[1], i & 1);
        exchange_chunks<0xB1>(c[2], c[3], i & 1);
        exchange_chunks<0x4E>(c[0], c[2], i & 2);                            // two lanes on in the quad
        exchange_chunks<0x4E>(c[1], c[3], i & 2);
    }
}

// two values in bfloat16, rounded to nearest even
__device__ inline uint32_t bf16_pair(float lo, float hi)
{
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    const f32x2_t pair = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2_t));
}

__device__ inline uint16_t f32_to_f16_rne(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

// The tables into LDS, behind the amplitude table: straight from memory, 1 KiB a wave and instruction, all of them on
// their way at once (through registers, a thread that copies 16 bytes at a time waits for each of them: 60 KiB for groups
// of 32 took 4 us of a small launch).
__device__ inline void tables_to_lds(unsigned char *lds, const walk_launch &wl)
{
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
    for (uint32_t at = kWalkHead + 1024u * wave; at < wl.p.bytes; at += 1024u * (blockDim.x / kWave))
        if (at + 16u * lane < wl.p.bytes)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(wl.blob + at + 16u * lane),
                                             (__attribute__((address_space(3))) void *)(lds + at), 16, 0, 0);
    float *sqrtc = reinterpret_cast<float *>(lds);
    if (wl.scale_bits > 0)
        for (int i = threadIdx.x; i < (1 << wl.scale_bits); i += blockDim.x) sqrtc[i] = wl.sqrtc[i];
    __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
    __syncthreads();
}

// Decode to a matrix.  Workgroups stay for the whole launch (the tables are copied once each); after the copy
// every wave works alone and takes (row, 64 consecutive groups) items in turn.  A lane's group is D consecutive
// outputs, NC chunks of 16 bytes, and lanes that stored their own would write 16 bytes out of every D * size.  The N lanes of
// a pair or quad exchange chunks instead (an N x N transposition in registers, by data-parallel-primitive moves), so that a
// store of a lane is one chunk of a group that all N store; and the lanes of a block of 4 N hold its groups in the order
// in which the four pairs or quads then store consecutive groups: runs of 128 (N = 2) or 256 bytes (NC = 4; 64 bytes out of
// every 128 for NC = 8).  28672 x 8192 in groups of 16 to float32 252 us, to bfloat16 144, 14336 x 4096 in groups of 32 to
// bfloat16 51, to float32 96; laid out in LDS, or with larger tables stored as they are: 378, 174, 60 and 114.
// Groups of 8 to float32 (STAGE, where LDS has room for it beside the tables) are laid out in LDS: the walk of so few
// coordinates leaves no instructions to hide the exchange's behind (2500 x 5000 14.9 us, exchanged 15.6).
template <int D, int W, int DX, int DA, int DB, int OUT, bool STAGE>
__global__ __launch_bounds__(kMaxThreads) void decode_walk_kernel(walk_launch wl, pvq_decode_args a, int tiles)
{
    using T = typename wide<W>::type;
    constexpr int OSZ = OUT == PVQ_F32 ? 4 : 2;
    constexpr int NC = D * OSZ / 16;                 // 16-byte chunks of one group
    constexpr int N = STAGE ? 1 : NC < 4 ? NC : 4;
    const int kWaves = (int)blockDim.x / kWave;
    extern __shared__ __align__(16) unsigned char lds[];
    const float *sqrtc = reinterpret_cast<const float *>(lds);
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    u32x4 *stage = reinterpret_cast<u32x4 *>(lds + wl.p.bytes) + wave * (kWave * NC);
    tables_to_lds(lds, wl);
    const int G = (int)a.groups;
    // lane 4 N x + N y + i holds the wave's group 4 N x + 4 i + y, and stores chunk i (mod N) of the groups 4 N x + 4 j + y
    const int i_t = lane % N, y_t = lane / N % 4, block = lane - lane % (4 * N);
    const int place = block + 4 * i_t + y_t;
    const int64_t items = a.rows * tiles, stride = (int64_t)gridDim.x * kWaves;
    // What an item needs from memory is requested one item ahead, in front of the current item's stores: a
    // wait for a load also waits for every memory operation issued before it, so loads that follow stores
    // would make each item wait for the stores of the one before.  A wave past its last item, and lanes
    // past a row's last group, fetch a valid place again and drop it.
    raw_group<W> nx;
    int g_nx = 0;
    const int64_t srow_bytes = wl.scale_bits == 0 ? a.groups * 4 : a.scale_row_words * 4;
    float norm_nx = 0.0f;
    // (row, tile) of an item without a division per item: a wave moves on by `stride` items at a time
    const int64_t step_rows = stride / tiles;
    const int step_tiles = (int)(stride - step_rows * tiles);
    auto fetch = [&](int64_t row, int tile) {
        const int g = tile * kWave + place;
        g_nx = g < G ? g : 0;
        fetch_group<W>(index_plane(a, row), 0u, reinterpret_cast<const unsigned char *>(a.scale) + row * srow_bytes, 0u,
                       g_nx, wl.index_bits, wl.scale_bits, nx);
        norm_nx = wl.scale_bits == 0 ? 1.0f : a.rownorm[row];
    };
    const int64_t first = (int64_t)blockIdx.x * kWaves + wave;
    int64_t row_n = first / tiles;                              // the item that is being fetched
    int tile_n = (int)(first - row_n * tiles);
    if (first < items) fetch(row_n, tile_n);
    // The first item has arrived before the loop is entered (vmcnt(0), the other counters left alone): the loop then
    // starts, on its first pass as on every other, with nothing but stores in flight behind the item it takes
    // apart, and its waits are counted from there; sized for the entry path they would wait for the stores too.
    __builtin_amdgcn_s_waitcnt(0x0F70);
    for (int64_t item = first; item < items; item += stride) {
        const int64_t row = row_n;
        const int g0 = tile_n * kWave;                          // the wave's first group
        const int g_mine = g_nx;                                // the lane's group: g0 + place, or 0 past the row's end
        const T c = group_index<W>(nx, g_mine, wl.index_bits);
        const float amp = group_amp<W>(nx, g_mine, wl.scale_bits, sqrtc) * sqrtf(norm_nx);
        row_n += step_rows;
        tile_n += step_tiles;
        if (tile_n >= tiles) { tile_n -= tiles; row_n++; }
        if (row_n >= a.rows) { row_n = a.rows - 1; tile_n = tiles - 1; }   // past the last item: its place again, dropped
        fetch(row_n, tile_n);
        float y[D];
        const float n2 = unrank_walk<D, W, DX, DA, DB, next_from_decode(W)>(c, lds, wl.p, [&](int i, float minus_y) { y[i] = minus_y; });
        // direction on the unit sphere times the amplitude (Sec. 2.4): w = amp * y / ||y||_2
        const float gain = norm_gain(-amp, n2);
        // gain * y + 0: the product as it is, and +0 for a zero coordinate
        auto value = [&](int i) { return fmaf(gain, y[i], 0.0f); };
        unsigned char *orow = reinterpret_cast<unsigned char *>(a.W_out) + row * a.ldw * OSZ;
#pragma unroll
        for (int h = 0; h < NC; h += N) {
            u32x4 chunk[N];
#pragma unroll
            for (int j = 0; j < N; j++) {
                if constexpr (OUT == PVQ_F32) {
#pragma unroll
                    for (int e = 0; e < 4; e++) chunk[j][e] = __float_as_uint(value(4 * (h + j) + e));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const float f0 = value(8 * (h + j) + 2 * e), f1 = value(8 * (h + j) + 2 * e + 1);
                        if constexpr (OUT == PVQ_F16) chunk[j][e] = (uint32_t)f32_to_f16_rne(f0) | ((uint32_t)f32_to_f16_rne(f1) << 16);
                        else chunk[j][e] = bf16_pair(f0, f1);
                    }
                }
            }
            if constexpr (STAGE) {
                stage[lane * NC + h] = chunk[0];
                continue;
            }
            transpose_chunks<N>(chunk, i_t);
            // a place past the row's end holds the row's first group, decoded once more, which is stored where it belongs (the
            // same bytes as its owner writes): no store is under a condition, so that the number of stores in flight is
            // known where the next item's words are waited for, and that wait does not have to cover them
#pragma unroll
            for (int j = 0; j < N; j++) {
                const int g = g0 + block + 4 * j + y_t;
                const uint32_t at = (uint32_t)(g < G ? g : 0) * (NC * 16u) + (uint32_t)(h + i_t) * 16u;      // (rows have at most 2^21 groups)
                *reinterpret_cast<u32x4 *>(orow + at) = chunk[j];
            }
        }
        if constexpr (STAGE) {
            // the item's groups are consecutive chunks of the output; lanes past the item's end store its last chunk once
            // more (no store under a condition here either)
            const int last = std::min(kWave, G - g0) * NC - 1;
#pragma unroll
            for (int j = 0; j < NC; j++) {
                const int ch = std::min(j * kWave + lane, last);
                const u32x4 v = stage[ch];                     // written by this wave only: no barrier
                *reinterpret_cast<u32x4 *>(orow + (uint32_t)(g0 * NC + ch) * 16u) = v;
            }
        }
    }
}

// Decode fused into y = W_hat x for up to 16 vectors in one pass.  A wave's 64 groups are R rows x 64/R neighbouring group
// columns (lane = row + R column), so that a lane's own pulses, exact in bfloat16, are its part of one operand of a
// matrix instruction that computes several blocks at once, each of a group column's rows with the column's activations:
// 16 x 16 x 4 with four blocks (R = 16, 16 vectors) or 4 x 4 x 4 with sixteen (R = 4, four vectors, NV of them for 4 NV).  R = 8 is
// 4 x 4 x 4 too: a group column is two blocks, which hold four vectors each and by the instruction's broadcast both take those of one
// of them.  A load of activations fetches R vectors of 64/R columns, 64 places that lie apart, so that with few rows a tile a
// unit's loads take as long as its arithmetic (5 to 8 vectors, R = 4: two loads a column for four rows; R = 8: one for eight).
// D/4 of these in a row give the dot products of whole groups, whose gains (one per row and block) are multiplied
// afterwards: products exact in float32, as on the vector ALUs.  A workgroup takes R rows at a time, its waves take the
// columns in turn, and their sums meet in LDS, so that a few rows fill the chip as well.  Where the tables leave room for one
// workgroup to a unit, its waves are several teams, each with a tile of its own.
// Bound by the vector instructions of the walk, 19 a coordinate in all for D = 16, K = 33 and 26 for D = 32, K = 60, and 3 to 4 LDS
// reads (10 and 17 us on 14336 x 4096).  14336 x 4096, D = 16, K = 33,
// float32 amplitudes, 1 / 4 / 5 / 8 / 16 vectors: 27 / 29 / 29 / 30 / 37 us (28 / 29 / 32 / 41 / 39 with tiles of 4 and 16 rows only and
// integers for doubles); D = 32, K = 60: 40 / 41 / 42 / 43 / 50 (45 / 48 / 52 / 57 / 50); passes of 4, 2 and 1 vectors on the vector
// ALUs, a wave per row, took 48 / 64 / 110 / - / 254 and 109 / 203 / 317 / - / 809.
struct gemv_teams {
    int waves, teams;
    int inverse;        // 256 / waves, rounded up: wave * inverse / 256 is the team of one of at most sixteen waves
};

// Waves of a SIMD that a kernel's registers are to leave room for: eight in tiles of 16 rows of groups of 16 and 32 with up to
// two words, which the schedule of the reads would pass by a few registers (next_from_product); else those of a workgroup of 1024 lanes.
constexpr int gemv_waves(int D, int W, int R) { return D >= 16 && W <= 2 && R == 16 ? 8 : 4; }

template <int D, int W, int DX, int DA, int DB, int R, int NV>
__global__ __launch_bounds__(kMaxThreads, gemv_waves(D, W, R)) void gemv_walk_kernel(walk_launch wl, pvq_decode_args a, int b0, int vectors, int row_tiles, gemv_teams split)
{
    static_assert(R == 16 ? NV == 4 : R == 8 ? NV <= 2 : R == 4, "tiles");
    using T = typename wide<W>::type;
    constexpr int CG = kWave / R;                  // group columns of a wave
    constexpr int XV = R == 4 ? NV : 1;            // vectors whose activations a lane holds
    constexpr int XW = D / 8;                      // 16-byte words of one group's activations
    constexpr int kSums = 4 * R * NV;              // of a tile: rows x vectors
    extern __shared__ __align__(16) unsigned char lds[];
    const float *sqrtc = reinterpret_cast<const float *>(lds);
    const int lane = threadIdx.x % kWave;
    const int wave_all = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int waves = split.waves, teams = split.teams, waves_all = waves * teams;
    const int team = wave_all * split.inverse >> 8, wave = wave_all - team * waves;
    float *gains = reinterpret_cast<float *>(lds + wl.p.bytes) + wave_all * kWave;
    float *sums = reinterpret_cast<float *>(lds + wl.p.bytes) + (R == 16 ? waves_all * kWave : 0) + team * waves * kSums;
    const int G = (int)a.groups;
    const int chunks = (G + CG - 1) / CG;
    const int row_l = lane % R, col_l = lane / R;
    const uint32_t scale_row_words = (uint32_t)(wl.scale_bits == 0 ? a.groups : a.scale_row_words);
    raw_group<W> nx;
    int g_nx = 0;
    // (rows and columns past the end fetch the last ones again; such rows are not written, such columns' dot products left out)
    auto fetch = [&](int tile, int chunk) {
        const int64_t row0 = (int64_t)tile * R;
        const uint32_t row = (uint32_t)std::min<int64_t>(row_l, a.rows - 1 - row0);
        g_nx = std::min(chunk * CG + col_l, G - 1);
        fetch_group<W>(index_plane(a, row0), 4u * __umul24(row, (uint32_t)a.index_row_words), reinterpret_cast<const uint32_t *>(a.scale) + row0 * scale_row_words,
                       4u * __umul24(row, scale_row_words), g_nx, wl.index_bits, wl.scale_bits, nx);
    };
    const uint16_t *x0[XV];
#pragma unroll
    for (int v = 0; v < XV; v++)
        x0[v] = reinterpret_cast<const uint16_t *>(a.x) + (int64_t)(b0 + std::min(R * v + lane % R, vectors - 1)) * a.ldx;
    const int stride = (int)gridDim.x * teams;
    // (a team without a tile of its own, in a workgroup's last turn, fetches the last one and leaves it)
    fetch(std::min((int)blockIdx.x * teams + team, row_tiles - 1), wave);   // (there are no more waves than chunks)
    tables_to_lds(lds, wl);
    int turn = 0;
    for (int first = (int)blockIdx.x * teams; first < row_tiles; first += stride, turn++) {
        const int tile = first + team;
        const bool live = tile < row_tiles;
        constexpr int AV = R == 16 ? 1 : NV;
        f32x4 acc[AV];                             // R = 16: rows 4 (lane / 16) + r, vector lane % 16; else the lane's own row, vector 4 v + r
#pragma unroll
        for (int v = 0; v < AV; v++) acc[v] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int chunk = live ? wave : chunks; chunk < chunks; chunk += waves) {
            const T c = group_index<W>(nx, g_nx, wl.index_bits);
            const float amp = group_amp<W>(nx, g_nx, wl.scale_bits, sqrtc);
            uint4 x[XV][XW];
#pragma unroll
            for (int v = 0; v < XV; v++)
#pragma unroll
                for (int w = 0; w < XW; w++) x[v][w] = *reinterpret_cast<const uint4 *>(x0[v] + ((int64_t)g_nx * D + 8 * w));
            // the wave's next groups: of this tile, or of its next one
            const bool here = chunk + waves < chunks;
            fetch(here ? tile : std::min(tile + stride, row_tiles - 1), here ? chunk + waves : wave);
            f32x16 out16;
            f32x4 out4[AV];
            if constexpr (R == 16) {
#pragma unroll
                for (int i = 0; i < 16; i++) out16[i] = 0.0f;
            } else {
#pragma unroll
                for (int v = 0; v < AV; v++) out4[v] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
            uint32_t pair[2];
            float even = 0.0f;
            const float n2 = unrank_walk<D, W, DX, DA, DB, next_from_product(D, W, DX, DA, R)>(c, lds, wl.p, [&](int i, float minus_y) {
                if ((i & 1) == 0) { even = minus_y; return; }
                pair[(i >> 1) & 1] = __builtin_amdgcn_perm(__float_as_uint(minus_y), __float_as_uint(even), 0x07060302u);
                if ((i & 3) != 3) return;
                const bf16x4 y4 = __builtin_bit_cast(bf16x4, make_uint2(pair[0], pair[1]));
                auto x4 = [&](int v) {
                    const uint4 q = x[v][i / 8];
                    return __builtin_bit_cast(bf16x4, (i & 4) ? make_uint2(q.z, q.w) : make_uint2(q.x, q.y));
                };
                // (R = 8: the two blocks of a group column take the activations of its first or second block)
                if constexpr (R == 16) {
                    out16 = __builtin_amdgcn_mfma_f32_16x16x4bf16_1k(y4, x4(0), out16, 0, 0, 0);
                } else if constexpr (R == 8) {
                    out4[0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(x4(0), y4, out4[0], 1, 0, 0);
                    if constexpr (NV == 2) out4[1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(x4(0), y4, out4[1], 1, 1, 0);
                } else {
#pragma unroll
                    for (int v = 0; v < NV; v++) out4[v] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(x4(v), y4, out4[v], 0, 0, 0);
                }
            });
            float gain = norm_gain(-amp, n2);
            if constexpr (R == 16) {
                gains[lane] = gain;                // (read by this wave only)
#pragma unroll
                for (int blk = 0; blk < 4; blk++) {
                    if (chunk * CG + blk >= G) break;
                    const f32x4 g4 = *reinterpret_cast<const f32x4 *>(gains + 16 * blk + 4 * (lane / 16));
#pragma unroll
                    for (int r = 0; r < 4; r++) acc[0][r] = fmaf(g4[r], out16[4 * blk + r], acc[0][r]);
                }
            } else {
                if ((chunk + 1) * CG > G) {        // (both 0: the gain and the dot products of the last group may be infinite)
                    gain = chunk * CG + col_l < G ? gain : 0.0f;
#pragma unroll
                    for (int v = 0; v < AV; v++)
#pragma unroll
                        for (int r = 0; r < 4; r++) out4[v][r] = chunk * CG + col_l < G ? out4[v][r] : 0.0f;
                }
#pragma unroll
                for (int v = 0; v < AV; v++)
#pragma unroll
                    for (int r = 0; r < 4; r++) acc[v][r] = fmaf(gain, out4[v][r], acc[v][r]);
            }
        }
        const int64_t row0 = (int64_t)tile * R;
        auto write = [&](const float *from, int t) {               // sum t of the tile, over the waves
            const int vec = R == 16 ? (t >> 2) & 15 : 4 * (t / (4 * R)) + (t & 3);
            const int64_t row = row0 + (R == 16 ? 4 * (t >> 6) + (t & 3) : t / 4 % R);
            if (vec >= vectors || row >= a.rows) return;           // (no row of a team without a tile)
            const float norm = wl.scale_bits == 0 ? 1.0f : sqrtf(a.rownorm[row]);
            float v = from[t];
            for (int w = 1; w < waves; w++) v += from[w * kSums + t];
            a.y[(int64_t)(b0 + vec) * a.ldy + row] = v * norm;
        };
        if constexpr (R != 16) {
            // The group columns' sums, then the waves': two places in turn, so that the wave that writes this tile is done
            // with its place when the others come to use it again, one barrier later.
            float *to = sums + (turn & 1) * (waves_all * kSums);
#pragma unroll
            for (int v = 0; v < AV; v++) {
#pragma unroll
                for (int r = 0; r < 4; r++) acc[v][r] = sum_over_columns<R>(acc[v][r]);
                if (lane < R) *reinterpret_cast<f32x4 *>(to + wave * kSums + 4 * R * v + 4 * lane) = acc[v];
            }
            __syncthreads();
            if (wave == turn % waves && lane < kSums) write(to, lane);
        } else {
            __syncthreads();                       // (the tile before has been read)
            *reinterpret_cast<f32x4 *>(sums + wave * kSums + 4 * lane) = acc[0];
            __syncthreads();
            for (int t = wave * kWave + lane; t < kSums; t += waves * kWave) write(sums, t);
        }
    }
}

int g_units = 0;

int units()
{
    if (g_units == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            g_units = n;
        else
            g_units = 256;
    }
    return g_units;
}

walk_launch make_launch(const pvq_ctx *c)
{
    walk_launch wl;
    wl.p = c->walk; wl.blob = c->walk_blob; wl.sqrtc = c->sqrtc;
    wl.index_bits = c->index_bits; wl.scale_bits = c->scale_bits;
    return wl;
}

// lanes of a workgroup for a context: small tables are copied by many small workgroups (eight to a unit's 160 KiB), large
// ones once per sixteen waves
int block_threads(const pvq_ctx *c) { return c->walk.bytes <= 20 * 1024 ? 256 : kMaxThreads; }

size_t lds_bytes(const pvq_ctx *c) { return (size_t)c->walk.bytes; }      // the tables

// What a launch of a kernel with `bytes` of dynamic LDS needs first.  table_at counts on dynamic LDS starting at byte 0: a
// kernel that has come to have static LDS as well (the compiler may move private arrays there) is refused; that is asked
// once per kernel.  Kernels that need more LDS than a kernel gets without asking (64 KiB) say so.
template <auto Kernel>
hipError_t allow_lds(size_t bytes)
{
    static std::atomic<bool> checked{false};
    if (!checked.load(std::memory_order_relaxed)) {
        hipFuncAttributes attributes;
        const hipError_t e = hipFuncGetAttributes(&attributes, reinterpret_cast<const void *>(Kernel));
        if (e != hipSuccess) return e;
        if (attributes.sharedSizeBytes != 0) return hipErrorInvalidDeviceFunction;
        checked.store(true, std::memory_order_relaxed);
    }
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Waves of a kernel that a SIMD holds by the kernel's registers, asked once per kernel (a workgroup of four waves has one on
// each SIMD).
template <auto Kernel>
int waves_per_simd()
{
    static std::atomic<int> known{0};
    int n = known.load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(Kernel), 4 * kWave, 0) != hipSuccess) {
            (void)hipGetLastError();
            n = 0;
        }
        n = std::min(std::max(n, 4), 8);           // (a workgroup of 1024 lanes has four)
        known.store(n, std::memory_order_relaxed);
    }
    return n;
}

// workgroups of a launch over `items` wave items: 32 waves per unit, fewer if the work is small
unsigned persistent_grid(const pvq_ctx *c, int64_t items)
{
    const int64_t per_block = block_threads(c) / kWave;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + per_block - 1) / per_block, (int64_t)units() * 32 / per_block));
}

template <int D, int W, int DX, int DA, int DB, int OUT, bool STAGE>
hipError_t launch_decode_staged(const pvq_ctx *c, const pvq_decode_args &a, size_t lds, hipStream_t s)
{
    const int tiles = (int)((a.groups + kWave - 1) / kWave);
    const hipError_t e = allow_lds<decode_walk_kernel<D, W, DX, DA, DB, OUT, STAGE>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_walk_kernel<D, W, DX, DA, DB, OUT, STAGE>), dim3(persistent_grid(c, a.rows * tiles)), dim3(block_threads(c)), lds, s,
                       make_launch(c), a, tiles);
    return hipGetLastError();
}

template <int D, int W, int DX, int DA, int DB, int OUT>
hipError_t launch_decode_out(const pvq_ctx *c, const pvq_decode_args &a, hipStream_t s)
{
    if constexpr (D == 8 && OUT == PVQ_F32) {
        // where the unit's 160 KiB still hold 32 waves with 64 groups each
        const size_t staged = lds_bytes(c) + (size_t)block_threads(c) * D * 4;
        if (staged * (2048 / block_threads(c)) <= 160 * 1024) return launch_decode_staged<D, W, DX, DA, DB, OUT, true>(c, a, staged, s);
    }
    return launch_decode_staged<D, W, DX, DA, DB, OUT, false>(c, a, lds_bytes(c), s);
}

template <int D, int W, int DX, int DA, int DB>
hipError_t launch_decode(const pvq_ctx *c, const pvq_decode_args &a, int out_dtype, hipStream_t s)
{
    switch (out_dtype) {
    case PVQ_F32: return launch_decode_out<D, W, DX, DA, DB, PVQ_F32>(c, a, s);
    case PVQ_F16: return launch_decode_out<D, W, DX, DA, DB, PVQ_F16>(c, a, s);
    default: return launch_decode_out<D, W, DX, DA, DB, PVQ_BF16>(c, a, s);
    }
}

// workgroups with so much LDS that a unit's 160 KiB hold (given out in steps of 1280 bytes)
int unit_copies(size_t lds) { return (int)(160 * 1024 / ((lds + 1279) / 1280 * 1280)); }

// How a pass is split: tiles of `rows` rows, `waves` waves for each, `teams` of so many waves per workgroup
struct gemv_split {
    int rows, waves, teams;
    unsigned grid;
};

// LDS of a pass: tables, a gain per lane, the waves' sums (rows x vectors; two places for tiles of four and eight rows)
size_t gemv_lds(const pvq_ctx *c, int waves, int R, int sums)
{
    return (size_t)c->walk.bytes + (size_t)waves * (R == 16 ? kWave + sums : 2 * sums) * sizeof(float);
}

// The split that should take least, from what a wave's 64 groups take in clocks: alone, as a chain of table reads; of
// a SIMD's issue slots, when several waves share it; of the unit's loads of activations, which a tile of four rows
// repeats four times as often (11 bytes a clock) and one of eight once for every eight vectors; and what a tile takes besides.  These
// are estimates (a line each through products of D = 8, 16 and 32), not a bound: of 234 products (six contexts, 64 x 4096 to
// 8192 x 28672, 1 to 16 vectors) the split picked among tiles of 4 and 16 rows is 6 % slower than the best one in the median, 18 % at
// the ninth decile, 47 % at the worst.  Tiles of 16 rows are for more than four vectors on large matrices (D = 32, 14336 x 4096, 16
// vectors: 50 us, with four rows 79), of four rows where those would leave units idle (1289 x 16384, 11 vectors: 37 us, with sixteen 50),
// of eight for up to eight vectors on large matrices (us, with eight rows / as it was with four or sixteen, 1 and 8 vectors):
//   14336 x 4096, D = 32, K = 60: 40 / 45, 43 / 57;  D = 16, K = 33: 28.5 / 27.2 (fewer waves in flight: four rows), 30 / 41
//   28672 x 8192, D = 16, K = 33: 92 / 108, 103 / 115;  14681 x 2560, D = 32, K = 60: 39 / 63, 42 / 33 (sixteen rows)
// Tiles of sixteen rows, where the estimate picked those, are slower than of eight with groups of up to 16 and no search behind the guess
// (above); with groups of 32 and with a search they are 6 % to 25 % faster or within 3 % (28672 x 8192, 8 vectors, D = 32, K = 60:
// 150 us, with eight 163; D = 16, K = 45: 130, 138).
// How many workgroups a unit holds follows from their LDS and from the kernel's registers (simd4, simd8, simd16: waves of a
// SIMD, for tiles of 4, 8 and 16 rows); a workgroup more than that waits for a whole one (D = 16, K = 59, one vector on
// 14336 x 4096: 114 us where three copies of the tables were thought to fit, with two 63).
// tile_rows: only tiles of so many rows are looked at (0: all).
gemv_split split_gemv(const pvq_ctx *c, int64_t rows, int64_t groups, int vectors, int tile_rows, int simd4, int simd8, int simd16)
{
    gemv_split best = {0, 0, 0, 0};
    double least = 0;
    int in_flight = 0;                             // waves of a unit with the best split
    const double chain = 280.0 * c->D, issue = 4.0 * (80.0 + c->D * (c->words == 1 ? 14.0 : c->words == 2 ? 17.0 : 25.0));
    for (const int R : {4, 16, 8}) {
        if (tile_rows ? R != tile_rows : R == 16 && vectors <= 4) continue;
        // (with one tile of four rows to a unit, eight would leave half of them idle)
        if (R == 8 && !tile_rows && (rows <= 4 * units() || (best.rows == 16 && (c->D > 16 || c->walk.more != 0)))) continue;
        const int nv = vectors <= 4 ? 1 : vectors <= 8 ? 2 : 4, sums = R == 16 ? 256 : 4 * R * nv;
        if (R == 8 && nv > 2) continue;
        const double loads = c->D * 128.0 / 11.0 * (R == 4 ? nv : R == 8 ? nv / 2.0 : 1.0);
        const int64_t tiles = (rows + R - 1) / R;
        const int chunks = ((int)groups + kWave / R - 1) / (kWave / R), tiles_unit = (int)((tiles + units() - 1) / units());
        gemv_split mine = {0, 0, 0, 0};            // the best of these tiles
        double cost_mine = 0;
        int waves_mine = 0;
        bool most = true;                          // the most waves that have a chunk each
        for (int waves = 16; waves >= 1; waves -= waves > 8 ? 4 : waves > 4 ? 2 : 1) {
            if (waves > chunks) continue;
            const bool all = most;
            most = false;
            const size_t lds = gemv_lds(c, waves, R, sums);
            if (lds > 160 * 1024) continue;
            const int resident = 4 * (R == 16 ? simd16 : R == 8 ? simd8 : simd4);            // waves of a unit
            const int blocks = std::max(1, std::min(std::min(resident / waves, unit_copies(lds)), tiles_unit));
            // One workgroup to a unit, and a row too short for its waves: more teams.  D = 32, one vector on 14336 x 4096,
            // K = 68 / 80 / 105: two teams of eight 57 / 63 / 71 us (before the walk's search became shorter eight waves took
            // 145 / 170 / 171, two teams 91 / 108 / 108).
            int teams = 1;
            if (all && unit_copies(c->walk.bytes) == 1)
                while (teams < tiles_unit && (teams + 1) * waves <= std::min(resident, 16) && gemv_lds(c, (teams + 1) * waves, R, sums) <= 160 * 1024) teams++;
            const double turns = (double)((tiles_unit + blocks * teams - 1) / (blocks * teams)), steps = (double)((chunks + waves - 1) / waves);
            const double cost = std::max(std::max(turns * steps * chain, (double)tiles_unit * steps * waves / 4.0 * issue),
                                         (double)tiles_unit * steps * waves * loads) + turns * (R == 16 ? 2500.0 : 1000.0);
            if (mine.rows == 0 || cost < cost_mine) {
                cost_mine = cost;
                waves_mine = blocks * teams * waves;
                mine = {R, waves, teams, (unsigned)std::min<int64_t>((tiles + teams - 1) / teams, (int64_t)units() * blocks)};
            }
        }
        if (mine.rows == 0) continue;
        // Tiles of eight rows with fewer waves in flight than the best of the others hide less (14336 x 4096, D = 16, K = 33, one
        // vector: 28 waves 28.5 us, with four rows 32 27.2; 8192 x 14336, D = 32, K = 80: 12 waves 122, 16 114), and groups of 32 gain
        // nothing where the estimates are equal (8173 x 22528, K = 50, one vector: 111, with four rows 107), those with integers of
        // one word only where it is well ahead (3001 x 11008, K = 4, five vectors, the estimate 5 % ahead: 24.6, with four rows 20.6;
        // 2048 x 8192, 25 % ahead: 19.0 and 20.6).
        if (R == 8 && best.rows != 0) {
            if (waves_mine < in_flight) cost_mine *= 1.5 - 0.5 * waves_mine / in_flight;
            cost_mine *= c->D < 32 ? 1.0 : c->words == 1 ? 1.1 : 1.01;
        }
        if (best.rows == 0 || cost_mine < least) {
            least = cost_mine;
            in_flight = waves_mine;
            best = mine;
        }
    }
    return best;
}

template <int D, int W, int DX, int DA, int DB, int R, int NV>
hipError_t launch_gemv_pass(const pvq_ctx *c, const pvq_decode_args &a, int b0, int vectors, const gemv_split &split, hipStream_t s)
{
    const size_t lds = gemv_lds(c, split.waves * split.teams, R, 4 * R * NV);
    const hipError_t e = allow_lds<gemv_walk_kernel<D, W, DX, DA, DB, R, NV>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemv_walk_kernel<D, W, DX, DA, DB, R, NV>), dim3(split.grid), dim3((unsigned)(split.waves * split.teams * kWave)), lds, s,
                       make_launch(c), a, b0, vectors, (int)((a.rows + R - 1) / R), gemv_teams{split.waves, split.teams, (256 + split.waves - 1) / split.waves});
    return hipGetLastError();
}

template <int D, int W, int DX, int DA, int DB>
hipError_t launch_gemv(const pvq_ctx *c, const pvq_decode_args &a, int tile_rows, hipStream_t s)
{
    for (int b0 = 0; b0 < a.batch; b0 += 16) {
        const int vectors = std::min(a.batch - b0, 16);
        const gemv_split split = split_gemv(c, a.rows, a.groups, vectors, tile_rows,
                                            vectors <= 4 ? waves_per_simd<gemv_walk_kernel<D, W, DX, DA, DB, 4, 1>>()
                                            : vectors <= 8 ? waves_per_simd<gemv_walk_kernel<D, W, DX, DA, DB, 4, 2>>()
                                                           : waves_per_simd<gemv_walk_kernel<D, W, DX, DA, DB, 4, 4>>(),
                                            vectors <= 4 ? waves_per_simd<gemv_walk_kernel<D, W, DX, DA, DB, 8, 1>>()
                                                         : waves_per_simd<gemv_walk_kernel<D, W, DX, DA, DB, 8, 2>>(),
                                            waves_per_simd<gemv_walk_kernel<D, W, DX, DA, DB, 16, 4>>());
        if (split.rows == 0) return hipErrorInvalidValue;          // (no LDS left beside the tables: only where tile_rows asks for 8 or 16)
        hipError_t e;
        if (split.rows == 8 && vectors <= 4) e = launch_gemv_pass<D, W, DX, DA, DB, 8, 1>(c, a, b0, vectors, split, s);
        else if (split.rows == 8) e = launch_gemv_pass<D, W, DX, DA, DB, 8, 2>(c, a, b0, vectors, split, s);
        else if (split.rows == 16) e = launch_gemv_pass<D, W, DX, DA, DB, 16, 4>(c, a, b0, vectors, split, s);
        else if (vectors <= 4) e = launch_gemv_pass<D, W, DX, DA, DB, 4, 1>(c, a, b0, vectors, split, s);
        else if (vectors <= 8) e = launch_gemv_pass<D, W, DX, DA, DB, 4, 2>(c, a, b0, vectors, split, s);
        else e = launch_gemv_pass<D, W, DX, DA, DB, 4, 4>(c, a, b0, vectors, split, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

bool pvq_walk_usable(const pvq_ctx *c)
{
    // the tables and the amplitude table must fit LDS
    return c->walk_blob != nullptr && lds_bytes(c) <= 160 * 1024;
}

hipError_t pvq_walk_launch_decode(const pvq_ctx *c, const pvq_decode_args &a, int out_dtype, hipStream_t s)
{
#define PVQ_WALK_DECODE(D, W, DX, DA, DB) launch_decode<D, W, DX, DA, DB>(c, a, out_dtype, s)
    PVQ_WALK_DISPATCH(PVQ_WALK_DECODE, c->D, c->words, c->walk.dX, c->walk.dA, c->walk.dB);
#undef PVQ_WALK_DECODE
}

hipError_t pvq_walk_launch_gemv(const pvq_ctx *c, const pvq_decode_args &a, int tile_rows, hipStream_t s)
{
#define PVQ_WALK_GEMV(D, W, DX, DA, DB) launch_gemv<D, W, DX, DA, DB>(c, a, tile_rows, s)
    PVQ_WALK_DISPATCH(PVQ_WALK_GEMV, c->D, c->words, c->walk.dX, c->walk.dA, c->walk.dB);
#undef PVQ_WALK_GEMV
}
