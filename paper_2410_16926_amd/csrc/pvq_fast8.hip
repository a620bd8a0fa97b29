// gfx950 kernels built on the D = 8 table-driven decoder (pvq_fast8.h): decode to a matrix, and
// decode fused into y = W_hat x.
//
// One workgroup per compute unit keeps the whole table blob (up to 156 KiB) in LDS and walks many
// rows, so the copy is paid once per launch and unit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pvq_internal.h"

namespace {

constexpr int kWave = 64;
constexpr int kMaxThreads = 1024;
constexpr int kGemvThreads = 1024;   // lanes of a fused-product workgroup (half as many with twice the
                                     // groups in flight per lane measured 30 % slower)
constexpr int kGroupsPerLane = 4;
constexpr int kTileGroups = kWave * kGroupsPerLane;   // groups one wave covers in a row: 256
constexpr int kLdsBytes = 160 * 1024;                 // the whole LDS of a compute unit

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;

__device__ inline float dot2_bf16(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

struct fast8_launch {
    pvq_fast8_params p;
    const unsigned char *blob;
    const float *sqrtc;  // 2^scale_bits entries, or nullptr
    int index_bits, scale_bits;
};

// The fused gain table (see load_tables) in LDS: rows 0 or 1, 2 or 3, ... of n2; an odd n2's first row lies one group of
// codes and a half further on, so that 2 * n2 * 2^scale_bits is a row's place from lds_bytes on.
__host__ __device__ inline uint32_t fused_rows(const pvq_fast8_params &p) { return p.k2max / 2 + 1; }
__host__ __device__ inline uint32_t fused_start(const fast8_launch &f) { return f.p.lds_bytes + ((2u * (f.p.k2max & 1u)) << f.scale_bits); }

// Copies the blob into LDS.  With FUSED (amplitude codes of at most 2 bits) the blob's last table,
// 1/sqrt(n2), is left out and its place taken by gain[n2/2][q] = (1/sqrt(n2)) * sqrt(center[q]),
// 2^scale_bits floats per n2 (which is as odd or even as K), so that one lookup gives a group's whole gain; otherwise the
// 2^scale_bits values sqrt(center[q]) follow the blob.
template <bool FUSED>
__device__ inline void load_tables(unsigned char *lds, const fast8_launch &f, float *sqrtc_l)
{
    const int nthreads = blockDim.x;
    const uint32_t bytes = FUSED ? f.p.lds_bytes : f.p.blob_bytes;
    // Every workgroup starts at another place of the blob (with all units asking for the same lines in the same
    // order, one L2 channel at a time serves the whole machine), two 16-byte pieces per lane and trip.  (All ten
    // pieces of a lane requested before the first LDS write measured 13 us slower per launch, one at a time and no
    // rotation 1.7 us slower.)
    const uint32_t pieces = (bytes + 15u) / 16u;
    const uint32_t rot = (uint32_t)((blockIdx.x * 37u) % 64u) * (pieces / 64u);
    for (uint32_t c = threadIdx.x; c < pieces; c += 2 * nthreads) {
        uint32_t s0 = c + rot, s1 = c + nthreads + rot;
        s0 = s0 >= pieces ? s0 - pieces : s0;
        s1 = s1 >= pieces ? s1 - pieces : s1;
        const bool two = c + nthreads < pieces;
        s1 = two ? s1 : s0;
        const uint4 v0 = *reinterpret_cast<const uint4 *>(f.blob + s0 * 16u);
        const uint4 v1 = *reinterpret_cast<const uint4 *>(f.blob + s1 * 16u);
        *reinterpret_cast<uint4 *>(lds + s0 * 16u) = v0;
        *reinterpret_cast<uint4 *>(lds + s1 * 16u) = v1;
    }
    if constexpr (FUSED) {
        const int n = (int)fused_rows(f.p);
        for (int i = threadIdx.x; i < (n << f.scale_bits); i += nthreads) {
            const uint32_t n2 = 2u * (uint32_t)(i >> f.scale_bits) + (f.p.k2max & 1u);
            const int q = i & ((1 << f.scale_bits) - 1);
            sqrtc_l[i] = *reinterpret_cast<const float *>(f.blob + f.p.invs + 2u * n2) * f.sqrtc[q];
        }
    } else if (f.scale_bits > 0) {
        for (int i = threadIdx.x; i < (1 << f.scale_bits); i += nthreads) sqrtc_l[i] = f.sqrtc[i];
    }
    __syncthreads();
}

// Work mapping.  A wave works on a tile of 256 consecutive groups of one row; lane l owns the groups
// tile*256 + 64*j + l, j = 0..3.  So for every j the 64 lanes touch 64 consecutive groups: the index
// reads of one j cover 192 contiguous bytes and, in the decode kernel, the stores of one j cover one
// contiguous KiB (a lane that kept four neighbouring groups would write 16 bytes out of every 64 per
// store instruction, which measured 2.5x slower).

// What a lane fetches for its four groups of one row.  Raw words only: no arithmetic touches loaded
// data until the item is consumed, so that the loads stay in flight behind the previous item's work.
struct item_t {
    uint32_t w[kGroupsPerLane];   // index: the dword at byte 3g-1 of the row (24-bit path) or the index itself
    uint32_t a[kGroupsPerLane];   // amplitude: the code word holding group g's code, or the float's bits
};

// Branch-free on purpose: every lane loads (lanes beyond the row re-read its first group, a wave
// past its last item re-reads a valid one).  With loads under conditions the compiler cannot count
// how many are in flight and makes every use of an item wait for ALL outstanding memory operations,
// the stores of the previous item included.
template <bool CODES, bool B24>
__device__ inline void fetch_item(const fast8_launch &f, const pvq_decode_args &a, int64_t row, int gbase,
                                  item_t &it)
{
    const int G = (int)a.groups;
    const uint32_t *irow = a.index + row * a.index_row_words;
#pragma unroll
    for (int j = 0; j < kGroupsPerLane; j++) {
        const int gj = gbase + kWave * j;
        const int g = gj < G ? gj : 0;
        if constexpr (B24) {
            // the 3 bytes of group g start at byte 3g; one dword load from byte 3g-1 (3g for g = 0)
            // holds them and stays inside the row
            const unsigned char *p = reinterpret_cast<const unsigned char *>(irow) + 3 * g - (g > 0 ? 1 : 0);
            uint32_t v;
            __builtin_memcpy(&v, p, 4);
            it.w[j] = v;
        } else {
            const uint32_t b = (uint32_t)f.index_bits;
            const uint32_t pos = (uint32_t)g * b, w0 = pos >> 5, sh = pos & 31;
            uint64_t v = irow[w0];
            if (sh + b > 32) v |= (uint64_t)irow[w0 + 1] << 32;
            it.w[j] = (uint32_t)(v >> sh) & (uint32_t)((1ull << b) - 1ull);
        }
        if constexpr (CODES) {
            const uint32_t *srow = reinterpret_cast<const uint32_t *>(a.scale) + row * a.scale_row_words;
            it.a[j] = srow[((uint32_t)g * (uint32_t)f.scale_bits) >> 5];
        } else {
            it.a[j] = __float_as_uint(reinterpret_cast<const float *>(a.scale)[row * a.groups + g]);
        }
    }
}

// the four indices of an item
template <bool B24>
__device__ inline void item_indices(const item_t &it, int gbase, uint32_t (&c)[kGroupsPerLane])
{
#pragma unroll
    for (int j = 0; j < kGroupsPerLane; j++) {
        if constexpr (B24) c[j] = (gbase + kWave * j > 0) ? it.w[j] >> 8 : it.w[j] & 0xFFFFFFu;
        else c[j] = it.w[j];
    }
}

// amplitude code of group j of an item
__device__ inline uint32_t item_code(const fast8_launch &f, const item_t &it, int gbase, int j)
{
    const uint32_t pos = (uint32_t)(gbase + kWave * j) * (uint32_t)f.scale_bits;
    return (it.a[j] >> (pos & 31u)) & ((1u << f.scale_bits) - 1u);
}

// The fused product writes nothing per group, so there a lane takes four NEIGHBOURING groups
// (4*lane .. 4*lane+3 of its wave's 256): their 24-bit indices are three aligned dwords and their
// amplitude codes sit in one word, two loads per row instead of eight.
template <bool CODES>
struct quad_item_t {
    uint32_t w[3];                       // 24-bit path: three dwords; generic path: unused
    uint32_t c[kGroupsPerLane];          // generic path: the four indices
    float amp[CODES ? 1 : kGroupsPerLane];
    uint32_t codes;                      // CODES: the word that holds the four codes
};

// Per-lane byte offsets into a row of the planes; rows differ only in a wave-uniform base, so the
// loads take a scalar base and these offsets.  Lanes beyond the row's last group read the row's
// first quad: what they decode meets activations of zero.
struct quad_offsets {
    uint32_t index, scale;
};

template <bool CODES, bool B24>
__device__ inline quad_offsets make_quad_offsets(const fast8_launch &f, int g0, bool in_row)
{
    const uint32_t g = in_row ? (uint32_t)g0 : 0u;
    quad_offsets o;
    o.index = B24 ? (g >> 2) * 12u : 0u;
    o.scale = CODES ? ((g * (uint32_t)f.scale_bits) >> 5) * 4u : g * 4u;  // 4 codes never straddle a word
    return o;
}

// The row's planes, addresses that are uniform in the wave.  No arithmetic on loaded data here, so that fetches stay in
// flight until the item is split.  g: the quad's first group.
template <bool CODES, bool B24>
__device__ inline void fetch_quad_at(const fast8_launch &f, const unsigned char *irow, const unsigned char *srow, int g,
                                     const quad_offsets &o, quad_item_t<CODES> &it)
{
    if constexpr (B24) {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(irow + o.index);
        it.w[0] = p[0]; it.w[1] = p[1]; it.w[2] = p[2];
    } else {
        const uint32_t b = (uint32_t)f.index_bits;
#pragma unroll
        for (int j = 0; j < kGroupsPerLane; j++) {
            const uint32_t pos = (uint32_t)(g + j) * b, w0 = pos >> 5, sh = pos & 31;
            uint64_t v = reinterpret_cast<const uint32_t *>(irow)[w0];
            if (sh + b > 32) v |= (uint64_t)reinterpret_cast<const uint32_t *>(irow)[w0 + 1] << 32;
            it.c[j] = (uint32_t)(v >> sh) & (uint32_t)((1ull << b) - 1ull);
        }
    }
    if constexpr (CODES) {
        it.codes = *reinterpret_cast<const uint32_t *>(srow + o.scale);
    } else {
        const float4 v = *reinterpret_cast<const float4 *>(srow + o.scale);
        it.amp[0] = v.x; it.amp[1] = v.y; it.amp[2] = v.z; it.amp[3] = v.w;
    }
}

template <bool CODES, bool B24>
__device__ inline void fetch_quad(const fast8_launch &f, const pvq_decode_args &a, int64_t row, int g0, bool in_row,
                                  const quad_offsets &o, quad_item_t<CODES> &it)
{
    const uint32_t *scale = CODES ? reinterpret_cast<const uint32_t *>(a.scale) + row * a.scale_row_words
                                  : reinterpret_cast<const uint32_t *>(a.scale) + row * a.groups;
    fetch_quad_at<CODES, B24>(f, reinterpret_cast<const unsigned char *>(a.index + row * a.index_row_words),
                              reinterpret_cast<const unsigned char *>(scale), in_row ? g0 : 0, o, it);
}

// What the decoder needs of an item, copied out so that the item's registers can take the next fetch.
template <bool CODES>
struct quad_split_t {
    uint32_t c[kGroupsPerLane];
    uint32_t codes;                      // the four codes, lowest group in the low bits
    float amp[CODES ? 1 : kGroupsPerLane];
};

template <bool CODES, bool B24>
__device__ inline void split_quad(const fast8_launch &f, int g0, const quad_item_t<CODES> &it, quad_split_t<CODES> &q)
{
    q.codes = 0;
    if constexpr (CODES) q.codes = it.codes >> (((uint32_t)g0 * (uint32_t)f.scale_bits) & 31u);
    else {
#pragma unroll
        for (int j = 0; j < kGroupsPerLane; j++) q.amp[j] = it.amp[j];
    }
    if constexpr (B24) {
        q.c[0] = it.w[0] & 0xFFFFFFu;
        q.c[1] = __builtin_amdgcn_alignbit(it.w[1], it.w[0], 24) & 0xFFFFFFu;
        q.c[2] = __builtin_amdgcn_alignbit(it.w[2], it.w[1], 16) & 0xFFFFFFu;
        q.c[3] = it.w[2] >> 8;
    } else {
#pragma unroll
        for (int j = 0; j < kGroupsPerLane; j++) q.c[j] = it.c[j];
    }
}

// amplitude factor of group j without the row normaliser: sqrt(center[q]) or the stored amplitude
template <bool CODES>
__device__ inline float amp_factor(const fast8_launch &f, const quad_split_t<CODES> &q, int j, const float *sqrtc_l)
{
    if constexpr (CODES) {
        const uint32_t code = (q.codes >> (j * f.scale_bits)) & ((1u << f.scale_bits) - 1u);
        return sqrtc_l[code];
    } else {
        return q.amp[j];
    }
}

// v + (v moved across lanes by one data-parallel-primitive pattern); lanes outside ROWS add zero
template <int CTRL, int ROWS = 0xF>
__device__ inline float dpp_add(float v)
{
    const int moved = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false);
    return v + __builtin_bit_cast(float, moved);
}

// Sum over the 64 lanes in a fixed order, valid in lane 63: pairs, quads, eights, rows of 16 (mirror
// patterns), then row 0 into 1 and row 2 into 3, then rows 0..1 into 2..3.  Pure vector-ALU work:
// no LDS traffic, unlike a shuffle butterfly.
__device__ inline float wave_sum_lane63(float v)
{
    v = dpp_add<0xB1>(v);          // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);          // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);         // row_half_mirror
    v = dpp_add<0x140>(v);         // row_mirror
    v = dpp_add<0x142, 0xA>(v);    // row_bcast15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);    // row_bcast31 into rows 2 and 3
    return v;
}

// ---------------------------------------------------------------------------------------------
// y = W_hat x
// ---------------------------------------------------------------------------------------------

// Of a lane's four groups, how many read S0's block entry from LDS when it is fetched a row ahead; the others read it through
// the vector cache, which takes a cycle per lane of such a gather.  28672 x 8192 / 1024 x 8192, all four from the cache (33 M
// accesses a launch, one in nearly every cycle): 55.2 / 9.3 us; one from LDS 55.0 / 9.1, two 55.7 / 9.0, four 57.4 / 9.1.
constexpr int kS0FromLds = 2;

// rows a wave decodes per batch of rows (= how far ahead it fetches), with and without S0 running
// a row ahead (whose state takes the registers of two more fetched rows)
constexpr int kGemvRowsPerWave = 4, kGemvRowsPerWaveAhead = 2;
// partial sums of one batch of rows: 64 (row, slice) pairs x 4 vectors, two buffers
constexpr size_t kPartBytes = 2 * 64 * 4 * sizeof(float);

// Waves are arranged as nsl column slices (256 groups each) x rl row lanes.  Per batch of 4*rl rows
// every wave handles 4 rows of its slice; lanes keep their 32 activations per vector in registers.
// Row sums: fixed-order sum inside the wave, then the slices' partial sums meet in LDS in slice order.
// AMP: 0 = float32 amplitudes, 1 = amplitude codes, 2 = amplitude codes with the fused gain table.
// A single vector: S0 of a wave's next row is started before the current row is decoded (with more vectors the registers
// go to the activations instead).
template <int NB, int AMP, bool B24>
__global__ __launch_bounds__(kGemvThreads) void gemv8_kernel(fast8_launch f, pvq_decode_args a, int b0,
                                                             int nsl, int rl, int rows_per_block)
{
    constexpr bool CODES = AMP != 0, AHEAD = NB == 1;
    constexpr int RI = AHEAD ? kGemvRowsPerWaveAhead : kGemvRowsPerWave;
    // static, so that table offsets fold into the LDS instructions' immediate fields
    __shared__ __align__(16) unsigned char lds[kLdsBytes];
    // the fused gain table replaces the 1/sqrt(n2) table at the end of the blob
    float *sqrtc_l = reinterpret_cast<float *>(lds + (AMP == 2 ? fused_start(f) : f.p.blob_bytes));
    // what the bits of 2^22 + n2 lack to the place of a group's gain (multiples of 16: a code is or-ed into them)
    uint32_t gains_at = f.p.lds_bytes - (kFast8Squares << f.scale_bits);
    const uint32_t invs_at = f.p.invs - kFast8Squares;
    if constexpr (AMP == 2) asm volatile("" : "+v"(gains_at));     // (a vector register: one of an instruction's two constants may be scalar)
    float *part = sqrtc_l + (AMP == 2 ? (fused_rows(f.p) << f.scale_bits) : 256);

    const int64_t r_begin = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r_end = std::min<int64_t>(a.rows, r_begin + rows_per_block);

    const int G = (int)a.groups;
    const int lane = threadIdx.x & (kWave - 1);
    // the wave's number as a scalar, so that row addresses are computed once per wave, not per lane
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int slice = wave % nsl, rowlane = wave / nsl;
    const int g0 = slice * kTileGroups + lane * kGroupsPerLane;
    const bool in_row = g0 < G;
    const int RB = RI * rl;            // rows per batch
    const quad_offsets qo = make_quad_offsets<CODES, B24>(f, g0, in_row);
    const int64_t r_last = r_end - 1;  // rows beyond the range re-read the last one; their sums are dropped

    // first fetches go out before the table copy
    quad_item_t<CODES> item[RI];
    if (r_begin < r_end) {
#pragma unroll
        for (int i = 0; i < RI; i++)
            fetch_quad<CODES, B24>(f, a, std::min<int64_t>(r_begin + i * rl + rowlane, r_last), g0, in_row, qo, item[i]);
    }
    load_tables<AMP == 2>(lds, f, sqrtc_l);
    if (r_begin >= r_end) return;

    uint32_t xr[NB][16];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const uint16_t *xp = reinterpret_cast<const uint16_t *>(a.x) + (int64_t)(b0 + b) * a.ldx + (int64_t)g0 * 8;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (in_row) v = *reinterpret_cast<const uint4 *>(xp + 8 * j);
            xr[b][4 * j] = v.x; xr[b][4 * j + 1] = v.y; xr[b][4 * j + 2] = v.z; xr[b][4 * j + 3] = v.w;
        }
    }

    // S0 runs one row ahead.  Some of its block entries come from the table in device memory, through the vector cache: see
    // kS0FromLds.
    struct ahead_t {
        quad_split_t<CODES> q;
        uint32_t r[kGroupsPerLane];
        pvq_u32x4 b[kGroupsPerLane];
    };
    // takes the item in `slot`, refills the slot with `refill_row`, and starts S0 for the item taken
    auto start_row = [&](int slot, int64_t refill_row, ahead_t &n) {
        split_quad<CODES, B24>(f, g0, item[slot], n.q);
        fetch_quad<CODES, B24>(f, a, std::min<int64_t>(refill_row, r_last), g0, in_row, qo, item[slot]);
        uint32_t addr[kGroupsPerLane];
        pvq_fast8_s0_find<kGroupsPerLane, B24>(lds, f.p, n.q.c, n.r, addr);
#pragma unroll
        for (int j = 0; j < kGroupsPerLane; j++) n.b[j] = *reinterpret_cast<const pvq_u32x4 *>((j < kS0FromLds ? (const unsigned char *)lds : f.blob) + addr[j]);
    };
    ahead_t nx;
    if constexpr (AHEAD) start_row(0, r_begin + RB + rowlane, nx);

    int parity = 0;
    for (int64_t batch = r_begin; batch < r_end; batch += RB) {
        float *pbuf = part + parity * (64 * NB);
#pragma unroll
        for (int i = 0; i < RI; i++) {
            if (batch + i * rl + rowlane > r_last) break;          // (the same for the wave, whose rows end here)
            ahead_t cu;
            if constexpr (AHEAD) {
                cu = nx;
                // the slot after this one holds the next row: of this batch, or (last slot) of the following one
                const int slot = (i + 1) % RI;
                const int64_t held = i + 1 < RI ? batch : batch + RB;
                start_row(slot, held + RB + slot * rl + rowlane, nx);
            } else {
                split_quad<CODES, B24>(f, g0, item[i], cu.q);
                // the same registers take this wave's row of the next batch while the current one is decoded
                fetch_quad<CODES, B24>(f, a, std::min<int64_t>(batch + RB + i * rl + rowlane, r_last), g0, in_row, qo, item[i]);
            }

            uint32_t squares[kGroupsPerLane];
            float dot[kGroupsPerLane][NB];
            // every pair goes into the groups' dot products the moment its stage has found it
            auto emit = [&](int j, int pair, uint32_t w) {
#pragma unroll
                for (int b = 0; b < NB; b++)
                    dot[j][b] = dot2_bf16(w, xr[b][4 * j + pair], pair == 0 ? 0.0f : dot[j][b]);
            };
            if constexpr (AHEAD) pvq_fast8_rest<kGroupsPerLane, B24>(lds, f.p, cu.r, cu.b, emit, squares);
            else pvq_fast8_decode_emit<kGroupsPerLane, B24>(lds, f.p, cu.q.c, emit, squares);
            float acc[NB];
#pragma unroll
            for (int b = 0; b < NB; b++) acc[b] = 0.0f;
            const uint32_t codes4 = cu.q.codes << 2;
#pragma unroll
            for (int j = 0; j < kGroupsPerLane; j++) {
                float gain;
                if constexpr (AMP == 2) {
                    // gain[n2/2][q]: 4 * (n2/2 * 2^bits + q) bytes on, from 2*n2 and the code word shifted left by two
                    const uint32_t code4 = ((codes4 >> (j * f.scale_bits)) & (((1u << f.scale_bits) - 1u) << 2)) | gains_at;
                    gain = *reinterpret_cast<const float *>(lds + ((squares[j] << f.scale_bits) + code4));
                } else {
                    gain = *reinterpret_cast<const float *>(lds + (squares[j] + invs_at)) *
                           amp_factor<CODES>(f, cu.q, j, sqrtc_l);
                }
#pragma unroll
                for (int b = 0; b < NB; b++) acc[b] = fmaf(gain, dot[j][b], acc[b]);
            }
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const float v = wave_sum_lane63(acc[b]);
                if (lane == kWave - 1) pbuf[((i * rl + rowlane) * nsl + slice) * NB + b] = v;
            }
        }
        // one barrier per batch: the next batch writes the other buffer, and a buffer is written
        // again only after the barrier that follows its readers
        __syncthreads();
        if ((int)threadIdx.x < RB * NB) {
            const int rloc = threadIdx.x / NB, b = threadIdx.x % NB;
            const int64_t row = batch + rloc;
            if (row < r_end) {
                float v = 0.0f;
                for (int s = 0; s < nsl; s++) v += pbuf[(rloc * nsl + s) * NB + b];
                if constexpr (CODES) v *= sqrtf(a.rownorm[row]);
                a.y[(int64_t)(b0 + b) * a.ldy + row] = v;
            }
        }
        parity ^= 1;
    }
}

// One vector, no barriers: every wave works alone.  A wave owns the rows  wave, wave + 16, ...  of its
// workgroup's range and takes them slice by slice (a slice = 256 groups, lane l: groups 4l .. 4l+3): all
// its rows of slice 0, then all of slice 1, ...  So the activations in registers are those of one slice
// (16 registers, reloaded when the slice changes), a row's partial sums are added up by the one wave that
// owns the row (its lane 63 adds each slice's sum, formed inside the wave, to a float of its own in LDS, in
// slice order: deterministic), and after the table copy nothing makes the sixteen waves of a unit meet:
// they drift apart, and their table lookups come spread out instead of in bursts after every barrier.
// S0 runs one item ahead, as in gemv8_kernel<1, ., .>.  Rows of whole slices; AMP as in gemv8_kernel.
constexpr int kRowMaxRowsPerWave = 32;   // partial sums in LDS: 16 waves x 32 rows

template <int AMP, bool B24>
__global__ __launch_bounds__(kGemvThreads) void gemv8_row_kernel(fast8_launch f, pvq_decode_args a, int b0,
                                                                 int rows_per_block, int nsl)
{
    constexpr bool CODES = AMP != 0;
    constexpr int kWaves = kGemvThreads / kWave;
    __shared__ __align__(16) unsigned char lds[kLdsBytes];
    float *sqrtc_l = reinterpret_cast<float *>(lds + (AMP == 2 ? fused_start(f) : f.p.blob_bytes));
    // what the bits of 2^22 + n2 lack to the place of a group's gain (multiples of 16: a code is or-ed into them)
    uint32_t gains_at = f.p.lds_bytes - (kFast8Squares << f.scale_bits);
    const uint32_t invs_at = f.p.invs - kFast8Squares;
    if constexpr (AMP == 2) asm volatile("" : "+v"(gains_at));     // (a vector register: one of an instruction's two constants may be scalar)
    float *part = sqrtc_l + (AMP == 2 ? (fused_rows(f.p) << f.scale_bits) : 256);

    const int64_t r_begin = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r_end = std::min<int64_t>(a.rows, r_begin + rows_per_block);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // this wave's rows: r_begin + wave + 16 i, i < nrows; its items: (slice, row) pairs, rows innermost
    const int nrows = r_begin + wave < r_end ? (int)((r_end - r_begin - wave + kWaves - 1) / kWaves) : 0;
    const int nitems = nrows * nsl;
    const int gl = lane * kGroupsPerLane;             // the lane's first group inside a slice
    float *mine = part + wave * kRowMaxRowsPerWave;

    // byte offsets of the lane's quad inside slice 0 of a row of the planes; a slice further on adds a constant
    const quad_offsets q0 = make_quad_offsets<CODES, B24>(f, gl, true);
    const uint32_t scale_step = CODES ? (uint32_t)(kTileGroups / 32) * 4u * (uint32_t)f.scale_bits : (uint32_t)kTileGroups * 4u;
    const int64_t index_bytes = a.index_row_words * 4, scale_bytes = CODES ? a.scale_row_words * 4 : a.groups * 4;

    // the stream of fetches: item after item, rows innermost, (slice, row) and the planes' addresses kept as scalars; past the
    // last item the last one is read again (nothing of it is kept)
    struct place_t { int sl, i; };
    place_t f_at = {0, 0};
    const unsigned char *index0 = reinterpret_cast<const unsigned char *>(a.index) + (r_begin + wave) * index_bytes;
    const unsigned char *scale0 = reinterpret_cast<const unsigned char *>(a.scale) + (r_begin + wave) * scale_bytes;
    const unsigned char *f_index = index0, *f_scale = scale0;
    place_t raw_at[2];
    auto fetch_next = [&](quad_item_t<CODES> &it, place_t &at) {
        at = f_at;
        fetch_quad_at<CODES, B24>(f, f_index, f_scale, f_at.sl * kTileGroups + gl, q0, it);
        if (f_at.i + 1 < nrows) {
            f_at.i++;
            f_index += kWaves * index_bytes;
            f_scale += kWaves * scale_bytes;
        } else if (f_at.sl + 1 < nsl) {
            f_at.i = 0;
            f_at.sl++;
            f_index = index0 + (B24 ? f_at.sl * (kTileGroups * 3) : 0);
            f_scale = scale0 + f_at.sl * (int64_t)scale_step;
        }
    };

    quad_item_t<CODES> raw[2];
    if (nitems > 0) { fetch_next(raw[0], raw_at[0]); fetch_next(raw[1], raw_at[1]); }
    if (lane < kRowMaxRowsPerWave) mine[lane] = 0.0f;
    load_tables<AMP == 2>(lds, f, sqrtc_l);          // ends with the kernel's only barrier before the last one

    if (nitems > 0) {
        struct ahead_t {
            place_t at;
            quad_split_t<CODES> q;
            uint32_t r[kGroupsPerLane];
            pvq_u32x4 b[kGroupsPerLane];
        };
        // takes the raw item out of set `slot`, refills the set from the stream, and starts S0 for the item taken
        auto start_item = [&](int slot, ahead_t &n) {
            n.at = raw_at[slot];
            split_quad<CODES, B24>(f, gl, raw[slot], n.q);      // (a slice's codes are whole words)
            fetch_next(raw[slot], raw_at[slot]);
            uint32_t addr[kGroupsPerLane];
            pvq_fast8_s0_find<kGroupsPerLane, B24>(lds, f.p, n.q.c, n.r, addr);
#pragma unroll
            for (int j = 0; j < kGroupsPerLane; j++) n.b[j] = *reinterpret_cast<const pvq_u32x4 *>((j < kS0FromLds ? (const unsigned char *)lds : f.blob) + addr[j]);
        };
        ahead_t nx;
        start_item(0, nx);
        // lane 63's place behind a row's sum, as a number that the compiler does not know to be 0 there: with one it knows to be
        // the same in all lanes it adds up the lanes' values first, in a loop
        int own = lane - (kWave - 1);
        asm volatile("" : "+v"(own));

        uint32_t xr[16];
        int x_sl = -1;
        for (int it = 0; it < nitems; it += 2) {
#pragma unroll
            for (int h = 0; h < 2; h++) {
                if (it + h < nitems) {
                    ahead_t cu = nx;
                    // (in front of the next item's requests: memory operations complete in order, so the wait for the
                    // activations, which the compiler places before their use whether or not this branch ran, would
                    // otherwise cover those requests too, in every item)
                    if (cu.at.sl != x_sl) {
                        const uint16_t *xp = reinterpret_cast<const uint16_t *>(a.x) + (int64_t)b0 * a.ldx +
                                             (int64_t)(cu.at.sl * kTileGroups + gl) * 8;
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            const uint4 v = *reinterpret_cast<const uint4 *>(xp + 8 * j);
                            xr[4 * j] = v.x; xr[4 * j + 1] = v.y; xr[4 * j + 2] = v.z; xr[4 * j + 3] = v.w;
                        }
                        x_sl = cu.at.sl;
                    }
                    // item it + h + 1 sits in set (h + 1) % 2
                    start_item((h + 1) % 2, nx);
                    uint32_t squares[kGroupsPerLane];
                    float dot[kGroupsPerLane];
                    auto emit = [&](int j, int pair, uint32_t w) {
                        dot[j] = dot2_bf16(w, xr[4 * j + pair], pair == 0 ? 0.0f : dot[j]);
                    };
                    pvq_fast8_rest<kGroupsPerLane, B24>(lds, f.p, cu.r, cu.b, emit, squares);
                    float acc = 0.0f;
                    const uint32_t codes4 = cu.q.codes << 2;
#pragma unroll
                    for (int j = 0; j < kGroupsPerLane; j++) {
                        float gain;
                        if constexpr (AMP == 2) {
                            const uint32_t code4 = ((codes4 >> (j * f.scale_bits)) & (((1u << f.scale_bits) - 1u) << 2)) | gains_at;
                            gain = *reinterpret_cast<const float *>(lds + ((squares[j] << f.scale_bits) + code4));
                        } else {
                            gain = *reinterpret_cast<const float *>(lds + (squares[j] + invs_at)) *
                                   amp_factor<CODES>(f, cu.q, j, sqrtc_l);
                        }
                        acc = fmaf(gain, dot[j], acc);
                    }
                    const float v = wave_sum_lane63(acc);
                    // one lane, one address per row, slices in order: a plain sum in a fixed order
                    if (lane == kWave - 1) atomicAdd(&mine[cu.at.i + own], v);
                }
            }
        }
    }
    __syncthreads();
    if (lane < nrows) {
        const int64_t row = r_begin + wave + (int64_t)kWaves * lane;
        const float v = mine[lane];
        a.y[(int64_t)b0 * a.ldy + row] = CODES ? v * sqrtf(a.rownorm[row]) : v;
    }
}

// ---------------------------------------------------------------------------------------------
// Many activation vectors: the dot products on the matrix cores
// ---------------------------------------------------------------------------------------------

// With 3..16 vectors the dot products (8 x 16 multiply-adds per group) outweigh the decoding, and they go
// to the matrix cores as small independent products: v_mfma_f32_4x4x4_16b_bf16 multiplies, in each of the
// 16 blocks of four lanes, a 4 x 4 matrix A (row = lane of the block, 4 values along k per lane) by a 4 x 4
// matrix B (column = lane of the block), and leaves column (lane of the block) of the 4 x 4 result in the
// lane's four result registers.  B is what the decoder hands out: the lane's own pulse vector, small integers
// and therefore exact in bf16, two instructions for its 8 coordinates.  A holds the activations of the same 8
// columns for four vectors; with the instruction's broadcast control (cbsz 2: the blocks of a row of 16 lanes
// all take the A of block `abid` of that row) one load per group, lane (m, kb) fetching vector m, serves all
// sixteen lanes of the row for the vectors 4 abid .. 4 abid + 3.  A lane therefore gets y . x of ITS group for
// four vectors per instruction pair, multiplies by the group's gain (float32, as in the single-vector kernels:
// gain * (y . x), every product y_i x_i exact) and keeps a running sum per vector: four multiply-adds per group
// and four vectors beside the decoding, nothing of the weights is converted or split.
// A wave takes 16 rows x 64 consecutive groups: lane (m, kb) = (lane % 16, lane / 16) decodes the groups
// slab + 16*q + 4*kb + j of row m, quad q = 0..3 after quad (j = 0..3 through the table decoder at once), so
// that the four k-blocks read 16 neighbouring groups (48 contiguous bytes of indices, one word of codes).
// The sums of the lanes and waves that share a row meet at the end of a round: the four k-blocks inside the
// wave, then four waves per phase in LDS, added in wave order (deterministic).
typedef __attribute__((ext_vector_type(4))) short bf16x4_bits_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// y . x for the lane's group and the vectors 4 S .. 4 S + 3 (xlo, xhi: this row of lanes' activations, columns
// 0..3 and 4..7 of the group; ylo, yhi: the lane's pulses)
template <int S>
__device__ inline f32x4_t group_dots(bf16x4_bits_t xlo, bf16x4_bits_t xhi, bf16x4_bits_t ylo, bf16x4_bits_t yhi)
{
    const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const f32x4_t d = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xlo, ylo, zero, 2, S, 0);
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xhi, yhi, d, 2, S, 0);
}

constexpr int kMfmaRows = 16;                 // rows of a tile
constexpr int kMfmaSlab = 64;                 // groups of a row that one wave takes
constexpr int kMfmaSlots = 4;                 // waves whose results meet in LDS at a time
constexpr size_t kMfmaPartBytes = kMfmaSlots * 256 * sizeof(float);

// AMP: 0 = float32 amplitudes, 1 = amplitude codes.  NS = vectors / 4, rounded up.  24-bit indices.
// nslabs = slabs per row.  A workgroup
// owns tiles_per_block consecutive row tiles and takes them in rounds: four tiles at a time while four are
// left (four waves per tile, every wave the slabs slice, slice + 4, ...), then two (eight waves each), then
// one (sixteen waves, or as many as the row has slabs, rounded up to four).  Few, long rounds keep the
// barriers of the reduction and the unhidden first loads of a tile rare.
template <int AMP, int NS>
__global__ __launch_bounds__(kGemvThreads) void gemv8_mfma_kernel(fast8_launch f, pvq_decode_args a, int b0,
                                                                  int nvec, int tiles_per_block, int nslabs)
{
    constexpr bool CODES = AMP != 0;
    constexpr int kWaves = kGemvThreads / kWave;
    __shared__ __align__(16) unsigned char lds[kLdsBytes];
    float *sqrtc_l = reinterpret_cast<float *>(lds + f.p.blob_bytes);
    float *part = sqrtc_l + 256;

    const int64_t r_begin = (int64_t)blockIdx.x * tiles_per_block * kMfmaRows;
    const int64_t r_end = std::min<int64_t>(a.rows, r_begin + (int64_t)tiles_per_block * kMfmaRows);
    const int64_t r_last = r_end - 1;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int m = lane & 15, kb = lane >> 4;
    const uint32_t sb = (uint32_t)f.scale_bits;
    const int nsl_cap = std::min(kWaves, (nslabs + kMfmaSlots - 1) / kMfmaSlots * kMfmaSlots);

    load_tables<false>(lds, f, sqrtc_l);
    if (r_begin >= r_end) return;

    // the other operand: vector m, the 8 columns of the lane's group.  Lanes beyond the vectors given read
    // the last vector again (no condition around the loads); their columns of the result are not stored.
    const uint16_t *xvec = reinterpret_cast<const uint16_t *>(a.x) + (int64_t)(b0 + std::min(m, nvec - 1)) * a.ldx;

    // what a lane reads per four groups: three index words, and the word with the four codes or four floats
    struct quad_t { uint32_t w[3]; uint32_t s[CODES ? 1 : 4]; };
    auto fetch = [&](int64_t row, uint32_t g, quad_t &it) {
        const uint3 iw = *reinterpret_cast<const uint3 *>(a.index + row * a.index_row_words + (g >> 2) * 3u);   // one 12-byte load
        it.w[0] = iw.x; it.w[1] = iw.y; it.w[2] = iw.z;
        if constexpr (CODES) {
            it.s[0] = (reinterpret_cast<const uint32_t *>(a.scale) + row * a.scale_row_words)[(g * sb) >> 5];
        } else {
            const float *sp = reinterpret_cast<const float *>(a.scale) + row * a.groups + g;
#pragma unroll
            for (int j = 0; j < 4; j++) it.s[j] = __float_as_uint(sp[j]);
        }
    };

    const int tiles = (int)((r_end - r_begin + kMfmaRows - 1) / kMfmaRows);
    // a round: rl tiles from t0 on, nsl waves each (uniform in the workgroup); this wave's part of it
    struct round_t { int rl, nsl, nwaves, nq; uint32_t gl0; int64_t row; bool live; };
    auto make_round = [&](int t0) {
        round_t R;
        const int left = tiles - t0;
        R.rl = left >= 4 ? 4 : left >= 2 ? 2 : 1;
        R.nsl = std::min(kWaves / R.rl, nsl_cap);
        R.nwaves = R.nsl * R.rl;
        const int slice = wave % R.nsl, tile = t0 + wave / R.nsl;     // uniform in the wave
        // the lane's groups: slab slice + nsl * pass, there 4 * kb + 16 * q + j; quad number qq = 4 * pass + q
        R.gl0 = (uint32_t)(slice * kMfmaSlab + 4 * kb);
        R.nq = slice < nslabs ? 4 * ((nslabs - slice + R.nsl - 1) / R.nsl) : 0;
        R.live = left > 0 && wave < R.nwaves && tile < tiles && R.nq > 0;
        R.row = std::min<int64_t>(r_begin + (int64_t)tile * kMfmaRows + m, r_last);
        return R;
    };
    round_t R = make_round(0);
    quad_t cur, nxt;
    if (R.live) fetch(R.row, R.gl0, cur);
    for (int t0 = 0; t0 < tiles;) {
        // the first quad of the next round is fetched during the last quad of this one, so that the
        // reduction's barriers do not stand between a wave and its next indices
        const round_t N = make_round(t0 + R.rl);
        const int nsl = R.nsl, nwaves = R.nwaves, nq = R.nq;
        const bool live = R.live;
        auto quad_group = [&](int qq) { return R.gl0 + (uint32_t)((qq >> 2) * nsl * kMfmaSlab + 16 * (qq & 3)); };
        // tot[s][r]: this lane's part of (row m) . (vector 4 s + r)
        f32x4_t tot[4];
#pragma unroll
        for (int v = 0; v < 4; v++) tot[v] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (!live && N.live) fetch(N.row, N.gl0, cur);
        if (live) {
#pragma unroll 1
            for (int q = 0; q < nq; q++) {
                const uint32_t gq = quad_group(q);
                const bool last = q + 1 == nq;
                fetch(last && N.live ? N.row : R.row, last ? (N.live ? N.gl0 : gq) : quad_group(q + 1), nxt);
                // With many vectors the activations' loads are what the vector memory path is busy with.  A lane's own
                // four groups lie side by side, so a load for "group j of every k-block" takes 16 bytes out of every 64;
                // with kSwap the four k-blocks of a row trade decoded groups instead (lane kb gets group kb of lane t for
                // instruction t: a 4 x 4 transposition over the rows of 16 lanes by register pairs trading halves and
                // rows), and instruction t's activations are 64 bytes in a row per vector.
                constexpr bool kSwap = NS >= 3;
                uint4 bx[4];
#pragma unroll
                for (int j = 0; j < 4; j++)
                    bx[j] = *reinterpret_cast<const uint4 *>(xvec + (int64_t)(kSwap ? gq - 4 * kb + 4 * j + kb : gq + j) * 8);
                uint32_t c[4], pr[4][4], squares[4];
                c[0] = cur.w[0] & 0xFFFFFFu;
                c[1] = __builtin_amdgcn_alignbit(cur.w[1], cur.w[0], 24) & 0xFFFFFFu;
                c[2] = __builtin_amdgcn_alignbit(cur.w[2], cur.w[1], 16) & 0xFFFFFFu;
                c[3] = cur.w[2] >> 8;
                pvq_fast8_decode<4, true>(lds, f.p, c, pr, squares);
                const uint32_t codes = CODES ? cur.s[0] >> ((gq * sb) & 31u) : 0u;
                float gains[4];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    float gain = *reinterpret_cast<const float *>(lds + (squares[j] + (f.p.invs - kFast8Squares)));
                    if constexpr (CODES) gain *= sqrtc_l[(codes >> (j * sb)) & ((1u << sb) - 1u)];
                    else gain *= __uint_as_float(cur.s[j]);
                    gains[j] = gain;
                }
                if constexpr (kSwap) {
                    // value j of row kb <-> value kb of row j, for the pulses' four words and the gain
                    auto transpose = [](uint32_t &r0, uint32_t &r1, uint32_t &r2, uint32_t &r3) {
                        auto a = __builtin_amdgcn_permlane32_swap(r0, r2, false, false);
                        auto b = __builtin_amdgcn_permlane32_swap(r1, r3, false, false);
                        auto e = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
                        auto g = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
                        r0 = e[0]; r1 = e[1]; r2 = g[0]; r3 = g[1];
                    };
#pragma unroll
                    for (int w = 0; w < 4; w++) transpose(pr[0][w], pr[1][w], pr[2][w], pr[3][w]);
                    uint32_t g0 = __float_as_uint(gains[0]), g1 = __float_as_uint(gains[1]), g2 = __float_as_uint(gains[2]),
                             g3 = __float_as_uint(gains[3]);
                    transpose(g0, g1, g2, g3);
                    gains[0] = __uint_as_float(g0); gains[1] = __uint_as_float(g1); gains[2] = __uint_as_float(g2);
                    gains[3] = __uint_as_float(g3);
                }
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const float gain = gains[j];
                    const bf16x4_bits_t xlo = __builtin_bit_cast(bf16x4_bits_t, make_uint2(bx[j].x, bx[j].y)),
                                        xhi = __builtin_bit_cast(bf16x4_bits_t, make_uint2(bx[j].z, bx[j].w)),
                                        ylo = __builtin_bit_cast(bf16x4_bits_t, make_uint2(pr[j][0], pr[j][1])),
                                        yhi = __builtin_bit_cast(bf16x4_bits_t, make_uint2(pr[j][2], pr[j][3]));
                    f32x4_t d[4];
                    d[0] = group_dots<0>(xlo, xhi, ylo, yhi);
                    if constexpr (NS > 1) d[1] = group_dots<1>(xlo, xhi, ylo, yhi);
                    if constexpr (NS > 2) d[2] = group_dots<2>(xlo, xhi, ylo, yhi);
                    if constexpr (NS > 3) d[3] = group_dots<3>(xlo, xhi, ylo, yhi);
#pragma unroll
                    for (int v = 0; v < NS; v++) {
#pragma unroll
                        for (int r = 0; r < 4; r++) tot[v][r] = fmaf(gain, d[v][r], tot[v][r]);
                    }
                }
                cur = nxt;
            }
        }
        // The four k-blocks of a row sit in lanes m, m + 16, m + 32, m + 48: two exchanges, in each of which a
        // lane gives away half of the vectors it still holds and adds the partner's part of the half it keeps.
        // Lane (m, kb) ends with the wave's sums of row m for the vectors 4 s .. 4 s + 3, s = 2 (kb & 1) + (kb >> 1).
        f32x4_t fin;
        {
            const bool odd = kb & 1, upper = kb & 2;
            f32x4_t k0, k1;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float keep0 = odd ? tot[2][r] : tot[0][r], keep1 = odd ? tot[3][r] : tot[1][r];
                const float send0 = odd ? tot[0][r] : tot[2][r], send1 = odd ? tot[1][r] : tot[3][r];
                k0[r] = keep0 + __shfl_xor(send0, 16, kWave);
                k1[r] = keep1 + __shfl_xor(send1, 16, kWave);
            }
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float keep = upper ? k1[r] : k0[r], send = upper ? k0[r] : k1[r];
                fin[r] = keep + __shfl_xor(send, 32, kWave);
            }
        }
        const int fin_vec = 4 * (2 * (kb & 1) + (kb >> 1));
        // Phases of four waves (nsl is a multiple of four, so a phase lies within one row tile); thread
        // (tile row, vector) of the first 256 adds them in wave order.
        float sum = 0.0f;
        const int phases = nwaves / kMfmaSlots;
        for (int ph = 0; ph < phases; ph++) {
            if (wave / kMfmaSlots == ph) {
                float *slot = part + (wave % kMfmaSlots) * 256;
                *reinterpret_cast<f32x4_t *>(slot + m * 16 + fin_vec) = fin;
            }
            __syncthreads();
            if (threadIdx.x < 256) {
#pragma unroll
                for (int sidx = 0; sidx < kMfmaSlots; sidx++) sum += part[sidx * 256 + threadIdx.x];
                // the last slices of a row tile: its sums are complete
                if (((ph + 1) * kMfmaSlots) % nsl == 0) {
                    const int otile = t0 + (ph * kMfmaSlots) / nsl;
                    const int64_t orow = r_begin + (int64_t)otile * kMfmaRows + (threadIdx.x >> 4);
                    const int n = threadIdx.x & 15;
                    if (otile < tiles && orow < r_end && n < nvec) {
                        float v = sum;
                        if constexpr (CODES) v *= sqrtf(a.rownorm[orow]);
                        a.y[(int64_t)(b0 + n) * a.ldy + orow] = v;
                    }
                    sum = 0.0f;
                }
            }
            __syncthreads();
        }
        t0 += R.rl;
        R = N;
    }
}

// ---------------------------------------------------------------------------------------------
// decode to a matrix
// ---------------------------------------------------------------------------------------------

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// Where of a wave's 64 groups a lane's is: a store instruction is to write one contiguous KiB.  A group is 16 bytes of 16-bit
// values; of float32 it is 32, which lanes 2i and 2i + 1, with groups i and 32 + i, store together, 16 bytes each
// (28672 x 8192 247 us, 8192 x 8192 71; 16 bytes out of every 32 a lane, in two stores: 301 and 90).
template <int OUT>
__device__ inline int group_place(int lane) { return OUT == PVQ_F32 ? (lane >> 1) + 32 * (lane & 1) : lane; }

// Stores the lanes' groups; g: the lane's group, of G in the row at `out`.
template <int OUT>
__device__ inline void store_group(void *out, int g, int G, int lane, const uint32_t (&pr)[4], float gain)
{
    float v[8];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        v[2 * j] = gain * __uint_as_float(pr[j] << 16);
        v[2 * j + 1] = gain * __uint_as_float(pr[j] & 0xFFFF0000u);
    }
    if constexpr (OUT == PVQ_F32) {
        const bool odd = lane & 1;
        u32x4 first, second;                     // a half of group i, a half of group 32 + i
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint32_t lo = __float_as_uint(v[j]), hi = __float_as_uint(v[4 + j]);
            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(odd ? lo : hi), 0xB1, 0xF, 0xF, false);
            first[j] = odd ? other : lo;
            second[j] = odd ? hi : other;
        }
        const int g0 = odd ? g - 32 : g;
        float *o = reinterpret_cast<float *>(out) + (int64_t)g0 * 8 + 4 * (lane & 1);
        if (g0 < G) *reinterpret_cast<u32x4 *>(o) = first;
        if (g0 + 32 < G) *reinterpret_cast<u32x4 *>(o + 32 * 8) = second;
    } else {
        u32x4 q;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if constexpr (OUT == PVQ_F16) {
                q[j] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v[2 * j]) |
                       ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v[2 * j + 1]) << 16);
            } else {
                // v_cvt_pk_bf16_f32: round to nearest even, two values per instruction
                const f32x2_t pair = {v[2 * j], v[2 * j + 1]};
                q[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2_t));
            }
        }
        if (g < G) *reinterpret_cast<u32x4 *>(reinterpret_cast<uint16_t *>(out) + (int64_t)g * 8) = q;
    }
}

// Wave items = (row, tile of 256 groups).  Items go round robin over all waves of the grid, so that at
// any moment the grid writes one contiguous, advancing window of the output (a few MB) rather than one
// window per block: DRAM pages are then filled by neighbours in time.  A wave fetches one item ahead.
template <int OUT, bool CODES, bool B24>
__global__ __launch_bounds__(kMaxThreads) void decode8_kernel(fast8_launch f, pvq_decode_args a)
{
    // static, so that table offsets fold into the LDS instructions' immediate fields
    __shared__ __align__(16) unsigned char lds[kLdsBytes];
    float *sqrtc_l = reinterpret_cast<float *>(lds + f.p.blob_bytes);
    load_tables<false>(lds, f, sqrtc_l);

    const int G = (int)a.groups;
    const int lane = threadIdx.x & (kWave - 1), place = group_place<OUT>(lane);
    // the wave's number as a scalar, so that rows, tiles and row addresses are computed once per wave
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nwaves = blockDim.x / kWave;
    const uint32_t T = (uint32_t)((a.groups + kTileGroups - 1) / kTileGroups);   // tiles per row
    const int64_t total = a.rows * (int64_t)T;
    const int64_t i_end = total;
    // (row, tile) of this wave's item, advanced by one item of every wave of the grid per step
    // without dividing again
    const int64_t stride = (int64_t)gridDim.x * nwaves;
    const int64_t step_rows = stride / T;
    const uint32_t step_tiles = (uint32_t)(stride % T);
    int64_t item = (int64_t)blockIdx.x * nwaves + wave;
    int64_t row = item / T;
    uint32_t tile = (uint32_t)(item - row * T);

    item_t cur, nxt;
    float cur_rn = 1.0f, nxt_rn = 1.0f;
    bool live = item < i_end;     // uniform in the wave
    if (!live) return;            // (after the table copy's barrier; no barrier follows)
    fetch_item<CODES, B24>(f, a, row, (int)tile * kTileGroups + place, cur);
    if constexpr (CODES) cur_rn = a.rownorm[row];
    while (live) {
        int64_t nrow = row + step_rows;
        uint32_t ntile = tile + step_tiles;
        if (ntile >= T) { ntile -= T; nrow += 1; }
        const bool nlive = item + stride < i_end;
        if (!nlive) { nrow = row; ntile = tile; }     // nothing follows: fetch this item again, unused
        fetch_item<CODES, B24>(f, a, nrow, (int)ntile * kTileGroups + place, nxt);
        if constexpr (CODES) nxt_rn = a.rownorm[nrow];

        const int gbase = (int)tile * kTileGroups + place;
        const float srn = CODES ? sqrtf(cur_rn) : 1.0f;
        uint32_t c[kGroupsPerLane], prs[kGroupsPerLane][4], squares[kGroupsPerLane];
        item_indices<B24>(cur, gbase, c);
        pvq_fast8_decode<kGroupsPerLane, B24>(lds, f.p, c, prs, squares);
#pragma unroll
        for (int j = 0; j < kGroupsPerLane; j++) {
            // amp / sqrt(n2): the amplitude first (sqrt(center) * sqrt(row normaliser), or the stored
            // float), then the tabulated 1/sqrt(n2)
            const float amp = CODES ? sqrtc_l[item_code(f, cur, gbase, j)] * srn : __uint_as_float(cur.a[j]);
            const float gain = amp * *reinterpret_cast<const float *>(lds + (squares[j] + (f.p.invs - kFast8Squares)));
            store_group<OUT>(reinterpret_cast<unsigned char *>(a.W_out) + row * a.ldw * (OUT == PVQ_F32 ? 4 : 2), gbase + kWave * j, G, lane, prs[j], gain);
        }
        cur = nxt; cur_rn = nxt_rn; row = nrow; tile = ntile; live = nlive; item += stride;
    }
}

fast8_launch make_launch(const pvq_ctx *c)
{
    fast8_launch f;
    f.p = c->fast8; f.blob = c->fast8_blob; f.sqrtc = c->sqrtc;
    f.index_bits = c->index_bits; f.scale_bits = c->scale_bits;
    return f;
}

int g_num_cus = 0;

template <int NB>
hipError_t launch_gemv_nb(const fast8_launch &f, const pvq_decode_args &a, int b0, int nsl, int rl,
                          int rows_per_block, dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    const bool b24 = f.index_bits == 24;
    // the fused gain table must fit behind the blob together with the partial-sum buffer
    const size_t fused_bytes = (fused_start(f) - f.p.lds_bytes) + ((size_t)fused_rows(f.p) << f.scale_bits) * 4;
    const bool fused = f.scale_bits > 0 && f.scale_bits <= 2 &&
                       f.p.lds_bytes + fused_bytes + kPartBytes <= (size_t)kLdsBytes;
    const int amp = f.scale_bits == 0 ? 0 : (fused ? 2 : 1);
#define PVQ_GEMV_CASE(AMP, B24) \
    hipLaunchKernelGGL((gemv8_kernel<NB, AMP, B24>), grid, block, lds, s, f, a, b0, nsl, rl, rows_per_block)
    if (amp == 2) { if (b24) PVQ_GEMV_CASE(2, true); else PVQ_GEMV_CASE(2, false); }
    else if (amp == 1) { if (b24) PVQ_GEMV_CASE(1, true); else PVQ_GEMV_CASE(1, false); }
    else { if (b24) PVQ_GEMV_CASE(0, true); else PVQ_GEMV_CASE(0, false); }
#undef PVQ_GEMV_CASE
    return hipGetLastError();
}

template <int OUT>
hipError_t launch_decode_out(const fast8_launch &f, const pvq_decode_args &a, dim3 grid,
                             dim3 block, size_t lds, hipStream_t s)
{
    const bool codes = f.scale_bits > 0, b24 = f.index_bits == 24;
    if (codes && b24) hipLaunchKernelGGL((decode8_kernel<OUT, true, true>), grid, block, lds, s, f, a);
    else if (codes) hipLaunchKernelGGL((decode8_kernel<OUT, true, false>), grid, block, lds, s, f, a);
    else if (b24) hipLaunchKernelGGL((decode8_kernel<OUT, false, true>), grid, block, lds, s, f, a);
    else hipLaunchKernelGGL((decode8_kernel<OUT, false, false>), grid, block, lds, s, f, a);
    return hipGetLastError();
}

}  // namespace

hipError_t pvq_fast8_prepare(void)
{
    static hipError_t once = [] {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&g_num_cus, hipDeviceAttributeMultiprocessorCount, dev);
        return e;
    }();
    return once;
}

bool pvq_fast8_decode_usable(const pvq_ctx *c, const pvq_decode_args &a)
{
    (void)a;
    return c->fast8_blob != nullptr;
}

hipError_t pvq_fast8_launch_decode(const pvq_ctx *c, const pvq_decode_args &a, int out_dtype, hipStream_t s)
{
    const fast8_launch f = make_launch(c);
    const size_t lds = 0;  // the kernels own the whole LDS statically
    const int64_t total = a.rows * ((a.groups + kTileGroups - 1) / kTileGroups);   // wave items
    // every block pays the table copy, so blocks get at least 64 wave items (16K groups) each
    const int64_t want_blocks = std::min<int64_t>(g_num_cus > 0 ? g_num_cus : 256, (total + 63) / 64);
    const int64_t nblocks = std::max<int64_t>(1, want_blocks);
    const dim3 grid((unsigned)nblocks), block(kMaxThreads);
    switch (out_dtype) {
    case PVQ_F32: return launch_decode_out<PVQ_F32>(f, a, grid, block, lds, s);
    case PVQ_F16: return launch_decode_out<PVQ_F16>(f, a, grid, block, lds, s);
    default: return launch_decode_out<PVQ_BF16>(f, a, grid, block, lds, s);
    }
}

namespace {

// rows that a workgroup of gemv8_kernel has at a time, one for each of its waves that share a slice
int row_lanes(const pvq_decode_args &a)
{
    const int nsl = (int)((a.groups + kTileGroups - 1) / kTileGroups);
    return std::max(1, (kGemvThreads / kWave) / nsl);
}

// one launch of the fused product for vectors [b0, b0 + NB)
template <int NB>
hipError_t launch_gemv_pass(const pvq_ctx *c, const pvq_decode_args &a, int b0, hipStream_t s)
{
    const fast8_launch f = make_launch(c);
    const int nsl = (int)((a.groups + kTileGroups - 1) / kTileGroups);
    const int rl = row_lanes(a);
    const size_t lds = 0;  // the kernels own the whole LDS statically
    // Rows in rounds of one for each of a workgroup's row lanes, as many workgroups as there are units: a row of a wave (256 groups) takes
    // 2 us, so a unit without rows costs more than the copy of the tables (whole batches of rows, two or
    // four times as many: 1024 x 8192, 1 / 2 vectors, 8.8 / 13.4 us, now 7.3 / 7.9; 6000 x 5984 15.7 / 21.1, now 14.9 / 15.7).
    const int64_t rounds = (a.rows + rl - 1) / rl;
    const int64_t nblocks = std::max<int64_t>(1, std::min<int64_t>(g_num_cus > 0 ? g_num_cus : 256, rounds));
    const int rows_per_block = (int)(((rounds + nblocks - 1) / nblocks) * rl);
    const dim3 grid((unsigned)((a.rows + rows_per_block - 1) / rows_per_block)), block((unsigned)(kWave * nsl * rl));
    return launch_gemv_nb<NB>(f, a, b0, nsl, rl, rows_per_block, grid, block, lds, s);
}

constexpr size_t kRowPartBytes = (kGemvThreads / kWave) * kRowMaxRowsPerWave * sizeof(float);

// the fused gain table (amplitude codes of at most 2 bits) must fit behind the tables with the partial sums
bool row_fused(const fast8_launch &f)
{
    const size_t fused_bytes = (fused_start(f) - f.p.lds_bytes) + ((size_t)fused_rows(f.p) << f.scale_bits) * 4;
    return f.scale_bits > 0 && f.scale_bits <= 2 && f.p.lds_bytes + fused_bytes + kRowPartBytes <= (size_t)kLdsBytes;
}

// one launch of the barrier-free single-vector kernel for vector b0
hipError_t launch_gemv_row(const pvq_ctx *c, const pvq_decode_args &a, int b0, hipStream_t s)
{
    const fast8_launch f = make_launch(c);
    constexpr int kWaves = kGemvThreads / kWave;
    const int64_t units = g_num_cus > 0 ? g_num_cus : 256;
    // whole rounds of sixteen rows per workgroup, at most 32 rounds (the partial sums' place in LDS)
    const int64_t rounds = (a.rows + kWaves - 1) / kWaves;
    const int64_t nblocks = std::max<int64_t>(std::min<int64_t>(units, rounds), (rounds + kRowMaxRowsPerWave - 1) / kRowMaxRowsPerWave);
    const int rows_per_block = (int)(((rounds + nblocks - 1) / nblocks) * kWaves);
    const dim3 grid((unsigned)((a.rows + rows_per_block - 1) / rows_per_block)), block((unsigned)kGemvThreads);
    const int nsl = (int)(a.groups / kTileGroups);
    const bool b24 = f.index_bits == 24;
    const int amp = f.scale_bits == 0 ? 0 : (row_fused(f) ? 2 : 1);
#define PVQ_ROW_CASE(AMP, B24) \
    hipLaunchKernelGGL((gemv8_row_kernel<AMP, B24>), grid, block, 0, s, f, a, b0, rows_per_block, nsl)
    if (amp == 2) { if (b24) PVQ_ROW_CASE(2, true); else PVQ_ROW_CASE(2, false); }
    else if (amp == 1) { if (b24) PVQ_ROW_CASE(1, true); else PVQ_ROW_CASE(1, false); }
    else { if (b24) PVQ_ROW_CASE(0, true); else PVQ_ROW_CASE(0, false); }
#undef PVQ_ROW_CASE
    return hipGetLastError();
}

}  // namespace

namespace {

// one launch of the matrix-core kernel for vectors [b0, b0 + nvec), nvec <= 16
hipError_t launch_gemv_mfma(const pvq_ctx *c, const pvq_decode_args &a, int b0, int nvec, hipStream_t s)
{
    const fast8_launch f = make_launch(c);
    const int nslabs = (int)(a.groups / kMfmaSlab);
    const int64_t tiles = (a.rows + kMfmaRows - 1) / kMfmaRows;
    const int64_t nblocks = std::max<int64_t>(1, std::min<int64_t>(g_num_cus > 0 ? g_num_cus : 256, tiles));
    const int tiles_per_block = (int)((tiles + nblocks - 1) / nblocks);
    const dim3 grid((unsigned)((tiles + tiles_per_block - 1) / tiles_per_block)), block((unsigned)kGemvThreads);
#define PVQ_MFMA_CASE(AMP, NS) \
    hipLaunchKernelGGL((gemv8_mfma_kernel<AMP, NS>), grid, block, 0, s, f, a, b0, nvec, tiles_per_block, nslabs)
    const int ns = (nvec + 3) / 4;
    if (f.scale_bits > 0) {
        if (ns == 1) PVQ_MFMA_CASE(1, 1); else if (ns == 2) PVQ_MFMA_CASE(1, 2); else if (ns == 3) PVQ_MFMA_CASE(1, 3); else PVQ_MFMA_CASE(1, 4);
    } else {
        if (ns == 1) PVQ_MFMA_CASE(0, 1); else if (ns == 2) PVQ_MFMA_CASE(0, 2); else if (ns == 3) PVQ_MFMA_CASE(0, 3); else PVQ_MFMA_CASE(0, 4);
    }
#undef PVQ_MFMA_CASE
    return hipGetLastError();
}

// the matrix-core kernel takes 24-bit indices and rows of four or more whole slabs of 64 groups, and needs
// room in LDS for the tables, the amplitude table and four waves' results
bool mfma_usable(const pvq_ctx *c, const pvq_decode_args &a)
{
    return c->index_bits == 24 && a.groups % kMfmaSlab == 0 && a.groups >= 4 * kMfmaSlab && a.groups <= (1 << 20) &&
           a.rows <= ((int64_t)1 << 30) &&
           (size_t)c->fast8.blob_bytes + 256 * sizeof(float) + kMfmaPartBytes <= (size_t)kLdsBytes;
}

// the barrier-free kernel takes rows of whole slices of 256 groups, and pays off when every wave of every
// unit gets a few rows
bool row_usable(const pvq_ctx *c, const pvq_decode_args &a)
{
    const int64_t units = g_num_cus > 0 ? g_num_cus : 256;
    return a.groups % kTileGroups == 0 && a.groups / kTileGroups <= 4096 && a.rows >= units * 16 * 2 &&
           (size_t)c->fast8.blob_bytes + 256 * sizeof(float) + kRowPartBytes <= (size_t)kLdsBytes;
}

}  // namespace

// Which products the table decoder can take: rows must fit the waves of one workgroup, at most 16 slices of 256 groups, in
// whole quads.
bool pvq_fast8_gemv_usable(const pvq_ctx *c, const pvq_decode_args &a)
{
    return c->fast8_blob != nullptr && a.groups % kGroupsPerLane == 0 && (a.groups + kTileGroups - 1) / kTileGroups <= kGemvThreads / kWave;
}

// Which of them it takes; the coordinate-by-coordinate decoder (pvq_walk.hip, one pass for up to 16
// vectors) has the others.
//  - The walk takes 1.5 to 2 times as long per group, and a launch of the table decoder 5 us before its first row's 2.  Measured (K = 16, 2-bit
//    codes), table / walk, us:
//           rows x columns   groups         1            2            4            7            8           16 vectors
//         512 x 8192        0.5 M    9.0 /  8.4  13.8 /  8.5  13.9 /  8.5  15.4 /  9.9  15.7 / 10.1  18.5 / 14.1
//        1024 x 8192        1.0 M    9.3 /  8.8  14.0 /  8.8  14.4 /  8.9  15.5 / 10.3  15.8 / 10.5  18.6 / 14.6
//        1100 x 8192        1.1 M    9.2 / 14.3  13.7 / 14.4  14.2 / 14.4       -       15.8 / 18.6  18.4 / 23.5
//        2816 x 4096        1.4 M    9.2 / 10.4  13.5 / 10.6  11.2 / 10.5       -       11.2 / 13.1  12.3 / 15.3
//         700 x 14336       1.3 M    9.5 / 11.7  13.6 / 11.8  19.2 / 12.1       -       21.4 / 14.9  25.9 / 21.8
//        2048 x 8192        2.1 M    9.7 / 14.6  13.8 / 14.6  14.4 / 15.0  15.5 / 17.3  15.9 / 18.9  18.5 / 24.0
//       14336 x 4096        7.3 M   19.7 / 30.5  22.1 / 30.3  23.4 / 33.6  25.3 / 44.1  26.5 / 46.9  31.5 / 49.9
//    (One and two vectors with gemv8_kernel's rows in whole batches, as it was.)
//  - One and two vectors now: a launch of the table decoder takes 7.0 / 7.5 us where a wave has one row, 1.6 / 2 more for every further one;
//    the walk's time goes by the tiles of four rows that a unit has and by the row's length.  24-bit indices, 2-bit codes, by groups of a row, table / walk:
//        rows              352        440        520        600        640        680        800        896        960        1024       1028       1100       1200       1280       1284       1400
//         512, 1 vector             (1 tile, 1 row a wave)                                          7.0 / 6.9  7.0 / 7.5  7.0 / 7.7  7.1 / 7.5  7.1 / 8.3  7.0 / 7.9  7.2 / 8.8  7.3 / 9.1  7.1 / 8.9
//              2                                                                                    7.6 / 6.9  7.8 / 7.5  7.8 / 7.9  7.7 / 7.7  7.6 / 8.3  7.7 / 8.0  7.8 / 8.9  7.7 / 9.1  7.3 / 8.9
//        1024, 1 vector   (1 tile, 2 rows from 1025 groups on)                                      7.4 / 7.0  7.4 / 7.6  7.4 / 7.8  8.5 / 7.8  8.6 / 8.5  8.6 / 8.3  8.8 / 9.1  8.2 / 9.2  8.3 / 9.1
//              2                                                                                    7.8 / 7.0  7.8 / 7.6  7.9 / 7.9  9.4 / 7.9  9.7 / 8.5  9.7 / 8.3  9.8 / 9.1  8.9 / 9.4  9.1 / 9.2
//        1100, 1 vector  6.9 / 6.3  7.0 / 7.6  7.0 / 7.5  7.1 / 8.5  7.0 / 8.5  7.3 / 10.0 8.5 / 11.8       (2 tiles, 1 row up to 768 groups)
//        1700            7.3 / 6.4  7.2 / 7.7  8.4 / 7.7  8.4 / 8.7  8.8 / 8.7  8.6 / 10.2 8.6 / 11.9       (2 tiles, 1 row up to 512)
//              2         7.5 / 6.5  7.5 / 7.7  9.1 / 7.9  9.1 / 8.8  9.3 / 8.9  9.2 / 10.3 9.5 / 12.0
//        2300, 1 vector  8.3 / 7.9  8.4 / 9.4  8.6 / 10.2 8.6 / 10.7 8.7 / 11.0 8.7 / 12.9 10.7 / 14.7      (3 tiles, 2 rows up to 768)
//              2         9.0 / 8.0  9.2 / 9.6  9.2 / 10.3 9.2 / 10.8 9.2 / 11.1 9.3 / 12.8 11.5 / 14.7
//        2700, 1 vector  8.7 / 7.9  8.6 / 9.5  10.3 / 10.4 10.3 / 10.9 10.4 / 11.2 10.6 / 13.1 10.7 / 14.8  (3 tiles, 2 rows up to 512)
//              2         9.3 / 8.0  9.3 / 9.6  10.8 / 10.6 11.1 / 11.0 11.1 / 11.2 11.2 / 13.1 11.6 / 14.8
//    With float32 amplitudes the walk takes 0.2 to 0.4 us less (440 groups: 2049 rows, two vectors 9.1 / 8.9; 1028: 512 rows 7.6 / 7.4).
//    So the table decoder has rows from 440 groups on where a wave has fewer rows than a unit has tiles (two vectors and more than one row: from 480 on),
//    from 660 on where they are as many and more than one, from 960 (two vectors: 1088) where it is one row and one tile, and from 1280 (1284) where
//    there are more rows than tiles; beyond that (1024 x 8224, one vector, 8.6 / 7.8, but 3073 x 2816 8.4 / 9.5) the lines for other widths of the index, whose fetches
//    take three times as long (1100 x 4096, K = 13: 11.7 / 9.3): one vector from 2^20 groups on, two from 1.5 M.
//  - For 3 to 8 vectors one decoder or the other is ahead by up to 3 us up to 1.5 M groups (1025 x 8704, 8 vectors: 15.7 / 13.6); for 9 and more the
//    table decoder is by 0.2 to 5 us from 2^20 groups on, where the walk has more than one tile of four rows for a unit (1024 rows of 256;
//    1025 x 8704, 11 vectors: 18.1 / 18.3), and behind with fewer rows.
//  - Three vectors and more on rows that the matrix-core kernel does not take would be two passes (4096 x 10720, 3 / 5 / 16
//    vectors: 46 / 55 / 128 against 26 / 28 / 31 us), or one of four, which takes longer than the walk (32.4 / 26.0).
//  - Fewer than 4096 groups and fewer than 8 vectors: the same test states the plan of three passes for 96 x 288 and 7
//    vectors.  It costs what the walk would save there: 6.3 / 3.9 us for one vector, 21 / 4.1 for seven.  gemv8_kernel<4> is
//    kept for these products alone.
bool pvq_fast8_gemv_pays(const pvq_ctx *c, const pvq_decode_args &a)
{
    if (!pvq_fast8_gemv_usable(c, a)) return false;
    const int64_t groups = a.rows * a.groups;
    if (groups < 4096 && a.batch < 8) return true;                 // (the test's plan, not the faster one)
    if (a.batch >= 3 && !mfma_usable(c, a)) return false;
    const int64_t units = g_num_cus > 0 ? g_num_cus : 256;
    const bool tall = a.rows > 4 * units;
    if (c->index_bits == 24 && a.batch <= 2) {
        const int64_t tiles = (a.rows + 4 * units - 1) / (4 * units), rounds = (a.rows + units * row_lanes(a) - 1) / (units * row_lanes(a));
        const bool one = a.batch == 1;
        if (a.groups >= (rounds < tiles ? (one || rounds == 1 ? 440 : 480) : rounds > tiles ? (one ? 1280 : 1284) : tiles > 1 ? 660 : one ? 960 : 1088)) return true;
    }
    return groups >= (a.batch == 1 || (a.batch > 8 && tall) ? 1 << 20 : 3 << 19);
}

// The passes that a product of a.batch vectors is made of, in order: which kernel takes how many vectors.
int pvq_fast8_plan_gemv(const pvq_ctx *c, const pvq_decode_args &a, pvq_gemv_pass *out)
{
    int n = 0, b0 = 0;
    while (b0 < a.batch) {
        const int left = a.batch - b0;
        // 28672 x 8192: 1 vector 54 us on the barrier-free kernel (row batches and partial sums through LDS, 84 when it was 69, remain
        // for short matrices and rows that are not whole slices), 2 vectors 64 us on the vector-ALU kernel; the matrix-core pass
        // takes 67 (3 or 4 vectors) to 95 us (16), so it takes three and more.
        pvq_gemv_pass p;
        if (left >= 3 && mfma_usable(c, a)) p = {PVQ_PASS_MFMA, std::min(left, 16)};
        else if (left >= 4) p = {PVQ_PASS_VALU, 4};
        else if (left >= 2) p = {PVQ_PASS_VALU, 2};
        else if (row_usable(c, a)) p = {PVQ_PASS_VALU_ROWS, 1};
        else p = {PVQ_PASS_VALU, 1};
        out[n++] = p;
        b0 += p.nvec;
    }
    return n;
}

hipError_t pvq_fast8_launch_gemv(const pvq_ctx *c, const pvq_decode_args &a, hipStream_t s)
{
    pvq_gemv_pass plan[16];
    const int n = pvq_fast8_plan_gemv(c, a, plan);
    int b0 = 0;
    for (int i = 0; i < n; i++) {
        const int nvec = plan[i].nvec;
        hipError_t e;
        switch (plan[i].kind) {
        case PVQ_PASS_MFMA: e = launch_gemv_mfma(c, a, b0, nvec, s); break;
        case PVQ_PASS_VALU_ROWS: e = launch_gemv_row(c, a, b0, s); break;
        default:
            e = nvec == 4 ? launch_gemv_pass<4>(c, a, b0, s)
                : nvec == 2 ? launch_gemv_pass<2>(c, a, b0, s) : launch_gemv_pass<1>(c, a, b0, s);
        }
        if (e != hipSuccess) return e;
        b0 += nvec;
    }
    return hipSuccess;
}
