// Device side of the block Walsh-Hadamard transform (Sec. 3.3 Step 1), shared by the rotation kernel and
// by the kernel that quantises activations right after rotating them.  A workgroup of L lanes holds 8L
// consecutive values of a row, 8 per lane; hadamard_stages runs the butterflies a,b -> a+b, a-b over
// strides 1, 2, 4, ..., n/2 in that order (every value of a stage is one rounded sum or difference of two
// values of the stage before, so the schedule does not change the bits).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pvq_hadamard_dev {

// one word of padding per 32: neighbouring groups of lanes that are 64 or 512 words apart fall into
// different banks
__device__ inline uint32_t pad(uint32_t a) { return a + (a >> 5); }

// butterflies over register distance 1, 2, 4 for the first `bits` of them
__device__ inline void stages_in_registers(float (&v)[8], int bits)
{
#pragma unroll
    for (int t = 0; t < 3; t++) {
        if (t < bits) {
            const int h = 1 << t;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                if ((j & h) == 0) {
                    const float a = v[j], b = v[j + h];
                    v[j] = a + b;
                    v[j + h] = a - b;
                }
            }
        }
    }
}

// Signs of 8 columns (a byte each, not zero for -1): bit 7 of every byte.
__device__ inline uint2 sign_bits(uint2 s8)
{
    return make_uint2((((s8.x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | s8.x) & 0x80808080u, (((s8.y & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | s8.y) & 0x80808080u);
}
// float32 value j, and bf16 values 2 j and 2 j + 1 in a word, with those signs
__device__ inline float with_sign(float v, uint2 bits, int j)
{
    return __uint_as_float(__float_as_uint(v) ^ (((j < 4 ? bits.x : bits.y) << (24 - 8 * (j & 3))) & 0x80000000u));
}
__device__ inline uint32_t with_signs(uint32_t pair, uint2 bits, int j)
{
    return pair ^ __builtin_amdgcn_perm(0u, j < 2 ? bits.x : bits.y, j & 1 ? 0x030C020Cu : 0x010C000Cu);
}

// Which 8 consecutive values of a workgroup's 8 L a lane loads (as a lane number), for blocks of 1024 values and more:
// its own, with the lanes of every second quad reversed.  The lane 4 places on in the order of values is then the mirror
// image inside 8 lanes, one lane pattern like the others; the exchange through LDS that follows puts lanes right.
template <int LOG2N>
__device__ inline int load_lane(int lane)
{
    if constexpr (LOG2N > 9) return lane & 4 ? lane ^ 3 : lane;
    else return lane;
}

// One butterfly stage between lanes whose places (in the order of values) differ in bit MASK: the lane whose bit is clear
// holds a and gets a + b, the other holds b and gets a - b.
// MASK 1, 2, 4, 8: the partner's value comes by a lane pattern inside the row of 16 lanes, as the operand of the
// addition: partner + (+-1) v, two instructions a value, of which the multiplication issues at twice the rate.  4: the
// mirror image inside 8 lanes where MIRRORED (load_lane), else two rotations.
// PERMUTE: through the LDS permute unit.
template <int MASK, bool PERMUTE = false, bool MIRRORED = false>
__device__ inline void stage_across_lanes(float (&v)[8], int place)
{
    static_assert(MASK <= 8 || PERMUTE, "16 and 32: stage_across_rows");
    float sign = place & MASK ? -1.0f : 1.0f;
    asm("" : "+v"(sign));                          // (else the product becomes a selection, which issues at half the rate)
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const float own = v[j] * sign;
        const int x = __builtin_bit_cast(int, v[j]);
        int moved;
        if constexpr (PERMUTE && MASK > 2) {
            moved = __builtin_bit_cast(int, __shfl_xor(v[j], MASK, 64));
        } else if constexpr (MASK == 1) {
            moved = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);           // quad_perm [1,0,3,2]
        } else if constexpr (MASK == 2) {
            moved = __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true);           // quad_perm [2,3,0,1]
        } else if constexpr (MASK == 4 && MIRRORED) {
            moved = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true);          // row_half_mirror
        } else if constexpr (MASK == 4) {
            moved = __builtin_amdgcn_update_dpp(0, x, 0x12C, 0xF, 0x5, false);         // row_ror:12 into lanes 0-3, 8-11
            moved = __builtin_amdgcn_update_dpp(moved, x, 0x124, 0xF, 0xA, false);     // row_ror:4 into lanes 4-7, 12-15
        } else {
            moved = __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true);          // row_ror:8
        }
        v[j] = __builtin_bit_cast(float, moved) + own;
    }
}

// The stage between lanes 16 (32) apart: two registers trade places.  v_permlane16_swap exchanges the odd rows of one
// register with the even rows of another (v_permlane32_swap: the upper half of one with the lower half of the other), after
// which every lane holds both partners of a butterfly, one in each register: the register number's bit STRIDE and the
// lane number's bit MASK have changed roles.  KEEP leaves it so; else the same exchange puts sums and differences back.
template <int MASK, int STRIDE, bool KEEP>
__device__ inline void stage_across_rows(float (&v)[8])
{
    static_assert(MASK == 16 || MASK == 32, "rows of 16 lanes, halves of a wave");
    auto trade = [](float &x, float &y) {
        if constexpr (MASK == 16) {
            const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
            x = __uint_as_float(t[0]); y = __uint_as_float(t[1]);
        } else {
            const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
            x = __uint_as_float(t[0]); y = __uint_as_float(t[1]);
        }
    };
#pragma unroll
    for (int j = 0; j < 8; j++) {
        if (j & STRIDE) continue;
        float a = v[j], b = v[j + STRIDE];
        trade(a, b);
        v[j] = a + b;
        v[j + STRIDE] = a - b;
        if constexpr (!KEEP) trade(v[j], v[j + STRIDE]);
    }
}

// Ownership (P, R): the lane holds the 8 values of its chunk whose index differs in bits 3P .. 3P+R-1 (the
// R low bits of the register number) and, for R < 3, in bits 0 .. 2-R (the other bits of the register
// number); the lane number fills the remaining index bits in order.  (0, 3) is 8 consecutive values.
// The index of register q is own_base(lane) | own_offset(q): the two never share a bit, so the padded
// address splits the same way and the register's part is a compile-time constant.
template <int P, int R>
__device__ inline uint32_t own_base(uint32_t lane)
{
    const uint32_t rest = lane << (3 - R);
    return (rest & ((1u << (3 * P)) - 1u)) | ((rest >> (3 * P)) << (3 * P + R));
}
template <int P, int R>
__device__ constexpr uint32_t own_offset(int q)
{
    return ((uint32_t)q >> R) + (((uint32_t)q & ((1u << R) - 1u)) << (3 * P));
}

// Through LDS from ownership (P0, R0) to (P1, R1).  Value i of the chunk always lies at place i of the buffer, so a lane writes where it
// (in a chunk's first exchange: its wave, whose LDS instructions are carried out in order) has read before and nobody else has:
// one buffer and one barrier per exchange are enough.
template <int P0, int R0, int P1, int R1>
__device__ inline void exchange(float (&v)[8], float *buf, uint32_t lane)
{
    float *w = buf + pad(own_base<P0, R0>(lane));
#pragma unroll
    for (int q = 0; q < 8; q++) w[pad(own_offset<P0, R0>(q))] = v[q];
    __syncthreads();
    const float *r = buf + pad(own_base<P1, R1>(lane));
#pragma unroll
    for (int q = 0; q < 8; q++) v[q] = r[pad(own_offset<P1, R1>(q))];
}

// The same to ownership (P1, R1) from where the stages inside a wave leave the values of blocks of 1024 and more: lanes as
// load_lane says, register bit 2 and lane bit 4, and register bit 1 and lane bit 5, with their roles changed.  (The lanes
// of a wave then write 64 words two apart, which all banks share evenly.)
template <int P1, int R1>
__device__ inline void exchange_from_rows(float (&v)[8], float *buf, uint32_t lane)
{
    const uint32_t place = (lane & 4 ? lane ^ 3 : lane) & 15;
    float *w = buf + pad((lane >> 4 & 2) | (lane >> 2 & 4) | place << 3 | (lane >> 6) << 9);
#pragma unroll
    for (int q = 0; q < 8; q++) w[pad((uint32_t)((q & 1) | (q & 4) << 5 | (q & 2) << 7))] = v[q];
    __syncthreads();
    const float *r = buf + pad(own_base<P1, R1>(lane));
#pragma unroll
    for (int q = 0; q < 8; q++) v[q] = r[pad(own_offset<P1, R1>(q))];
}

// All stages of blocks of 2^log2n values (LOG2N = 9: any block of up to 512 values, log2n says which;
// 10 .. 13: that block size).  smem: pad(8 L) + 1 floats when LOG2N > 9.  v: the 8 values of load_lane<LOG2N>(lane).
// STAY: blocks of 1024 and 8192 values end with a single stage, whose ownership (P, 1), P = 3 or 4, still
// has runs of four consecutive values per lane; with STAY the values are left there (register q holds
// column own_base<P,1>(lane) + (q >> 1) + (q & 1) * 8^P of the chunk) instead of going through LDS once
// more.  Otherwise the lane ends with its 8 consecutive values.
// (With a barrier in front of every exchange too, 8192 x 8192 rotated in blocks of 8192 and encoded took 81.3 us with float32 amplitudes
// and 105.5 with 2-bit codes, now 72.0 and 99.0.)
template <int LOG2N, bool STAY, int PERMUTED = 0>
__device__ inline void hadamard_stages(float (&v)[8], int lane, int log2n, float *smem)
{
    if constexpr (LOG2N > 9) log2n = LOG2N;
    constexpr bool kMirrored = LOG2N > 9;
    const int place = load_lane<LOG2N>(lane);
    // index bits 0..2 are the register number, bits 3..8 the lane number inside the wave
    stages_in_registers(v, log2n < 3 ? log2n : 3);
    if (log2n > 3) stage_across_lanes<1>(v, place);
    if (log2n > 4) stage_across_lanes<2>(v, place);
    if (log2n > 5) stage_across_lanes<4, (PERMUTED & 4) != 0 && !kMirrored, kMirrored>(v, place);
    if (log2n > 6) stage_across_lanes<8, (PERMUTED & 8) != 0>(v, place);
    if constexpr (LOG2N > 9) {
        stage_across_rows<16, 4, true>(v);
        stage_across_rows<32, 2, true>(v);
    } else {
        if (log2n > 7) {
            if constexpr ((PERMUTED & 16) != 0) stage_across_lanes<16, true>(v, place);
            else stage_across_rows<16, 1, false>(v);
        }
        if (log2n > 8) {
            if constexpr ((PERMUTED & 32) != 0) stage_across_lanes<32, true>(v, place);
            else stage_across_rows<32, 1, false>(v);
        }
    }
    // from bit 9 on the partners sit in other waves
    if constexpr (LOG2N > 9) {
        constexpr int R3 = LOG2N - 9 < 3 ? LOG2N - 9 : 3;
        constexpr bool kSingleLast = LOG2N == 10 || LOG2N == 13;
        exchange_from_rows<3, R3>(v, smem, lane);
        stages_in_registers(v, R3);
        if constexpr (LOG2N > 12) {
            exchange<3, R3, 4, LOG2N - 12>(v, smem, lane);
            stages_in_registers(v, LOG2N - 12);
            if constexpr (!(STAY && kSingleLast)) exchange<4, LOG2N - 12, 0, 3>(v, smem, lane);
        } else if constexpr (!(STAY && kSingleLast)) {
            exchange<3, R3, 0, 3>(v, smem, lane);
        }
    }
}

}  // namespace pvq_hadamard_dev
