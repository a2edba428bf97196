// pa_sweep.h -- device helpers shared by the sweep kernels: Philox4x32-10, byte
// operations, fences, loops over a replica's lanes and sums over a wave.
#pragma once

#include "pa_device.h"

namespace pa {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t PHILOX_M0 = 0xD2511F53u;
constexpr uint32_t PHILOX_M1 = 0xCD9E8D57u;
constexpr uint32_t PHILOX_W0 = 0x9E3779B9u;
constexpr uint32_t PHILOX_W1 = 0xBB67AE85u;

// Philox4x32-10 (Salmon et al., SC'11), all in registers.  The two xors of
// each output word are one three-input bitop (truth table 0x96 = a ^ b ^ c).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The truth table of a three-input bitop weighs its operands 0xF0, 0xCC, 0xAA.
// Bitwise select m ? a : b.
__device__ __forceinline__ uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, m, 0xE4);
}

// ~a & b.
__device__ __forceinline__ uint32_t and_not(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, 0u, 0x0C);
}

// Rounds 2..10 of Philox after a first round whose product M0 * c0 is given.
__device__ __forceinline__ uint4 philox_from(uint64_t p0, uint32_t c1, uint32_t c2, uint32_t c3,
                                             uint32_t k0, uint32_t k1) {
    {
        const uint64_t p1 = (uint64_t)PHILOX_M1 * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        uint32_t c0 = n0;
        c2 = n2;
        k0 += PHILOX_W0;
        k1 += PHILOX_W1;
#pragma unroll
        for (int r = 1; r < 10; ++r) {
            const uint64_t q0 = (uint64_t)PHILOX_M0 * c0;
            const uint64_t q1 = (uint64_t)PHILOX_M1 * c2;
            const uint32_t m0 = xor3((uint32_t)(q1 >> 32), c1, k0);
            const uint32_t m2 = xor3((uint32_t)(q0 >> 32), c3, k1);
            c1 = (uint32_t)q1;
            c3 = (uint32_t)q0;
            c0 = m0;
            c2 = m2;
            k0 += PHILOX_W0;
            k1 += PHILOX_W1;
        }
        return make_uint4(c0, c1, c2, c3);
    }
}

__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        uint32_t k0, uint32_t k1) {
    return philox_from((uint64_t)PHILOX_M0 * c0, c1, c2, c3, k0, k1);
}

// Digest term of one dword of a replica: r * d mod 2^64, r the 64-bit word of
// Philox(n, k, step, DIGEST) made odd (so any change of d changes the term).
__device__ __forceinline__ uint64_t digest_term(uint32_t n, uint32_t k, uint32_t step, uint32_t d,
                                                uint32_t key0, uint32_t key1) {
    const uint4 w = philox(n, k, step, DOM_DIGEST << 28, key0, key1);
    return ((((uint64_t)w.y << 32) | (uint64_t)w.x) | 1ull) * (uint64_t)d;
}

__device__ __forceinline__ uint32_t mulhi32(uint32_t w, uint32_t n) { return __umulhi(w, n); }

// floor(w * n / 2^32) through the full 32x32->64 multiply: v_mad_u64_u32
// issues at about twice the rate of v_mul_hi_u32 on gfx950, but the compiler
// picks the latter when only the high half is used.
__device__ __forceinline__ uint32_t mulhi32_wide(uint32_t w, uint32_t n) {
    uint64_t prod, carry;
    asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(prod), "=s"(carry) : "v"(w), "s"(n));
    return (uint32_t)(prod >> 32);
}

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);   // byte sel 0-3 from lo, 4-7 from hi
}

// Number of equal bytes between two words.
__device__ __forceinline__ uint32_t eq_bytes(uint32_t a, uint32_t b) {
    const uint32_t x = a ^ b;
    const uint32_t nz = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
    return 4u - __popc(nz);
}

// Philox for the sweep counter (p, k, step, c3) with k, step, c3 and the key
// wave-uniform: the first two rounds are half scalar.  P0 = M0 * p.
struct SweepKey {
    uint32_t n0, n1, c3k1, k0[10], k1[10];
};

__device__ __forceinline__ SweepKey sweep_key(uint32_t k, uint32_t step, uint32_t c3, uint32_t key0,
                                              uint32_t key1) {
    SweepKey s;
    uint32_t a0 = key0, a1 = key1;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        s.k0[r] = a0;
        s.k1[r] = a1;
        a0 += PHILOX_W0;
        a1 += PHILOX_W1;
    }
    const uint64_t p1 = (uint64_t)PHILOX_M1 * step;
    s.n0 = (uint32_t)(p1 >> 32) ^ k ^ key0;
    s.n1 = (uint32_t)p1;
    s.c3k1 = c3 ^ key1;
    return s;
}

__device__ __forceinline__ uint4 philox_sweep(uint64_t P0, const SweepKey &s) {
    // round 1
    const uint32_t a2 = (uint32_t)(P0 >> 32) ^ s.c3k1;
    const uint32_t a3 = (uint32_t)P0;
    // round 2: M0 * n0 is uniform
    const uint64_t q0 = (uint64_t)PHILOX_M0 * s.n0;
    const uint64_t q1 = (uint64_t)PHILOX_M1 * a2;
    uint32_t c0 = (uint32_t)(q1 >> 32) ^ (s.n1 ^ s.k0[1]);
    uint32_t c1 = (uint32_t)q1;
    uint32_t c2 = a3 ^ ((uint32_t)(q0 >> 32) ^ s.k1[1]);
    uint32_t c3 = (uint32_t)q0;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        const uint64_t r0 = (uint64_t)PHILOX_M0 * c0;
        const uint64_t r1 = (uint64_t)PHILOX_M1 * c2;
        const uint32_t m0 = xor3((uint32_t)(r1 >> 32), c1, s.k0[r]);
        const uint32_t m2 = xor3((uint32_t)(r0 >> 32), c3, s.k1[r]);
        c1 = (uint32_t)r1;
        c3 = (uint32_t)r0;
        c0 = m0;
        c2 = m2;
    }
    return make_uint4(c0, c1, c2, c3);
}

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Separates half-sweeps: within one wave LDS operations execute in order, so a
// compiler fence suffices; a replica spread over several waves needs the
// workgroup barrier.
__device__ __forceinline__ void replica_fence(bool multiwave) {
    if (multiwave) __syncthreads();
    else wave_fence();
}

// f(i) for i = g, g + G, ... below n.  With the count and the stride known at
// compile time (NC, GC != 0) the loop has a constant trip count, so that its
// independent iterations (the loads of a gather) issue together.
template <uint32_t NC, uint32_t GC, typename F>
__device__ __forceinline__ void lane_stride(uint32_t g, uint32_t n, uint32_t G, F f) {
    if constexpr (NC != 0 && GC != 0) {
#pragma unroll
        for (uint32_t c = 0; c < (NC + GC - 1) / GC; ++c) {
            const uint32_t i = g + c * GC;
            if (NC % GC == 0 || i < NC) f(i);
        }
    } else {
        for (uint32_t i = g; i < n; i += G) f(i);
    }
}

// Sum over the 64 lanes of a wave (all active), wave-uniform: four DPP adds
// (quad_perm [1,0,3,2] and [2,3,0,1], row_ror 4 and 8) leave every lane of a
// row of 16 with the row's sum; the four row sums are read from lanes 0, 16,
// 32 and 48.
__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);
    return (uint32_t)(__builtin_amdgcn_readlane((int)v, 0) + __builtin_amdgcn_readlane((int)v, 16) +
                      __builtin_amdgcn_readlane((int)v, 32) + __builtin_amdgcn_readlane((int)v, 48));
}

// The same for 4- and 8-byte integers.
__device__ __forceinline__ uint32_t wave_sum_all(uint32_t v) { return wave_total(v); }
__device__ __forceinline__ unsigned long long wave_sum_all(unsigned long long v) {
    for (uint32_t off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Workgroup -> (replica, tile): each XCD takes a contiguous range, so that
// neighbouring tiles of a replica share their halo rows in one L2.
__device__ __forceinline__ void tile_of(uint32_t tiles, uint32_t &k, uint32_t &tile) {
    uint32_t b = blockIdx.x;
    if ((gridDim.x & 7u) == 0) b = (b & 7u) * (gridDim.x >> 3) + (b >> 3);
    k = b / tiles;
    tile = b % tiles;
}

// Index of the segment holding `block`: the last r < n with start[r] <= block
// (start is non-decreasing from start[0] = 0, so segments without workgroups
// are skipped).  Each wave counts the starts not after `block`, 64 per round
// of vector loads, instead of following a chain of dependent loads through a
// binary search; every thread of the workgroup must call it.
__device__ __forceinline__ uint32_t segment_of(const uint32_t *start, uint32_t n, uint32_t block) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t count = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += 64u) {
        const uint32_t i = i0 + lane;
        const bool before = i < n && start[i] <= block;
        count += (uint32_t)__popcll(__ballot(before));
    }
    return __builtin_amdgcn_readfirstlane(count - 1u);
}

}  // namespace

}  // namespace pa
