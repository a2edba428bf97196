// pa_quad.h -- the sweep of replicas held in LDS as two colour planes, four
// sites of one colour per dword ("quads"): q <= 32, lattice sides with a
// compile-time shape (quad_shape).  Part of pa_kernels.hip, which includes it
// inside its namespaces after the helpers it uses.
//
// What bounds it: the issue of vector integer instructions, like the dword
// kernel (sweeps_fixed), so the layout is chosen to need fewer of them.
//   - The plane of colour c holds the sites of that colour row by row, L/2
//     bytes a row.  A dword is four sites whose neighbours are four dwords of
//     the other plane: the same dword (one horizontal neighbour of each), that
//     dword shifted by one byte (the other one; one perm), and the dwords a
//     row above and below.  No neighbour is packed by permutes, and proposals,
//     comparisons and flag sums run on four sites at a time.
//   - A flag (equal / unequal neighbour) is bit 4 (q <= 16) or 5 of its byte,
//     so the eight flags of a site add up in its byte to 16 or 32 times
//     dE + 4, and one dot product with (1, 9) per two sites turns the bytes
//     into the LDS address of their two acceptance thresholds.
//   - A lane updates the same quad of NR replicas: rounds 1-2 of Philox and
//     half of round 3 do not depend on the replica (quad_prefix) and are
//     computed once for all of them; the other half of round 3 depends on
//     neither sweep nor colour and is kept in registers.
// Vector instructions per four attempts: 104 with NR = 4, 107 with 2, 112
// with 1, against 124 of the dword kernel.  Sweep rate on MI355X (q = 10, a
// population of 268 MB, theta = 10), dword kernel / quads with NR = 1 / best
// NR, attempts per ns: 8x8 1263 / 1426 / 1523, 16x16 1269 / 1411 / 1534,
// 24x24 1174 / 1381 / 1424, 32x32 1274 / 1430 / 1511, 48x48 1089 / 1333 / 1377,
// 64x64 1267 / 1422 / 1529, 96x96 1193 / 1386 / 1419, 128x128 (theta = 20)
// 1290 / 1434 / 1475, 192x192 1139 / 1370, 256x256 1182 / 1280.
#pragma once

// Compile-time shape of the quads of lattice side L with G lanes per replica
// (0: none): the largest NR, the waves per SIMD the registers are held to for
// it and for NR = 1, and whether round 3's half is kept in registers.
//   - G is a multiple of L/8 (a lane keeps its quad column) and divides L*L/8.
//   - NR is as large as the registers allow: four words per quad and replica
//     are kept (48 registers for the 8 quads of a lane at 256x256, where they
//     are recomputed instead: 1280 against 1168 attempts/ns with half the
//     waves).
//   - Workgroups of a multiple of four waves: 9- and 6-wave workgroups load
//     the four SIMDs unevenly between barriers (24x24 with 72 lanes in 9
//     waves 1156 attempts/ns, 24 lanes in 12 waves 1424; 96x96 with 384 lanes
//     in 6 waves 1156, in 12 waves 1419).
//   - nr_waves: NR > 1 is used from launches of that many waves (counted with
//     one replica per lane) on, four rounds of the GPU's 8192 wave slots, or
//     twelve where 12-wave workgroups make the last round coarser (NR = 1 /
//     largest, attempts per ns at theta = 10: 32x32 1142 / 1085 with 16000
//     waves, 1250 / 1242 with 32000, 1336 / 1343 with 64000, and the same for
//     8x8, 16x16 and 64x64; 96x96 1257 / 1194 with 32000, 1325 / 1320 with
//     64000).
struct QuadShape { uint32_t max_nr, nr_waves, wpe_max, wpe_one; bool hoist; };
constexpr QuadShape quad_shape(uint32_t L, uint32_t G) {
    if (L == 8 && G == 8) return {4, 32768, 7, 8, true};
    if (L == 16 && G == 32) return {4, 32768, 6, 8, true};
    if (L == 24 && G == 24) return {2, 98304, 6, 8, true};
    if (L == 32 && G == 128) return {4, 32768, 8, 8, true};
    if (L == 48 && G == 96) return {2, 98304, 6, 6, true};
    if (L == 64 && G == 512) return {4, 32768, 8, 8, true};
    if (L == 96 && G == 384) return {2, 98304, 6, 6, true};
    if (L == 128 && G == 1024) return {2, 24576, 8, 8, true};
    if (L == 128 && G == 512) return {1, 0, 8, 8, true};
    if (L == 192 && G == 768) return {1, 0, 6, 6, true};
    if (L == 256 && G == 1024) return {1, 0, 8, 8, false};
    return {0, 0, 0, 0, false};
}

// Threshold table: entry (i0, i1), i = dE + 4 of two sites, holds both 32-bit
// thresholds (as in load_thresholds) at byte UNIT * (i0 + 9 i1), UNIT the value
// of a flag; the UNIT / 8 copies in the gaps serve the lanes in turn, which
// spreads equal entries over the banks.
__host__ __device__ constexpr uint32_t quad_unit(uint32_t q) { return q <= 16u ? 16u : 32u; }
__host__ __device__ constexpr uint32_t quad_tab_bytes(uint32_t q) { return 81u * quad_unit(q); }

// LDS of a workgroup: its replicas (N bytes each), the sums of replicas that
// are not inside one wave (digest 8 bytes, bonds and q_counters state counts
// 4 bytes each per replica), the threshold table.
__host__ __device__ inline uint32_t quad_tab_off(uint32_t N, uint32_t G, uint32_t rpb, uint32_t q_counters) {
    const uint32_t sums = 64u % G != 0 ? rpb * (12u + 4u * q_counters) : 0u;
    return (rpb * N + sums + 15u) & ~15u;
}

// Rounds 1-2 of Philox and the half of round 3 that do not depend on the
// replica: the counter is (p, k, step, c3), and k enters only word 2 of round 2.
struct QuadPrefix {
    uint32_t q1_lo;
    uint64_t r0;
};

__device__ __forceinline__ QuadPrefix quad_prefix(uint32_t P0_hi, uint32_t c3k1, const SweepKey &s) {
    const uint64_t q1 = (uint64_t)PHILOX_M1 * (P0_hi ^ c3k1);
    const uint32_t c0 = (uint32_t)(q1 >> 32) ^ (s.n1 ^ s.k0[1]);
    return QuadPrefix{(uint32_t)q1, (uint64_t)PHILOX_M0 * c0};
}

// Rounds 3 (rest) to 10.  r1: the other product of round 3, which depends on
// the pair and the replica only (r1k: its high word xor the round key); c3k:
// word 3 after round 2 xor the second key of round 3.
__device__ __forceinline__ uint4 quad_rounds(const QuadPrefix &f, uint32_t r1_lo, uint32_t r1k, uint32_t c3k,
                                             const SweepKey &s) {
    uint32_t c0 = r1k ^ f.q1_lo, c1 = r1_lo;
    uint32_t c2 = (uint32_t)(f.r0 >> 32) ^ c3k, c3 = (uint32_t)f.r0;
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        const uint64_t x0 = (uint64_t)PHILOX_M0 * c0;
        const uint64_t x1 = (uint64_t)PHILOX_M1 * c2;
        const uint32_t m0 = xor3((uint32_t)(x1 >> 32), c1, s.k0[r]);
        const uint32_t m2 = xor3((uint32_t)(x0 >> 32), c3, s.k1[r]);
        c1 = (uint32_t)x1;
        c3 = (uint32_t)x0;
        c0 = m0;
        c2 = m2;
    }
    return make_uint4(c0, c1, c2, c3);
}

// Flags (UNIT per byte) of the unequal / equal bytes of a and b, all below UNIT.
template <uint32_t UNIT>
__device__ __forceinline__ uint32_t quad_ne(uint32_t a, uint32_t b) {
    return ((a ^ b) + (UNIT - 1u) * 0x01010101u) & (UNIT * 0x01010101u);
}
template <uint32_t UNIT>
__device__ __forceinline__ uint32_t quad_eq(uint32_t a, uint32_t b) {
    return and_not((a ^ b) + (UNIT - 1u) * 0x01010101u, UNIT * 0x01010101u);
}

// Metropolis update (proposal and acceptance as in the header comment of pa.h)
// of the four sites of D, one per byte.  N0 .. N3: their neighbours, one dword
// per direction.  wa, wb: the Philox blocks of sites 0-1 and 2-3.  base: LDS
// byte address of the lane's copy of the threshold table.
template <uint32_t UNIT>
__device__ __forceinline__ uint32_t update_quad(uint32_t D, uint32_t N0, uint32_t N1, uint32_t N2, uint32_t N3,
                                                uint4 wa, uint4 wb, uint32_t qm1, uint32_t base) {
    const uint32_t r0 = mulhi32_wide(wa.x, qm1), r1 = mulhi32_wide(wa.z, qm1);
    const uint32_t r2 = mulhi32_wide(wb.x, qm1), r3 = mulhi32_wide(wb.z, qm1);
    // R = r + 0x80 per byte; bit 7 of R - D: r >= s; P = r + (r >= s)
    const uint32_t R = __builtin_amdgcn_bitop3_b32(perm(r1, r0, 0x0C0C0400u), perm(r3, r2, 0x04000C0Cu),
                                                   0x80808080u, 0xFE);
    const uint32_t P = (R ^ 0x80808080u) + (((R - D) >> 7) & 0x01010101u);
    // #unequal(proposed) + #equal(current) = 4 + dE, times UNIT, per byte: up
    // to 128 for q <= 16; for q <= 32 the two halves stay apart (each up to 128)
    uint32_t p = quad_ne<UNIT>(N0, P) + quad_ne<UNIT>(N1, P) + quad_ne<UNIT>(N2, P);
    uint32_t at01 = base, at23 = base;
    if constexpr (UNIT <= 16u) {
        p = p + quad_ne<UNIT>(N3, P) + quad_eq<UNIT>(N0, D);
        p = p + quad_eq<UNIT>(N1, D) + quad_eq<UNIT>(N2, D);
        p = p + quad_eq<UNIT>(N3, D);
    } else {
        p = p + quad_ne<UNIT>(N3, P);
        uint32_t s = quad_eq<UNIT>(N0, D) + quad_eq<UNIT>(N1, D) + quad_eq<UNIT>(N2, D);
        s = s + quad_eq<UNIT>(N3, D);
        at01 = __builtin_amdgcn_udot4(s, 0x00000901u, at01, false);
        at23 = __builtin_amdgcn_udot4(s, 0x09010000u, at23, false);
    }
    at01 = __builtin_amdgcn_udot4(p, 0x00000901u, at01, false);
    at23 = __builtin_amdgcn_udot4(p, 0x09010000u, at23, false);
    const u32x2 Ta = *(const __attribute__((address_space(3))) u32x2 *)(uintptr_t)at01;
    const u32x2 Tb = *(const __attribute__((address_space(3))) u32x2 *)(uintptr_t)at23;
    // byte i of D becomes byte i of P where w <= T (SDWA: the select reads and
    // writes one byte); a compare's VCC is read two wait states later
    asm("v_cmp_le_u32 vcc, %[w0], %[t0]\n\t"
        "s_nop 1\n\t"
        "v_cndmask_b32_sdwa %[D], %[D], %[P], vcc dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_0 src1_sel:BYTE_0\n\t"
        "v_cmp_le_u32 vcc, %[w1], %[t1]\n\t"
        "s_nop 1\n\t"
        "v_cndmask_b32_sdwa %[D], %[D], %[P], vcc dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_1 src1_sel:BYTE_1"
        : [D] "+v"(D)
        : [w0] "v"(wa.y), [t0] "v"(Ta.x), [w1] "v"(wa.w), [t1] "v"(Ta.y), [P] "v"(P)
        : "vcc");
    asm("v_cmp_le_u32 vcc, %[w0], %[t0]\n\t"
        "s_nop 1\n\t"
        "v_cndmask_b32_sdwa %[D], %[D], %[P], vcc dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_2 src1_sel:BYTE_2\n\t"
        "v_cmp_le_u32 vcc, %[w1], %[t1]\n\t"
        "s_nop 1\n\t"
        "v_cndmask_b32_sdwa %[D], %[D], %[P], vcc dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_3 src1_sel:BYTE_3"
        : [D] "+v"(D)
        : [w0] "v"(wb.y), [t0] "v"(Tb.x), [w1] "v"(wb.w), [t1] "v"(Tb.y), [P] "v"(P)
        : "vcc");
    return D;
}

// theta sweeps of the NR replicas k[] at lds32 (N bytes each).  Quad qd =
// g + j G of a lane is row qd / (L/8), dword qd mod (L/8) of a plane, and takes
// Philox pairs 2 qd and 2 qd + 1.
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__device__ __forceinline__ void sweeps_quad(uint32_t *lds32, uint32_t g, const uint32_t (&k)[NR], const SweepArgs &a,
                                            uint32_t base, uint32_t theta) {
    constexpr uint32_t L = LT, N = L * L, DPQ = L / 8, G = GT, NQ = N / 8;
    constexpr uint32_t PPQ = NQ / G, RS = G / DPQ;         // quads per lane, rows between them
    constexpr uint32_t PLANE = L * DPQ, REP = 2 * PLANE;   // dwords of a plane and of a replica
    constexpr bool HOIST = quad_shape(L, G).hoist;
    static_assert(G % DPQ == 0 && NQ % G == 0 && (PPQ == 1 || RS % 2 == 0), "shape");
    const uint32_t d = g % DPQ, y0 = g / DPQ;
    const uint32_t left = d == 0 ? g + (DPQ - 1) : g - 1, right = d == DPQ - 1 ? g - (DPQ - 1) : g + 1;
    // the rows above the lane's first and below its last quad (periodic);
    // between them a neighbour is a row away
    const uint32_t up0 = y0 == 0 ? g + (L - 1) * DPQ : g - DPQ;
    constexpr uint32_t LAST = (PPQ - 1) * G;
    const uint32_t dn1 = y0 + (PPQ - 1) * RS == L - 1 ? d : g + LAST + DPQ;
    const bool odd = (y0 & 1u) != 0;
    const uint32_t qm1 = a.q - 1u;
    constexpr uint32_t PH = HOIST ? PPQ : 1, NH = HOIST ? NR : 1;
    uint32_t hi[PPQ][2], r1_lo[PH][NH][2], r1k[PH][NH][2], c3k[NR], u2[NR];
    const uint32_t lo0 = PHILOX_M0 * (2u * g);
    const SweepKey key = sweep_key(0, a.step, 0, a.key0, a.key1);   // (k and c3 enter below)
#pragma unroll
    for (uint32_t j = 0; j < PPQ; ++j)
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) hi[j][h] = (uint32_t)(((uint64_t)PHILOX_M0 * (2u * (g + j * G) + h)) >> 32);
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r) {
        const uint64_t q0 = (uint64_t)PHILOX_M0 * (key.n0 ^ k[r]);
        c3k[r] = (uint32_t)q0 ^ key.k1[2];
        u2[r] = (uint32_t)(q0 >> 32) ^ key.k1[1];
        if constexpr (HOIST) {
#pragma unroll
            for (uint32_t j = 0; j < PPQ; ++j)
#pragma unroll
                for (uint32_t h = 0; h < 2; ++h) {
                    const uint64_t r1 = (uint64_t)PHILOX_M1 * ((PHILOX_M0 * (2u * (g + j * G) + h)) ^ u2[r]);
                    r1_lo[j][r][h] = (uint32_t)r1;
                    r1k[j][r][h] = (uint32_t)(r1 >> 32) ^ key.k0[2];
                }
        }
    }
    for (uint32_t t = 0; t < theta; ++t) {
#pragma unroll   // both colours in one body: plane offsets stay constants
        for (uint32_t c = 0; c < 2u; ++c) {
            const uint32_t c3k1 = ((DOM_SWEEP << 28) | (t << 1) | c) ^ a.key1;
            // (y + c) even: the sites are at even x, the same dword of the
            // other plane holds their right neighbours and the shifted one,
            // from the dword to the left, their left ones; odd: the reverse
            const bool par = odd != (c != 0);
            const uint32_t adj = par ? right : left, sel = par ? 0x04030201u : 0x02010007u;
            const uint32_t po = c * PLANE, pp = PLANE - po;   // own and other plane
#pragma unroll
            for (uint32_t j = 0; j < PPQ; ++j) {
                const QuadPrefix f0 = quad_prefix(hi[j][0], c3k1, key), f1 = quad_prefix(hi[j][1], c3k1, key);
#pragma unroll
                for (uint32_t r = 0; r < NR; ++r) {
                    uint32_t *own = lds32 + r * REP + po + j * G;
                    const uint32_t *opp = lds32 + r * REP + pp + j * G;
                    const uint32_t D = own[g], A = opp[g], Ax = opp[adj];
                    const uint32_t U = j == 0 ? opp[up0] : (opp - DPQ)[g];
                    const uint32_t Dn = j == PPQ - 1 ? (opp - LAST)[dn1] : (opp + DPQ)[g];
                    uint32_t la, ka, lb, kb;
                    if constexpr (HOIST) {
                        la = r1_lo[j][r][0]; ka = r1k[j][r][0];
                        lb = r1_lo[j][r][1]; kb = r1k[j][r][1];
                    } else {
                        uint32_t lo = lo0 + PHILOX_M0 * (2u * j * G);
                        asm("" : "+v"(lo));        // recomputed per half-sweep, not kept
                        const uint64_t ra = (uint64_t)PHILOX_M1 * (lo ^ u2[r]);
                        const uint64_t rb = (uint64_t)PHILOX_M1 * ((lo + PHILOX_M0) ^ u2[r]);
                        la = (uint32_t)ra; ka = (uint32_t)(ra >> 32) ^ key.k0[2];
                        lb = (uint32_t)rb; kb = (uint32_t)(rb >> 32) ^ key.k0[2];
                    }
                    const uint4 wa = quad_rounds(f0, la, ka, c3k[r], key);
                    const uint4 wb = quad_rounds(f1, lb, kb, c3k[r], key);
                    own[g] = update_quad<UNIT>(D, perm(Ax, A, sel), A, U, Dn, wa, wb, qm1, base);
                }
            }
            replica_fence(64u % G != 0u);
        }
    }
}

// One workgroup `block` of a quad sweep launch: gather or create its replicas,
// theta sweeps, energies (and M~), store, as sweep_body does.  The workgroup
// holds blockDim / G groups of G lanes, each NR replicas with consecutive
// slots.
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__device__ __forceinline__ void sweep_quad_body(const SweepArgs &a, uint32_t block) {
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr uint32_t L = LT, N = L * L, G = GT, NQ = N / 8, HB = N / 2;   // HB: bytes of a plane
    constexpr bool WAVE = 64u % G == 0;          // every replica inside one wave: no workgroup barriers
    const uint32_t tid = threadIdx.x, nthreads = blockDim.x;
    const uint32_t groups = nthreads / G, gi = tid / G, g = tid % G;
    const uint32_t rpb = groups * NR;
    const uint32_t qc = a.Mt_out ? a.q : 0u;

    // sums of replicas spread over waves: digest [rpb] u64, bonds [rpb],
    // per-state counts [rpb][qc] u32
    unsigned long long *acc_d = reinterpret_cast<unsigned long long *>(smem + rpb * N);
    uint32_t *acc_e = reinterpret_cast<uint32_t *>(smem + rpb * N + 8u * rpb);
    uint32_t *acc_m = acc_e + rpb;
    if (!WAVE)
        for (uint32_t t = tid; t < rpb * (3u + qc); t += nthreads) reinterpret_cast<uint32_t *>(acc_d)[t] = 0u;
    const uint32_t tab = quad_tab_off(N, G, rpb, qc);
    for (uint32_t t = tid; t < 81u * (UNIT / 8u); t += nthreads) {
        const uint32_t e = t / (UNIT / 8u), i0 = e % 9u, i1 = e / 9u;
        const uint32_t x = i0 <= 4u ? 0xFFFFFFFFu : (uint32_t)(a.T[i0 - 5u] - 1u);
        const uint32_t y = i1 <= 4u ? 0xFFFFFFFFu : (uint32_t)(a.T[i1 - 5u] - 1u);
        *reinterpret_cast<uint2 *>(smem + tab + 8u * t) = make_uint2(x, y);
    }

    uint32_t k[NR];
    const uint64_t k0 = ((uint64_t)block * groups + gi) * NR;
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r)
        k[r] = G % 64u == 0 ? __builtin_amdgcn_readfirstlane((uint32_t)k0 + r) : (uint32_t)k0 + r;
    auto live = [&](uint32_t r) { return k0 + r < a.R_new; };
    uint8_t *rep0 = smem + (size_t)gi * NR * N;

    // ---- load or create the replicas: site (y, x) is byte x / 2 of row y of
    // the plane of colour (x + y) mod 2
    // W sites from x = W * (o mod L/W) of row o / (L/W) on, as even and odd bytes
    constexpr uint32_t W = L % 16 == 0 ? 16 : 8;
    auto plane_even = [&](uint8_t *rep, uint32_t o) {     // the even-x bytes of chunk o
        const uint32_t y = o / (L / W);
        return rep + (y & 1u) * HB + o * (W / 2);
    };
    auto plane_odd = [&](uint8_t *rep, uint32_t o) {
        const uint32_t y = o / (L / W);
        return rep + (1u - (y & 1u)) * HB + o * (W / 2);
    };
    if (a.mode == SWEEP_UPDATE) {
#pragma unroll
        for (uint32_t r = 0; r < NR; ++r) {
            uint8_t *rep = rep0 + r * N;
            const bool in = live(r);
            const uint32_t src = in ? (a.anc ? a.anc[k[r]] : k[r]) : 0u;
            const uint8_t *gsrc = a.old_pop + (size_t)src * N;
            lane_stride<N / W, G>(g, N / W, G, [&](uint32_t o) {
                if constexpr (W == 16) {
                    const uint4 v = in ? reinterpret_cast<const uint4 *>(gsrc)[o] : make_uint4(0, 0, 0, 0);
                    *reinterpret_cast<uint2 *>(plane_even(rep, o)) =
                        make_uint2(perm(v.y, v.x, 0x06040200u), perm(v.w, v.z, 0x06040200u));
                    *reinterpret_cast<uint2 *>(plane_odd(rep, o)) =
                        make_uint2(perm(v.y, v.x, 0x07050301u), perm(v.w, v.z, 0x07050301u));
                } else {
                    const uint2 v = in ? reinterpret_cast<const uint2 *>(gsrc)[o] : make_uint2(0, 0);
                    *reinterpret_cast<uint32_t *>(plane_even(rep, o)) = perm(v.y, v.x, 0x06040200u);
                    *reinterpret_cast<uint32_t *>(plane_odd(rep, o)) = perm(v.y, v.x, 0x07050301u);
                }
            });
        }
    } else {
#pragma unroll
        for (uint32_t r = 0; r < NR; ++r) {
            uint8_t *rep = rep0 + r * N;
            if (a.mode == SWEEP_INIT_RANDOM) {
                // site n takes word n mod 4 of Philox(n / 4, k, 0, INIT)
                for (uint32_t dd = g; dd < N / 4u; dd += G) {
                    const uint4 w = philox(dd, k[r], 0u, DOM_INIT << 28, a.key0, a.key1);
                    const uint32_t y = dd / (L / 4u);
                    *reinterpret_cast<uint16_t *>(rep + (y & 1u) * HB + 2u * dd) =
                        (uint16_t)(mulhi32(w.x, a.q) | (mulhi32(w.z, a.q) << 8));
                    *reinterpret_cast<uint16_t *>(rep + (1u - (y & 1u)) * HB + 2u * dd) =
                        (uint16_t)(mulhi32(w.y, a.q) | (mulhi32(w.w, a.q) << 8));
                }
            } else {
                // eq. (6): all spins alpha, alpha uniform over the q states
                const uint4 w = philox(0u, k[r], 0u, DOM_GROUND << 28, a.key0, a.key1);
                const uint32_t alpha = mulhi32(w.x, a.q) * 0x01010101u;
                lane_stride<N / 4, G>(g, N / 4u, G,
                                      [&](uint32_t dd) { reinterpret_cast<uint32_t *>(rep)[dd] = alpha; });
            }
        }
    }
    __syncthreads();
    if (WAVE && (uint64_t)block * rpb + (uint64_t)((tid & ~63u) / G) * NR >= a.R_new) return;   // an idle wave

    const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)smem + tab +
                          8u * (tid % (UNIT / 8u));
    const uint32_t theta = a.mode == SWEEP_UPDATE ? a.theta : 0u;
    sweeps_quad<L, G, NR, UNIT>(reinterpret_cast<uint32_t *>(rep0), g, k, a, base, theta);

    // ---- energy (eq. (3)): every bond joins a colour-0 site to a neighbour
    constexpr uint32_t DPQ = L / 8, PLANE = HB / 4;
    auto group_sum = [&](uint32_t v) {           // over the group's lanes inside this wave
        if constexpr (G % 64u == 0) return wave_total(v);
        if constexpr (WAVE) {
#pragma unroll
            for (uint32_t off = G >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        }
        return v;                                // (a group across waves: the lane's own)
    };
    const bool adds = G % 64u != 0 || (tid & 63u) == 0;      // lanes that add to a spread replica's sums
    uint32_t bonds[NR], mt[NR];
    uint64_t dig[NR];
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r) {
        const uint32_t *p0 = reinterpret_cast<const uint32_t *>(rep0 + r * N), *p1 = p0 + PLANE;
        const uint32_t li = gi * NR + r;
        uint32_t ne = 0;
        lane_stride<NQ, G>(g, NQ, G, [&](uint32_t qd) {
            const uint32_t y = qd / DPQ, d = qd % DPQ;
            const uint32_t D = p0[qd], A = p1[qd];
            const uint32_t Ax = p1[(y & 1u) ? (d == DPQ - 1 ? qd - (DPQ - 1) : qd + 1)
                                            : (d == 0 ? qd + (DPQ - 1) : qd - 1)];
            const uint32_t U = p1[y == 0 ? qd + (L - 1) * DPQ : qd - DPQ], Dn = p1[y == L - 1 ? d : qd + DPQ];
            const uint32_t X = perm(Ax, A, (y & 1u) ? 0x04030201u : 0x02010007u);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, A), 0u, ne);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, X), 0u, ne);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, U), 0u, ne);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, Dn), 0u, ne);
        });
        bonds[r] = group_sum(ne / UNIT);         // unequal neighbours; 2N bonds less these are equal
        if (!WAVE && adds) atomicAdd(&acc_e[li], bonds[r]);
        // ---- magnetisation (eq. (5)): the largest number of sites in one state
        mt[r] = 0;
        if (a.Mt_out)
            for (uint32_t st = 0; st < a.q; ++st) {
                uint32_t c = 0;
                lane_stride<N / 4, G>(g, N / 4u, G, [&](uint32_t dd) {
                    c = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(p0[dd], st * 0x01010101u), 0u, c);
                });
                c = group_sum(c / UNIT);
                if (WAVE) mt[r] = max(mt[r], c);
                else if (adds) atomicAdd(&acc_m[li * qc + st], c);
            }
        // ---- digest term (order-free sum over the dwords of four sites of a row)
        dig[r] = 0;
        if (a.H_out) {
            for (uint32_t dd = g; dd < N / 4u; dd += G) {
                const uint8_t *rep = rep0 + r * N;
                const uint32_t y = dd / (L / 4u);
                const uint32_t e = *reinterpret_cast<const uint16_t *>(rep + (y & 1u) * HB + 2u * dd);
                const uint32_t o = *reinterpret_cast<const uint16_t *>(rep + (1u - (y & 1u)) * HB + 2u * dd);
                dig[r] += digest_term(dd, k[r], a.step, perm(o, e, 0x05010400u), a.key0, a.key1);
            }
            if constexpr (WAVE || G % 64u == 0)
                for (uint32_t off = (G < 64u ? G : 64u) >> 1; off > 0; off >>= 1) dig[r] += __shfl_xor(dig[r], off, 64);
            if (!WAVE && adds) atomicAdd(&acc_d[li], (unsigned long long)dig[r]);
        }
    }
    if (!WAVE) __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r) {
        if (!live(r)) continue;
        const uint32_t li = gi * NR + r;
        if (!WAVE) {
            bonds[r] = acc_e[li];
            if (a.Mt_out)
                for (uint32_t st = 0; st < a.q; ++st) mt[r] = max(mt[r], acc_m[li * qc + st]);
            if (a.H_out) dig[r] = acc_d[li];
        }
        if (g == 0) {
            a.E_out[k[r]] = (int32_t)bonds[r] - (int32_t)(2u * N);
            if (a.Mt_out) a.Mt_out[k[r]] = mt[r];
            if (a.H_out) a.H_out[k[r]] = dig[r];
        }
        // streaming stores, as in sweep_body
        uint8_t *rep = rep0 + r * N;
        uint8_t *gdst = a.new_pop + (size_t)k[r] * N;
        lane_stride<N / W, G>(g, N / W, G, [&](uint32_t o) {
            if constexpr (W == 16) {
                const uint2 e = *reinterpret_cast<const uint2 *>(plane_even(rep, o));
                const uint2 d = *reinterpret_cast<const uint2 *>(plane_odd(rep, o));
                const u32x4 v = {perm(d.x, e.x, 0x05010400u), perm(d.x, e.x, 0x07030602u),
                                 perm(d.y, e.y, 0x05010400u), perm(d.y, e.y, 0x07030602u)};
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(gdst) + o);
            } else {
                const uint32_t e = *reinterpret_cast<const uint32_t *>(plane_even(rep, o));
                const uint32_t d = *reinterpret_cast<const uint32_t *>(plane_odd(rep, o));
                const u32x2 v = {perm(d, e, 0x05010400u), perm(d, e, 0x07030602u)};
                __builtin_nontemporal_store(v, reinterpret_cast<u32x2 *>(gdst) + o);
            }
        });
    }
}

constexpr uint32_t quad_wpe(uint32_t L, uint32_t G, uint32_t NR) {
    return NR == 1 ? quad_shape(L, G).wpe_one : quad_shape(L, G).wpe_max;
}

template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 1024), amdgpu_waves_per_eu(quad_wpe(LT, GT, NR))))
k_sweep_quad(SweepArgs a) {
    sweep_quad_body<LT, GT, NR, UNIT>(a, blockIdx.x);
}

// Batched form: run r owns workgroups start[r] .. start[r+1]-1.
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 1024), amdgpu_waves_per_eu(quad_wpe(LT, GT, NR))))
k_sweep_quad_batch(const SweepArgs *runs, const uint32_t *start, uint32_t n) {
    const uint32_t r = segment_of(start, n, blockIdx.x);
    const SweepArgs &a = runs[r];    // by reference: a copy would go to scratch memory
    sweep_quad_body<LT, GT, NR, UNIT>(a, blockIdx.x - start[r]);
}
