// pa_quad.h -- the sweep of replicas held in LDS as two colour planes, four
// sites of one colour per dword ("quads"): q <= 32, the lattice sides 8, 16, 24,
// 32, 48, 64, 96, 128, 192 and 256 with a shape from a table (quad_shape) and,
// with a shape found by rule (quad_any), the even sides from 10 to 254 without
// lane choices.  Sides 12 and 20, whose lane choices have no such shape, and 2,
// 4 and 6 keep the dword and byte kernels.
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

#include "pa_sweep.h"

namespace pa {

namespace {

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
//   - A launch holds its first replicas NR per lane and the last `rounds`
//     rounds of the GPU's wave slots one per lane: the short waves at the end
//     leave fewer slots empty than a last partial round of long ones.  Rate at
//     theta = 10, all one per lane / all NR / mixed so, attempts per ns: 32x32
//     R = 20000 1283 / 1287 / 1315, 50000 1359 / 1406 / 1440; 64x64 4000 1266 /
//     1267 / 1290, 16000 1377 / 1422 / 1450; 16x16 100000 1318 / 1290 / 1380;
//     96x96 5000 1298 / 1333 / 1331, 5333 1257 / 1194; 128x128 2000 1328 / 1358
//     / 1347.  Two rounds, not one and a half, for NR = 2 (96x96 R = 2000: 1186
//     with 36 % of the replicas in pairs, 1250 with none).
struct QuadShape { uint32_t max_nr, wpe_max, wpe_one; bool hoist; };
constexpr QuadShape quad_shape(uint32_t L, uint32_t G) {
    if (L == 8 && G == 8) return {4, 7, 8, true};
    if (L == 16 && G == 32) return {4, 6, 8, true};
    if (L == 24 && G == 24) return {2, 6, 8, true};
    if (L == 32 && G == 128) return {4, 8, 8, true};
    if (L == 48 && G == 96) return {2, 6, 6, true};
    if (L == 64 && G == 512) return {4, 8, 8, true};
    if (L == 96 && G == 384) return {2, 6, 6, true};
    if (L == 128 && G == 1024) return {2, 8, 8, true};
    if (L == 128 && G == 512) return {1, 8, 8, true};
    if (L == 192 && G == 768) return {1, 6, 6, true};
    if (L == 256 && G == 1024) return {1, 8, 8, false};
    return {0, 0, 0, false};
}

// How the rows of a side lie in a plane.  A row has H = L/2 sites of a colour in
// DPQ dwords.  Quads never cross rows, and the pairs of sites that share a
// Philox block (2m and 2m+1 of the colour's sites in row-major order) are
// always the first or second half of one: where H is odd, an odd row starts at
// a second site of a pair and its slots are shifted by one.  Slots outside
// shift .. shift + H - 1 are padding: they hold some spin and are never read as
// a neighbour.
template <uint32_t L, uint32_t G>
struct QuadGeo {
    static constexpr uint32_t H = L / 2, ODD = H & 1u, DPQ = (H + ODD + 3u) / 4u;
    static constexpr bool FULL = H % 4u == 0;                // no padding
    static constexpr uint32_t RS = G / DPQ, J = (L + RS - 1) / RS;   // rows between a lane's quads, quads per lane
    static constexpr uint32_t PLANE = L * DPQ, REP = 2 * PLANE;      // dwords of a plane and of a replica
    static_assert(G % DPQ == 0 && RS <= L && (J == 1 || RS % 2 == 0), "shape");
};
__host__ __device__ constexpr uint32_t quad_rep_bytes(uint32_t L) { return 2u * L * 4u * ((L / 2u + ((L / 2u) & 1u) + 3u) / 4u); }

// The shape of a side without a table entry: RS rows of lanes (even, so that a
// lane's rows have one parity) and workgroups of 4, 8, 12 or 16 waves, chosen
// for the largest share of lane time spent on sites (lanes beyond the last
// whole replica, padding slots and rows past L are lost), less
//   - 3 % for each quad per lane beyond the first, which make waves longer and
//     fewer (50x50, 3001 / 30000 replicas, 8 waves, attempts per ns: 5 quads
//     743 / 1040, 3 quads 877 / 1025), 5 % for a single one (no independent
//     work: 950 at 30000),
//   - 8 % and 12 % for workgroups of 12 and 16 waves, which wait longer at
//     their barriers (100x100, 5003 / 30000 replicas: 16 waves 995 / 1175 with
//     0.92 of the lane time, 8 waves 1053 / 1115 with 0.81),
//   - 5 % beyond 6 quads per lane, where round 3's half is not kept,
// and a part where the registers leave fewer than 24 waves on a compute unit.
// Against the other shapes of a side (16 sides, up to nine shapes each: the next
// scores, and the best of every workgroup size and number of quads), the rule's
// rate over the fastest one's: at 30000 replicas (1 GiB from 206 on) 1.00 at 36,
// 44, 62, 118, 136, 150, 180, 206, 240 and 254, 0.99 at 14, 0.98 at 90, 0.97 at
// 30 and 72, 0.96 at 80, 0.89 at 22; at 3000 replicas 0.98 to 1.00 from 62 on,
// and 0.80 to 0.92 at 22, 30, 36 and 44, where such a launch is one partial
// round and the number of its waves decides.
struct QuadAny { uint32_t G, waves, wpe; bool hoist; };
constexpr QuadAny quad_any(uint32_t L) {
    QuadAny best{0, 0, 0, false};
    if (L < 8 || L > 254 || (L & 1u)) return best;
    const uint32_t H = L / 2, DPQ = (H + (H & 1u) + 3) / 4;
    double best_score = 0.0;
    for (uint32_t w = 4; w <= 16; w += 4)
        for (uint32_t RS = 2; RS <= L; RS += 2) {
            const uint32_t G = RS * DPQ, J = (L + RS - 1) / RS;
            if (G > 64 * w || J > 12) continue;
            const bool hoist = J <= 6;
            const uint32_t wpe = J <= 4 ? 8 : hoist ? 6 : 7;
            const uint32_t reps = 64 * w / G, lds = reps * quad_rep_bytes(L) + 4096;
            uint32_t blocks = 4 * wpe / w;
            if (blocks * lds > 163840) blocks = 163840 / lds;
            if (blocks == 0) continue;
            const double share = (double)(reps * L * H) / (double)(64 * w * J * 4);
            const double score = share * (J == 1 ? 0.95 : 1.0 - 0.03 * (J - 1)) *
                                 (w == 16 ? 0.88 : w == 12 ? 0.92 : 1.0) * (hoist ? 1.0 : 0.95) *
                                 (blocks * w >= 24 ? 1.0 : 0.6 + blocks * w / 60.0);
            if (score > best_score + 1e-9) {
                best_score = score;
                best = QuadAny{G, w, wpe, hoist};
            }
        }
    return best;
}

// Threshold table: entry (i0, i1), i = dE + 4 of two sites, holds both 32-bit
// thresholds (as in load_thresholds) at byte UNIT * (i0 + 9 i1), UNIT the value
// of a flag; the UNIT / 8 copies in the gaps serve the lanes in turn, which
// spreads equal entries over the banks.
__host__ __device__ constexpr uint32_t quad_unit(uint32_t q) { return q <= 16u ? 16u : 32u; }
__host__ __device__ constexpr uint32_t quad_tab_bytes(uint32_t q) { return 81u * quad_unit(q); }

// LDS of a workgroup: its replicas (quad_rep_bytes each), the sums of replicas that
// are not inside one wave (digest 8 bytes, bonds and q_counters state counts
// 4 bytes each per replica), the threshold table.
__host__ __device__ inline uint32_t quad_tab_off(uint32_t L, uint32_t G, uint32_t rpb, uint32_t q_counters) {
    const uint32_t sums = 64u % G != 0 ? rpb * (12u + 4u * q_counters) : 0u;
    return (rpb * quad_rep_bytes(L) + sums + 15u) & ~15u;
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

// Rounds 4 to 10 after round 3's words.
__device__ __forceinline__ uint4 quad_rounds(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, const SweepKey &s) {
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

// Rounds 3 (rest) to 10.  r1: the other product of round 3, which depends on
// the pair and the replica only, whole or as its low word and its high word
// xor the round key; c3k: word 3 after round 2 xor the second key of round 3.
__device__ __forceinline__ uint4 quad_block(const QuadPrefix &f, uint32_t r1_lo, uint32_t r1k, uint32_t c3k,
                                            const SweepKey &s) {
    return quad_rounds(r1k ^ f.q1_lo, r1_lo, (uint32_t)(f.r0 >> 32) ^ c3k, (uint32_t)f.r0, s);
}
__device__ __forceinline__ uint4 quad_block(const QuadPrefix &f, uint64_t r1, uint32_t c3k, const SweepKey &s) {
    return quad_rounds(xor3((uint32_t)(r1 >> 32), f.q1_lo, s.k0[2]), (uint32_t)r1, (uint32_t)(f.r0 >> 32) ^ c3k,
                       (uint32_t)f.r0, s);
}

// Flags (UNIT per byte) of the unequal / equal bytes of a and b, all below UNIT.
template <uint32_t UNIT>
__device__ __forceinline__ uint32_t quad_ne(uint32_t a, uint32_t b, uint32_t mask = UNIT * 0x01010101u) {
    return ((a ^ b) + (UNIT - 1u) * 0x01010101u) & mask;
}
template <uint32_t UNIT>
__device__ __forceinline__ uint32_t quad_eq(uint32_t a, uint32_t b, uint32_t mask = UNIT * 0x01010101u) {
    return and_not((a ^ b) + (UNIT - 1u) * 0x01010101u, mask);
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

// theta sweeps of the NR replicas k[] at lds32 (REP dwords each).  A lane's
// quads are dword d of rows y0, y0 + RS, ... of a plane, dword index g + j G;
// quad (y, d) takes Philox pairs floor(y H / 2) + 2d and the next.  `on`: a
// lane of a replica (lanes beyond the last whole one only meet the barriers).
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT, bool HOIST>
__device__ __forceinline__ void sweeps_quad(uint32_t *lds32, uint32_t g, bool on, const uint32_t (&k)[NR],
                                            const SweepArgs &a, uint32_t base, uint32_t theta) {
    using Geo = QuadGeo<LT, GT>;
    constexpr uint32_t L = LT, G = GT, H = Geo::H, DPQ = Geo::DPQ, J = Geo::J, RS = Geo::RS;
    constexpr uint32_t PLANE = Geo::PLANE, REP = Geo::REP;
    const uint32_t d = g % DPQ, y0 = g / DPQ;
    const bool odd = (y0 & 1u) != 0;
    const uint32_t sh = Geo::ODD && odd ? 1u : 0u;
    // the horizontal neighbours that are not in the same dword of the other
    // plane: to the left (dword left, bytes by sel_l) or to the right; the ends
    // of a row meet (periodic)
    const uint32_t last = (H - 1 + sh) / 4u, lb = (H - 1 + sh) % 4u;       // the last site's dword and byte
    uint32_t left = g - 1, sel_l = 0x02010007u, right = g + 1, sel_r = 0x04030201u;
    if (d == 0) {
        left = g + last;
        sel_l = sh ? 0x02010007u | ((4u + lb) << 8) : 0x02010000u | (4u + lb);
    }
    if (d == last) {
        right = g - last;
        sel_r = (sel_r & ~(0xFFu << (8u * lb))) | ((4u + sh) << (8u * lb));
    }
    // the rows above the lane's first and below its last quad (periodic);
    // between them a neighbour is a row away
    const uint32_t up0 = y0 == 0 ? g + (L - 1) * DPQ : g - DPQ;
    constexpr uint32_t LAST = (J - 1) * G;
    const uint32_t dn1 = y0 + (J - 1) * RS == L - 1 ? d : g + LAST + DPQ;
    // where H is odd, those rows are shifted the other way: their neighbours
    // reach into the next dword (even rows) or the one before
    const uint32_t vs = !Geo::ODD ? 0u : sh ? (d == 0 ? 0u : ~0u) : (d == DPQ - 1 ? 0u : 1u);
    const uint32_t sel_v = sh ? 0x02010007u : 0x04030201u;
    const bool on_last = on && (L % RS == 0 || y0 + (J - 1) * RS < L);
    const uint32_t qm1 = a.q - 1u;
    constexpr uint32_t PH = HOIST ? J : 1, NH = HOIST ? NR : 1;
    uint32_t hi[J][2], r1_lo[PH][NH][2], r1k[PH][NH][2], c3k[NR], u2[NR];
    const uint32_t pair0 = ((y0 * H) >> 1) + 2u * d;
    const uint32_t lo0 = PHILOX_M0 * pair0;
    auto pair = [&](uint32_t j, uint32_t h) { return pair0 + j * (RS * H / 2u) + h; };
    const SweepKey key = sweep_key(0, a.step, 0, a.key0, a.key1);   // (k and c3 enter below)
#pragma unroll
    for (uint32_t j = 0; j < J; ++j)
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) hi[j][h] = (uint32_t)(((uint64_t)PHILOX_M0 * pair(j, h)) >> 32);
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r) {
        const uint64_t q0 = (uint64_t)PHILOX_M0 * (key.n0 ^ k[r]);
        c3k[r] = (uint32_t)q0 ^ key.k1[2];
        u2[r] = (uint32_t)(q0 >> 32) ^ key.k1[1];
        if constexpr (HOIST) {
#pragma unroll
            for (uint32_t j = 0; j < J; ++j)
#pragma unroll
                for (uint32_t h = 0; h < 2; ++h) {
                    const uint64_t r1 = (uint64_t)PHILOX_M1 * ((PHILOX_M0 * pair(j, h)) ^ u2[r]);
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
            const uint32_t adj = par ? right : left, sel = par ? sel_r : sel_l;
            constexpr uint32_t PO[2] = {0, PLANE};
            const uint32_t po = PO[c], pp = PLANE - po;   // own and other plane
#pragma unroll
            for (uint32_t j = 0; j < J; ++j) {
                if (!(j == J - 1 ? on_last : on)) continue;
                const QuadPrefix f0 = quad_prefix(hi[j][0], c3k1, key), f1 = quad_prefix(hi[j][1], c3k1, key);
#pragma unroll
                for (uint32_t r = 0; r < NR; ++r) {
                    uint32_t *own = lds32 + r * REP + po + j * G;
                    const uint32_t *opp = lds32 + r * REP + pp + j * G;
                    const uint32_t D = own[g], A = opp[g], Ax = opp[adj];
                    const uint32_t *up = j == 0 ? opp + up0 : opp - DPQ + g;
                    const uint32_t *dn = j == J - 1 ? opp - LAST + dn1 : opp + DPQ + g;
                    uint32_t U = up[0], Dn = dn[0];
                    if constexpr (Geo::ODD != 0) {
                        U = perm(up[(int32_t)vs], U, sel_v);
                        Dn = perm(dn[(int32_t)vs], Dn, sel_v);
                    }
                    uint4 wa, wb;
                    if constexpr (HOIST) {
                        wa = quad_block(f0, r1_lo[j][r][0], r1k[j][r][0], c3k[r], key);
                        wb = quad_block(f1, r1_lo[j][r][1], r1k[j][r][1], c3k[r], key);
                    } else {
                        uint32_t lo = lo0 + PHILOX_M0 * (j * (RS * H / 2u));
                        asm("" : "+v"(lo));        // recomputed per half-sweep, not kept
                        wa = quad_block(f0, (uint64_t)PHILOX_M1 * (lo ^ u2[r]), c3k[r], key);
                        wb = quad_block(f1, (uint64_t)PHILOX_M1 * ((lo + PHILOX_M0) ^ u2[r]), c3k[r], key);
                    }
                    own[g] = update_quad<UNIT>(D, perm(Ax, A, sel), A, U, Dn, wa, wb, qm1, base);
                }
            }
            replica_fence(64u % G != 0u);
        }
    }
}

// Plane byte of site (y, x) of a replica.
template <uint32_t L>
__device__ __forceinline__ uint8_t *quad_site(uint8_t *rep, uint32_t y, uint32_t x) {
    using Geo = QuadGeo<L, 2 * ((L / 2 + ((L / 2) & 1u) + 3) / 4)>;
    const uint32_t sh = Geo::ODD ? (y & 1u) : 0u;
    return rep + ((x + y) & 1u) * (4u * Geo::PLANE) + y * (4u * Geo::DPQ) + (x >> 1) + sh;
}

// One workgroup `block` of a quad sweep launch: gather or create its replicas,
// theta sweeps, energies (and M~), store, as sweep_body does.  The workgroup
// holds blockDim / G groups of G lanes, each NR replicas with consecutive
// slots, from slot `first` on.  ANY: a side without a table entry (lanes may be
// left over).
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT, bool HOIST, bool ANY>
__device__ __forceinline__ void sweep_quad_body(const SweepArgs &a, uint32_t block, uint32_t first) {
    extern __shared__ __align__(16) uint8_t smem[];
    using Geo = QuadGeo<LT, GT>;
    constexpr uint32_t L = LT, N = L * L, G = GT, DPQ = Geo::DPQ, PLANE = Geo::PLANE;
    constexpr uint32_t REPB = 4 * Geo::REP, PB = 4 * PLANE;   // bytes of a replica and of a plane
    constexpr bool WAVE = 64u % G == 0;          // every replica inside one wave: no workgroup barriers
    const uint32_t tid = threadIdx.x, nthreads = blockDim.x;
    const uint32_t groups = nthreads / G, gi = tid / G, g = tid % G;
    const uint32_t rpb = groups * NR;
    const uint32_t qc = a.Mt_out ? a.q : 0u;
    const bool on = !ANY || gi < groups;

    // sums of replicas spread over waves: digest [rpb] u64, bonds [rpb],
    // per-state counts [rpb][qc] u32
    unsigned long long *acc_d = reinterpret_cast<unsigned long long *>(smem + rpb * REPB);
    uint32_t *acc_e = reinterpret_cast<uint32_t *>(smem + rpb * REPB + 8u * rpb);
    uint32_t *acc_m = acc_e + rpb;
    if (!WAVE)
        for (uint32_t t = tid; t < rpb * (3u + qc); t += nthreads) reinterpret_cast<uint32_t *>(acc_d)[t] = 0u;
    const uint32_t tab = quad_tab_off(L, G, rpb, qc);
    for (uint32_t t = tid; t < 81u * (UNIT / 8u); t += nthreads) {
        const uint32_t e = t / (UNIT / 8u), i0 = e % 9u, i1 = e / 9u;
        const uint32_t x = i0 <= 4u ? 0xFFFFFFFFu : (uint32_t)(a.T[i0 - 5u] - 1u);
        const uint32_t y = i1 <= 4u ? 0xFFFFFFFFu : (uint32_t)(a.T[i1 - 5u] - 1u);
        *reinterpret_cast<uint2 *>(smem + tab + 8u * t) = make_uint2(x, y);
    }

    uint32_t k[NR];
    const uint64_t k0 = first + ((uint64_t)block * groups + gi) * NR;
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r)
        k[r] = G % 64u == 0 ? __builtin_amdgcn_readfirstlane((uint32_t)k0 + r) : (uint32_t)k0 + r;
    auto live = [&](uint32_t r) { return on && k0 + r < a.R_new; };
    uint8_t *rep0 = smem + (size_t)(on ? gi : 0u) * NR * REPB;

    // ---- load or create the replicas: site (y, x) is byte x / 2 (+ shift) of
    // row y of the plane of colour (x + y) mod 2
    // L a multiple of 8: W sites from x = W * (o mod L/W) of row o / (L/W) on, as
    // their even and odd bytes
    constexpr uint32_t W = L % 16 == 0 ? 16 : L % 8 == 0 ? 8 : 4;
    auto plane_even = [&](uint8_t *rep, uint32_t o) {     // the even-x bytes of chunk o
        const uint32_t y = o / (L / W);
        return rep + (y & 1u) * PB + o * (W / 2);
    };
    auto plane_odd = [&](uint8_t *rep, uint32_t o) {
        const uint32_t y = o / (L / W);
        return rep + (1u - (y & 1u)) * PB + o * (W / 2);
    };
    // other L: the four sites of dword o of the replica, two by two (a pair of
    // sites x, x + 1 with x even never crosses a row)
    auto sites2 = [&](uint8_t *rep, uint32_t m, uint8_t *&e, uint8_t *&o) {
        const uint32_t y = m / Geo::H, x = 2u * (m % Geo::H);
        e = quad_site<L>(rep, y, x);
        o = quad_site<L>(rep, y, x + 1u);
    };
    auto put4 = [&](uint8_t *rep, uint32_t dd, uint32_t v) {
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
            uint8_t *e, *o;
            sites2(rep, 2u * dd + h, e, o);
            *e = (uint8_t)(v >> (16u * h));
            *o = (uint8_t)(v >> (16u * h + 8u));
        }
    };
    auto get4 = [&](uint8_t *rep, uint32_t dd) {
        // (two bytes from each plane, on the sides whose launches the digest
        // weighs in: 256x256, R = 3e3, theta = 1 1820 -> 1660 us a run of five steps;
        // at 64x64 nothing, and the batch kernel's sweeps lost 0.8 % with it to
        // another register allocation)
        if constexpr (Geo::FULL && L >= 128) {
            const uint32_t p = dd / (L / 4u) & 1u;
            const uint32_t e = *reinterpret_cast<const uint16_t *>(rep + p * PB + 2u * dd);
            const uint32_t o = *reinterpret_cast<const uint16_t *>(rep + (1u - p) * PB + 2u * dd);
            return perm(o, e, 0x05010400u);
        }
        uint32_t v = 0;
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
            uint8_t *e, *o;
            sites2(rep, 2u * dd + h, e, o);
            v |= ((uint32_t)*e | ((uint32_t)*o << 8)) << (16u * h);
        }
        return v;
    };
    if constexpr (!Geo::FULL) {   // padding slots: some spin
        if (on)
            for (uint32_t o = g; o < 2u * L * NR; o += G) {
                uint8_t *row = rep0 + o * (4u * DPQ);
                const uint32_t sh = Geo::ODD ? ((o % L) & 1u) : 0u;
                if (sh) row[0] = 0;
                for (uint32_t i = sh + Geo::H; i < 4u * DPQ; ++i) row[i] = 0;
            }
    }
    if (a.mode == SWEEP_UPDATE) {
#pragma unroll
        for (uint32_t r = 0; r < NR; ++r) {
            uint8_t *rep = rep0 + r * REPB;
            const bool in = live(r);
            const uint32_t src = in ? (a.anc ? a.anc[k[r]] : k[r]) : 0u;
            const uint8_t *gsrc = a.old_pop + (size_t)src * N;
            if (on)
            lane_stride<N / W, G>(g, N / W, G, [&](uint32_t o) {
                if constexpr (W == 16) {
                    const uint4 v = in ? reinterpret_cast<const uint4 *>(gsrc)[o] : make_uint4(0, 0, 0, 0);
                    *reinterpret_cast<uint2 *>(plane_even(rep, o)) =
                        make_uint2(perm(v.y, v.x, 0x06040200u), perm(v.w, v.z, 0x06040200u));
                    *reinterpret_cast<uint2 *>(plane_odd(rep, o)) =
                        make_uint2(perm(v.y, v.x, 0x07050301u), perm(v.w, v.z, 0x07050301u));
                } else if constexpr (W == 8) {
                    const uint2 v = in ? reinterpret_cast<const uint2 *>(gsrc)[o] : make_uint2(0, 0);
                    *reinterpret_cast<uint32_t *>(plane_even(rep, o)) = perm(v.y, v.x, 0x06040200u);
                    *reinterpret_cast<uint32_t *>(plane_odd(rep, o)) = perm(v.y, v.x, 0x07050301u);
                } else {
                    put4(rep, o, in ? reinterpret_cast<const uint32_t *>(gsrc)[o] : 0u);
                }
            });
        }
    } else if (on) {
#pragma unroll
        for (uint32_t r = 0; r < NR; ++r) {
            uint8_t *rep = rep0 + r * REPB;
            if (a.mode == SWEEP_INIT_RANDOM) {
                // site n takes word n mod 4 of Philox(n / 4, k, 0, INIT)
                for (uint32_t dd = g; dd < N / 4u; dd += G) {
                    const uint4 w = philox(dd, k[r], 0u, DOM_INIT << 28, a.key0, a.key1);
                    put4(rep, dd, mulhi32(w.x, a.q) | (mulhi32(w.y, a.q) << 8) | (mulhi32(w.z, a.q) << 16) |
                                      (mulhi32(w.w, a.q) << 24));
                }
            } else {
                // eq. (6): all spins alpha, alpha uniform over the q states
                const uint4 w = philox(0u, k[r], 0u, DOM_GROUND << 28, a.key0, a.key1);
                const uint32_t alpha = mulhi32(w.x, a.q) * 0x01010101u;
                for (uint32_t dd = g; dd < Geo::REP; dd += G) reinterpret_cast<uint32_t *>(rep)[dd] = alpha;
            }
        }
    }
    __syncthreads();
    if (WAVE && first + (uint64_t)block * rpb + (uint64_t)((tid & ~63u) / G) * NR >= a.R_new) return;   // an idle wave

    const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)smem + tab +
                          8u * (tid % (UNIT / 8u));
    const uint32_t theta = a.mode == SWEEP_UPDATE ? a.theta : 0u;
    sweeps_quad<L, G, NR, UNIT, HOIST>(reinterpret_cast<uint32_t *>(rep0), g, on, k, a, base, theta);

    // ---- energy (eq. (3)): every bond joins a colour-0 site to a neighbour
    auto group_sum = [&](uint32_t v) {           // over the lanes of a group inside one wave
#pragma unroll
        for (uint32_t off = G >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        return v;
    };
    // v summed over the lanes of each group of this wave into at(group): whole
    // waves of a group, or the two groups a wave of G > 64 lanes meets, by lane
    // moves and one atomic each (64 atomics on one address serialise); small
    // groups lane by lane.  Lanes left over count, with nothing, as the last group's.
    const uint32_t gj = on ? gi : groups - 1u;
    auto spread_add = [&](auto v, auto at) {
        if (!on) v = 0;
        if constexpr (G > 64u || G % 64u == 0) {
            const uint32_t first = __builtin_amdgcn_readfirstlane(gj);
            const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)gj, 63);
            const auto own = wave_sum_all(gj == first ? v : decltype(v)(0));
            if ((tid & 63u) == 0) atomicAdd(at(first), own);
            if (G % 64u != 0 && end != first) {
                const auto next = wave_sum_all(gj == first ? decltype(v)(0) : v);
                if ((tid & 63u) == 0) atomicAdd(at(end), next);
            }
        } else if (on) {
            atomicAdd(at(gi), v);
        }
    };
    // flag mask of the slots of dword d of row y that hold sites
    auto site_mask = [&](uint32_t y, uint32_t d) {
        uint32_t m = UNIT * 0x01010101u;
        if constexpr (!Geo::FULL) {
            const uint32_t sh = Geo::ODD ? (y & 1u) : 0u;
            if (sh && d == 0) m &= 0xFFFFFF00u;
            if (4u * d + 4u > sh + Geo::H) m &= 0xFFFFFFFFu >> (8u * (4u * d + 4u - sh - Geo::H));
        }
        return m;
    };
    uint32_t bonds[NR], mt[NR];
    uint64_t dig[NR];
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r) {
        const uint32_t *p0 = reinterpret_cast<const uint32_t *>(rep0 + r * REPB), *p1 = p0 + PLANE;
        uint32_t ne = 0;
        if (on)
        lane_stride<PLANE, G>(g, PLANE, G, [&](uint32_t qd) {
            const uint32_t y = qd / DPQ, d = qd % DPQ, sh = Geo::ODD ? (y & 1u) : 0u;
            const uint32_t last = (Geo::H - 1 + sh) / 4u, lb = (Geo::H - 1 + sh) % 4u;
            const uint32_t D = p0[qd], A = p1[qd];
            uint32_t adj, sel;
            if (y & 1u) {
                adj = d == last ? qd - last : qd + 1;
                sel = d == last ? (0x04030201u & ~(0xFFu << (8u * lb))) | ((4u + sh) << (8u * lb)) : 0x04030201u;
            } else {             // (an even row has no shift)
                adj = d == 0 ? qd + last : qd - 1;
                sel = d == 0 ? 0x02010000u | (4u + lb) : 0x02010007u;
            }
            const uint32_t X = perm(p1[adj], A, sel);
            const uint32_t up = y == 0 ? qd + (L - 1) * DPQ : qd - DPQ, dn = y == L - 1 ? d : qd + DPQ;
            uint32_t U = p1[up], Dn = p1[dn];
            if constexpr (Geo::ODD != 0) {
                const uint32_t vs = sh ? (d == 0 ? 0u : ~0u) : (d == DPQ - 1 ? 0u : 1u);
                const uint32_t sv = sh ? 0x02010007u : 0x04030201u;
                U = perm(p1[up + vs], U, sv);
                Dn = perm(p1[dn + vs], Dn, sv);
            }
            const uint32_t m = site_mask(y, d);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, A, m), 0u, ne);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, X, m), 0u, ne);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, U, m), 0u, ne);
            ne = __builtin_amdgcn_sad_u8(quad_ne<UNIT>(D, Dn, m), 0u, ne);
        });
        bonds[r] = WAVE ? group_sum(ne / UNIT) : 0u;   // unequal neighbours; 2N bonds less these are equal
        if (!WAVE) spread_add(ne / UNIT, [&](uint32_t q) { return &acc_e[q * NR + r]; });
        // ---- magnetisation (eq. (5)): the largest number of sites in one state
        mt[r] = 0;
        if (a.Mt_out) {
            // two states' counts share a word where N < 2^16
            constexpr uint32_t PER = N < 65536u ? 2u : 1u;
            for (uint32_t st = 0; st < a.q; st += PER) {
                uint32_t c0 = 0, c1 = 0;
                if (on)
                lane_stride<Geo::REP, G>(g, Geo::REP, G, [&](uint32_t dd) {
                    const uint32_t m = site_mask((dd / DPQ) % L, dd % DPQ);
                    c0 = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(p0[dd], st * 0x01010101u, m), 0u, c0);
                    if (PER == 2u) c1 = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(p0[dd], (st + 1u) * 0x01010101u, m), 0u, c1);
                });
                const uint32_t c = c0 / UNIT | (c1 / UNIT) << 16;
                if constexpr (WAVE) {
                    const uint32_t w = group_sum(c);
                    mt[r] = max(mt[r], max(w & 0xFFFFu, w >> 16));
                } else {
                    spread_add(c, [&](uint32_t q) { return &acc_m[(q * NR + r) * qc + st / PER]; });
                }
            }
        }
        // ---- digest term (order-free sum over the dwords of four sites of a row)
        dig[r] = 0;
        if (a.H_out) {
            if (on)
                for (uint32_t dd = g; dd < N / 4u; dd += G)
                    dig[r] += digest_term(dd, k[r], a.step, get4(rep0 + r * REPB, dd), a.key0, a.key1);
            if constexpr (WAVE) {
                for (uint32_t off = G >> 1; off > 0; off >>= 1) dig[r] += __shfl_xor(dig[r], off, 64);
            } else {
                spread_add((unsigned long long)dig[r], [&](uint32_t q) { return &acc_d[q * NR + r]; });
            }
        }
    }
    if (!WAVE) __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < NR; ++r) {
        if (!live(r)) continue;
        if (g == 0) {
            const uint32_t li = gi * NR + r;
            if constexpr (!WAVE) {
                bonds[r] = acc_e[li];
                if (a.Mt_out)
                    for (uint32_t st = 0; st < a.q; ++st) {
                        const uint32_t w = acc_m[li * qc + (N < 65536u ? st / 2u : st)];
                        mt[r] = max(mt[r], N < 65536u ? (w >> (16u * (st & 1u))) & 0xFFFFu : w);
                    }
                if (a.H_out) dig[r] = acc_d[li];
            }
            a.E_out[k[r]] = (int32_t)bonds[r] - (int32_t)(2u * N);
            if (a.Mt_out) a.Mt_out[k[r]] = mt[r];
            if (a.H_out) a.H_out[k[r]] = dig[r];
        }
        // streaming stores, as in sweep_body
        uint8_t *rep = rep0 + r * REPB;
        uint8_t *gdst = a.new_pop + (size_t)k[r] * N;
        lane_stride<N / W, G>(g, N / W, G, [&](uint32_t o) {
            if constexpr (W == 16) {
                const uint2 e = *reinterpret_cast<const uint2 *>(plane_even(rep, o));
                const uint2 d = *reinterpret_cast<const uint2 *>(plane_odd(rep, o));
                const u32x4 v = {perm(d.x, e.x, 0x05010400u), perm(d.x, e.x, 0x07030602u),
                                 perm(d.y, e.y, 0x05010400u), perm(d.y, e.y, 0x07030602u)};
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(gdst) + o);
            } else if constexpr (W == 8) {
                const uint32_t e = *reinterpret_cast<const uint32_t *>(plane_even(rep, o));
                const uint32_t d = *reinterpret_cast<const uint32_t *>(plane_odd(rep, o));
                const u32x2 v = {perm(d, e, 0x05010400u), perm(d, e, 0x07030602u)};
                __builtin_nontemporal_store(v, reinterpret_cast<u32x2 *>(gdst) + o);
            } else {
                __builtin_nontemporal_store(get4(rep, o), reinterpret_cast<uint32_t *>(gdst) + o);
            }
        });
    }
}

constexpr uint32_t quad_wpe(uint32_t L, uint32_t G, uint32_t NR) {
    return NR == 1 ? quad_shape(L, G).wpe_one : quad_shape(L, G).wpe_max;
}

// The first a.big workgroups hold NR replicas per lane, the rest one: long waves
// first, short ones fill the end of the launch.
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__device__ __forceinline__ void sweep_quad_mixed(const SweepArgs &a, uint32_t block) {
    constexpr bool HOIST = quad_shape(LT, GT).hoist;
    if (NR == 1 || block < a.big) {
        sweep_quad_body<LT, GT, NR, UNIT, HOIST, false>(a, block, 0);
    } else {
        sweep_quad_body<LT, GT, 1, UNIT, HOIST, false>(a, block - a.big, a.big * (blockDim.x / GT) * NR);
    }
}

template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 1024), amdgpu_waves_per_eu(quad_wpe(LT, GT, NR))))
k_sweep_quad(SweepArgs a) {
    sweep_quad_mixed<LT, GT, NR, UNIT>(a, blockIdx.x);
}

// Batched form: run r owns workgroups start[r] .. start[r+1]-1.
template <uint32_t LT, uint32_t GT, uint32_t NR, uint32_t UNIT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 1024), amdgpu_waves_per_eu(quad_wpe(LT, GT, NR))))
k_sweep_quad_batch(const SweepArgs *runs, const uint32_t *start, uint32_t n) {
    const uint32_t r = segment_of(start, n, blockIdx.x);
    const SweepArgs &a = runs[r];    // by reference: a copy would go to scratch memory
    sweep_quad_mixed<LT, GT, NR, UNIT>(a, blockIdx.x - start[r]);
}

// The sides without a table entry (shape quad_any, 32 states).
template <uint32_t LT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 64 * quad_any(LT).waves), amdgpu_waves_per_eu(quad_any(LT).wpe)))
k_sweep_any(SweepArgs a) {
    sweep_quad_body<LT, quad_any(LT).G, 1, 32, quad_any(LT).hoist, true>(a, blockIdx.x, 0);
}

template <uint32_t LT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 64 * quad_any(LT).waves), amdgpu_waves_per_eu(quad_any(LT).wpe)))
k_sweep_any_batch(const SweepArgs *runs, const uint32_t *start, uint32_t n) {
    const uint32_t r = segment_of(start, n, blockIdx.x);
    const SweepArgs &a = runs[r];
    sweep_quad_body<LT, quad_any(LT).G, 1, 32, quad_any(LT).hoist, true>(a, blockIdx.x - start[r], 0);
}

}  // namespace

// Kernels of the sides without a table entry (pa_quad_any.hip, one translation
// unit each); null for a side of another part.
void *quad_any_part0(uint32_t L, bool batch);
void *quad_any_part1(uint32_t L, bool batch);
void *quad_any_part2(uint32_t L, bool batch);
void *quad_any_part3(uint32_t L, bool batch);

}  // namespace pa
