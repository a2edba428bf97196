// pa_quad_tiled.h -- the quad update (pa_quad.h) for lattices beyond one
// workgroup's LDS: q <= 32, 32-bit thresholds.
//
// As in k_tiled_half, a workgroup stages its tile of rows and two rows on each
// side in LDS, runs the two half-sweeps of a sweep on them and writes its own rows;
// here a row is held as its colour-0 sites followed by its colour-1 sites, L/2
// bytes (DPQ dwords) each.  Between the launches of one step the rows stay in
// that order in memory too (src_planar, dst_planar; L a multiple of 8), so that
// only the first launch of a step splits the ancestor's rows and only the last
// one joins them.
//
// The last launch of a step also counts the bonds (`fuse`): every bond joins
// two colours, and after the last half-sweep, of colour 1, the colour-0 sites
// of the row next to the tile are final too (the half-sweep before reached
// them), so the colour-1 sites of the tile see their four final neighbours.  A
// pass over the population per step goes away (33 us of 1000 at 1024x1024, 96
// replicas).
//
// Bound by vector instruction issue (125 per quad; 142 of the dword form) and,
// for sides that are no power of two, by the staging of rows: it costs as many
// instructions as it has pieces, so split rows are copied flat, and rows to
// split are taken by whole waves (scalar row addresses), several loads in
// flight.  Sweeps with their measuring, q = 10, theta = 10, attempts per ns,
// dword form / this one: 512 (400 replicas) 917 / 1110, 1024 (300) 994 / 1144,
// 2048 (24) 868 / 1037, 4096 (8) 813 / 955; 264 (1000) 567 / 759, 600 (200)
// 606 / 791, 1000 (96) 631 / 899; 260 (1000) 534 / 589, 300 (800) 566 / 654,
// 4092 (8) 513 / 631.
#pragma once

#include "pa_quad.h"

#include <type_traits>

namespace pa {

namespace {

// P sites of a row (16, 8 or 4, x even first) as they lie in memory, split into
// their even and odd bytes in the two halves of an LDS row and joined again.
template <uint32_t P> struct Piece;
template <> struct Piece<16> {
    typedef uint4 V;
    static __device__ __forceinline__ void put(uint8_t *e, uint8_t *o, uint32_t x, V v) {
        reinterpret_cast<uint2 *>(e)[x] = make_uint2(perm(v.y, v.x, 0x06040200u), perm(v.w, v.z, 0x06040200u));
        reinterpret_cast<uint2 *>(o)[x] = make_uint2(perm(v.y, v.x, 0x07050301u), perm(v.w, v.z, 0x07050301u));
    }
    static __device__ __forceinline__ V get(const uint8_t *e, const uint8_t *o, uint32_t x) {
        const uint2 a = reinterpret_cast<const uint2 *>(e)[x], b = reinterpret_cast<const uint2 *>(o)[x];
        return make_uint4(perm(b.x, a.x, 0x05010400u), perm(b.x, a.x, 0x07030602u), perm(b.y, a.y, 0x05010400u),
                          perm(b.y, a.y, 0x07030602u));
    }
};
template <> struct Piece<8> {
    typedef uint2 V;
    static __device__ __forceinline__ void put(uint8_t *e, uint8_t *o, uint32_t x, V v) {
        reinterpret_cast<uint32_t *>(e)[x] = perm(v.y, v.x, 0x06040200u);
        reinterpret_cast<uint32_t *>(o)[x] = perm(v.y, v.x, 0x07050301u);
    }
    static __device__ __forceinline__ V get(const uint8_t *e, const uint8_t *o, uint32_t x) {
        const uint32_t a = reinterpret_cast<const uint32_t *>(e)[x], b = reinterpret_cast<const uint32_t *>(o)[x];
        return make_uint2(perm(b, a, 0x05010400u), perm(b, a, 0x07030602u));
    }
};
template <> struct Piece<4> {
    typedef uint32_t V;
    static __device__ __forceinline__ void put(uint8_t *e, uint8_t *o, uint32_t x, V v) {
        reinterpret_cast<uint16_t *>(e)[x] = (uint16_t)perm(0u, v, 0x0C0C0200u);
        reinterpret_cast<uint16_t *>(o)[x] = (uint16_t)perm(0u, v, 0x0C0C0301u);
    }
    static __device__ __forceinline__ V get(const uint8_t *e, const uint8_t *o, uint32_t x) {
        return perm(reinterpret_cast<const uint16_t *>(o)[x], reinterpret_cast<const uint16_t *>(e)[x], 0x05010400u);
    }
};

// f(r, x, v) for the W pieces x of the rows r < nr, v = load(r, x); the loads
// of a batch are issued together (one round of memory latency each).  NRC, NTC,
// WC: rows, threads and pieces where known at compile time (0: not).  Otherwise a
// wave takes a row, so that the row's address is scalar, four rows a batch.
template <uint32_t NRC, uint32_t NTC, uint32_t WC, typename Load, typename F>
__device__ __forceinline__ void tile_pieces(uint32_t nr, uint32_t NT, uint32_t W, Load load, F f) {
    if constexpr (NRC != 0) {
        constexpr uint32_t M = (NRC * WC + NTC - 1) / NTC;
        decltype(load(0u, 0u)) v[M];
#pragma unroll
        for (uint32_t m = 0; m < M; ++m) {
            const uint32_t i = threadIdx.x + m * NTC;
            if (NRC * WC % NTC == 0 || i < NRC * WC) v[m] = load(i / WC, i % WC);
        }
#pragma unroll
        for (uint32_t m = 0; m < M; ++m) {
            const uint32_t i = threadIdx.x + m * NTC;
            if (NRC * WC % NTC == 0 || i < NRC * WC) f(i / WC, i % WC, v[m]);
        }
    } else {
        constexpr uint32_t B = 4;
        const uint32_t waves = NT >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        for (uint32_t r = wave; r < nr; r += B * waves)
            for (uint32_t x = threadIdx.x & 63u; x < W; x += 64u) {
                decltype(load(0u, 0u)) v[B];
#pragma unroll
                for (uint32_t m = 0; m < B; ++m)
                    if (r + m * waves < nr) v[m] = load(r + m * waves, x);
#pragma unroll
                for (uint32_t m = 0; m < B; ++m)
                    if (r + m * waves < nr) f(r + m * waves, x, v[m]);
            }
    }
}

// Copies n pieces, four loads in flight per lane: dst[i] = src(i).
template <typename V, typename Src, typename Dst>
__device__ __forceinline__ void tile_copy(uint32_t n, uint32_t NT, Src src, Dst dst) {
    for (uint32_t i = threadIdx.x; i < n; i += 4u * NT) {
        V v[4];
#pragma unroll
        for (uint32_t m = 0; m < 4; ++m)
            if (i + m * NT < n) v[m] = src(i + m * NT);
#pragma unroll
        for (uint32_t m = 0; m < 4; ++m)
            if (i + m * NT < n) dst(i + m * NT, v[m]);
    }
}

template <uint32_t UNIT>
__device__ __forceinline__ void quad_table(uint8_t *tab, const uint64_t *T, uint32_t tid, uint32_t nthreads) {
    for (uint32_t t = tid; t < 81u * (UNIT / 8u); t += nthreads) {
        const uint32_t e = t / (UNIT / 8u), i0 = e % 9u, i1 = e / 9u;
        const uint32_t x = i0 <= 4u ? 0xFFFFFFFFu : (uint32_t)(T[i0 - 5u] - 1u);
        const uint32_t y = i1 <= 4u ? 0xFFFFFFFFu : (uint32_t)(T[i1 - 5u] - 1u);
        *reinterpret_cast<uint2 *>(tab + 8u * t) = make_uint2(x, y);
    }
}

// Words of Philox shared by all pairs of a replica and step (k uniform).
struct TileKey {
    SweepKey s;
    uint32_t c3k, u2;
    __device__ __forceinline__ TileKey(uint32_t k, uint32_t step, uint32_t key0, uint32_t key1)
        : s(sweep_key(k, step, 0, key0, key1)) {
        const uint64_t q0 = (uint64_t)PHILOX_M0 * s.n0;
        c3k = (uint32_t)q0 ^ s.k1[2];
        u2 = (uint32_t)(q0 >> 32) ^ s.k1[1];
    }
    // the block of pair p, P0 = M0 * p
    __device__ __forceinline__ uint4 block(uint64_t P0, uint32_t c3k1) const {
        const QuadPrefix f = quad_prefix((uint32_t)(P0 >> 32), c3k1, s);
        return quad_block(f, (uint64_t)PHILOX_M1 * ((uint32_t)P0 ^ u2), c3k, s);
    }
};

// One launch: two half-sweeps, of colour 0 and then of colour 1, of one tile.  A
// lane keeps dword d of a row and takes every RS-th row, two at a time, whose
// parities stay fixed.  LT, NTT: the side and the workgroup of a compile-time
// form (512 .. 4096, powers of two), or 0: any side divisible by 4 with a.rs
// rows of lanes (the lanes left over of the last wave idle); where L is not a
// multiple of 8, a colour's last dword in a row is half filled, its padding
// updated like sites and never read as a neighbour.
constexpr uint32_t QT_HALVES = 2;

template <uint32_t LT, uint32_t NTT, uint32_t UNIT>
__global__ void __launch_bounds__(NTT ? NTT : 512) k_tiled_quad(TiledArgs a) {
    constexpr uint32_t S = QT_HALVES;
    extern __shared__ __align__(16) uint8_t smem[];
    uint32_t k, tile;
    tile_of(a.tiles, k, tile);
    const uint32_t tid = threadIdx.x, NT = NTT ? NTT : blockDim.x;
    const uint32_t L = LT ? LT : a.L, H = L >> 1, DPQ = (L + 4u) >> 3;
    const uint32_t RS = LT ? NTT / (LT / 8u ? LT / 8u : 1u) : a.rs;
    const bool full = LT != 0 || (L & 7u) == 0;
    const uint32_t n = LT ? 16384u / (LT ? LT : 1u) : min(a.rows, L - tile * a.rows);   // (rows of a tile: tiled_rows)
    const uint32_t y0 = tile * (LT ? n : a.rows), nl = n + 2 * S;
    const uint32_t ROW = 2 * DPQ, COL = DPQ;     // LDS: the two colours of a row side by side
    auto row_of = [&](uint32_t r) {            // global row of local row r (periodic)
        uint32_t gy = y0 + r + L - S;
        if constexpr (LT != 0) return gy & (LT - 1u);
        gy = gy >= L ? gy - L : gy;
        return gy >= L ? gy - L : gy;
    };
    uint32_t *lds32 = reinterpret_cast<uint32_t *>(smem);
    const uint32_t tab = (nl * DPQ * 8u + 15u) & ~15u;
    quad_table<UNIT>(smem + tab, a.T, tid, NT);
    const uint32_t src = a.anc ? a.anc[k] : k;
    const uint8_t *gsrc = a.src + (size_t)src * a.N;
    constexpr uint32_t NLC = LT ? 16384u / LT + 2 * S : 0u;      // rows of a compile-time side
    auto stage_in = [&](auto piece) {
        using Pc = decltype(piece);
        using V = typename Pc::V;
        constexpr uint32_t B = sizeof(V);
        tile_pieces<NLC, NTT, LT / B>(
            nl, NT, L / B, [&](uint32_t r, uint32_t x) { return reinterpret_cast<const V *>(gsrc + (size_t)row_of(r) * L)[x]; },
            [&](uint32_t r, uint32_t x, V v) {
                uint8_t *row = smem + r * ROW * 4u;
                if (LT != 0 && a.src_planar) {
                    reinterpret_cast<V *>(row)[x] = v;
                } else {                                       // even x: colour of the row's parity
                    const uint32_t p = row_of(r) & 1u;
                    Pc::put(row + p * 4u * COL, row + (1u - p) * 4u * COL, x, v);
                }
            });
    };
    // rows split by colour are the LDS rows as they stand: the tile's are
    // consecutive in memory but for the wrap from row L - 1 to row 0
    auto copy_in = [&](auto zero) {
        using V = decltype(zero);
        const uint32_t first = row_of(0) * L;
        tile_copy<V>(nl * L / sizeof(V), NT,
                     [&](uint32_t i) {
                         const uint32_t at = first + i * (uint32_t)sizeof(V);
                         return *reinterpret_cast<const V *>(gsrc + (at >= a.N ? at - a.N : at));
                     },
                     [&](uint32_t i, V v) { reinterpret_cast<V *>(smem)[i] = v; });
    };
    if (LT == 0 && a.src_planar) {
        if ((L & 15u) == 0) copy_in(uint4{});
        else copy_in(uint2{});
    } else if (LT != 0 || (L & 15u) == 0) {
        stage_in(Piece<16>{});
    } else if (full) {
        stage_in(Piece<8>{});
    } else {
        stage_in(Piece<4>{});
        for (uint32_t i = tid; i < 2u * nl; i += NT) *reinterpret_cast<uint16_t *>(smem + 4u * DPQ * i + H) = 0;   // padding
    }
    __syncthreads();
    const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)smem + tab +
                          8u * (tid % (UNIT / 8u));
    const uint32_t qm1 = a.q - 1u;
    const uint32_t d = tid % DPQ;
    uint32_t roff = tid / DPQ;
    if constexpr (LT != 0) roff = NTT == LT / 8u ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane(roff);
    const bool on = LT != 0 || roff < RS;
    // the horizontal neighbours that are not in the same dword of the other
    // colour: the dword and the selector where they are to the left and right
    const uint32_t last = DPQ - 1, lb = (H - 1u) & 3u;        // the last site's dword and byte
    const uint32_t left = d == 0 ? last : d - 1, right = d == last ? 0 : d + 1;
    uint32_t sel_l = 0x02010007u, sel_r = 0x04030201u;
    if (!full) {
        if (d == 0) sel_l = 0x02010000u | (4u + lb);
        if (d == last) sel_r = (sel_r & ~(0xFFu << (8u * lb))) | (4u << (8u * lb));
    }
    const TileKey key(k, a.step, a.key0, a.key1);
    const uint64_t mg = (uint64_t)PHILOX_M0 * (2u * d);
    auto half = [&](auto colour) {
        constexpr uint32_t c = decltype(colour)::value;
        const uint32_t c3k1 = ((DOM_SWEEP << 28) | a.h0 | c) ^ a.key1;     // (sweep h0 / 2, colour c)
        constexpr uint32_t r0 = 1 + c;
        const uint32_t nr = nl - 2 * r0;                                     // rows r0 .. nl - 1 - r0
        const uint32_t oo = c ? COL : 0u, po = COL - oo;                     // own and other colour
        // the row parities of a lane's two rows
        const uint32_t par0 = (y0 + r0 + roff + L - S + c) & 1u;
        uint32_t adj[2], sel[2];
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u) {
            const uint32_t par = (par0 + u * RS) & 1u;
            adj[u] = par ? right : left;
            sel[u] = par ? sel_r : sel_l;
        }
        uint32_t *pb = lds32 + (r0 - 1 + roff) * ROW;          // the row above
        const uint32_t pairs = L * (L >> 2), step = RS * (L >> 2);          // of a replica; between a lane's rows
        uint32_t pr = row_of(r0 + roff) * (L >> 2);                         // first pair of the row
        auto quad = [&](uint32_t *row, uint32_t pru, uint32_t u) {
            const uint32_t *o = row + po;
            const uint32_t D = row[ROW + oo + d], A = o[ROW + d], Ax = o[ROW + adj[u]];
            const uint32_t U = o[d], Dn = o[2 * ROW + d];
            const uint64_t P0 = mg + (uint64_t)PHILOX_M0 * pru;
            const uint4 wa = key.block(P0, c3k1), wb = key.block(P0 + PHILOX_M0, c3k1);
            row[ROW + oo + d] = update_quad<UNIT>(D, perm(Ax, A, sel[u]), A, U, Dn, wa, wb, qm1, base);
        };
        auto next = [&](uint32_t p) -> uint32_t {
            p += step;
            if constexpr (LT != 0) return p & (LT * (LT / 4u) - 1u);
            const uint32_t w = p - pairs;
            return p < w ? p : w;                  // (p - pairs wraps to a large number below it)
        };
        if (on) {
            uint32_t rr = roff;
            for (; rr + RS < nr; rr += 2 * RS) {
                const uint32_t p1 = next(pr);
                quad(pb, pr, 0);
                quad(pb + RS * ROW, p1, 1);
                pb += 2 * RS * ROW;
                pr = next(p1);
            }
            if (rr < nr) quad(pb, pr, 0);
        }
        __syncthreads();
    };
    half(std::integral_constant<uint32_t, 0>{});
    half(std::integral_constant<uint32_t, 1>{});
    uint8_t *gdst = a.dst + (size_t)k * a.N + (size_t)y0 * L;
    auto stage_out = [&](auto piece) {
        using Pc = decltype(piece);
        using V = typename Pc::V;
        constexpr uint32_t B = sizeof(V);
        tile_pieces<LT ? NLC - 2 * S : 0u, NTT, LT / B>(
            n, NT, L / B,
            [&](uint32_t r, uint32_t x) {
                const uint8_t *row = smem + (S + r) * ROW * 4u;
                if (LT != 0 && a.dst_planar) return reinterpret_cast<const V *>(row)[x];
                const uint32_t p = (y0 + r) & 1u;
                return Pc::get(row + p * 4u * COL, row + (1u - p) * 4u * COL, x);
            },
            [&](uint32_t r, uint32_t x, V v) { reinterpret_cast<V *>(gdst + (size_t)r * L)[x] = v; });
    };
    auto copy_out = [&](auto zero) {
        using V = decltype(zero);
        const V *rows = reinterpret_cast<const V *>(smem + S * ROW * 4u);
        tile_copy<V>(n * L / sizeof(V), NT, [&](uint32_t i) { return rows[i]; },
                     [&](uint32_t i, V v) { reinterpret_cast<V *>(gdst)[i] = v; });
    };
    if (LT == 0 && a.dst_planar) {
        if ((L & 15u) == 0) copy_out(uint4{});
        else copy_out(uint2{});
    } else if (LT != 0 || (L & 15u) == 0) {
        stage_out(Piece<16>{});
    } else if (full) {
        stage_out(Piece<8>{});
    } else {
        stage_out(Piece<4>{});
    }
    if (a.fuse) {
        uint32_t eq = 0;
        const uint32_t m = (UNIT * 0x01010101u) & (!full && d == last ? 0x0000FFFFu : 0xFFFFFFFFu);
        if (on)
            for (uint32_t r = roff; r < n; r += RS) {
                const uint32_t *row = lds32 + (S + r - 1) * ROW;        // the row above
                const bool par = ((y0 + r + 1u) & 1u) != 0;              // colour 1
                const uint32_t D = row[ROW + COL + d], A = row[ROW + d], Ax = row[ROW + (par ? right : left)];
                eq = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(D, A, m), 0u, eq);
                eq = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(D, perm(Ax, A, par ? sel_r : sel_l), m), 0u, eq);
                eq = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(D, row[d], m), 0u, eq);
                eq = __builtin_amdgcn_sad_u8(quad_eq<UNIT>(D, row[2 * ROW + d], m), 0u, eq);
            }
        // one atomic per workgroup: those of a replica's tiles meet on one address
        const uint32_t w = wave_total(eq / UNIT);
        __shared__ uint32_t s_bonds;
        if (tid == 0) s_bonds = 0u;
        __syncthreads();
        if ((tid & 63u) == 0) atomicAdd(&s_bonds, w);
        __syncthreads();
        if (tid == 0) atomicAdd(&a.bonds[k], s_bonds);
    }
}

}  // namespace

}  // namespace pa
