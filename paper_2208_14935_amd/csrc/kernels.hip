// Device side of the hybrid-transfer traversal, written for gfx950 (wave64).
//
// Per iteration (Sec. 4 overview, Algorithm 1):
//   k_unit_stats    one wave per unit (512 to 4,096 vertices) of a partition: active vertices,
//                   active edges and request lines from the frontier bitmap, then (in
//                   k_part_combine for partitions of several runs) the engine choice of
//                   Sec. 5.1 (Eq. 1-3, alpha/beta rule) in exact integer arithmetic;
//   k_scan_*        per-engine prefix sums over partitions (tile totals, tile bases,
//                   offsets), which place every partition's active vertices in one list
//                   ordered by engine segment and partition ("pre-combine" of Vc and Vz,
//                   Algorithm 1);
//   k_build_lists   one wave per run of a scheduled partition: ordered compaction of its active
//                   vertices into the list plus the work prefix (edges, or 128-byte
//                   lines for zero-copy) used for load balancing;
//   k_push_edges    edge-balanced push over a list slice reading device memory
//                   (resident cache, filter staging, or compaction buffer);
//   k_push_lines    line-balanced push reading mapped pinned host memory: each half
//                   wave loads one whole 128-byte line (merged, aligned zero-copy
//                   access, Sec. 2.3 / Sec. 3.2);
// with push operators for BFS, SSSP (atomicMin), CC (atomicMin on labels) and
// PageRank (FP32 atomic add), and a bitmap-directed next frontier (Sec. 6.3).
#include <hip/hip_runtime.h>

#include <type_traits>

#include <mutex>

#include "hytm_kernels.h"

namespace hytm {
namespace {

constexpr uint32_t UNREACHED = 0xFFFFFFFFu;
typedef unsigned __int128 u128;

__device__ __forceinline__ uint64_t lines_of(uint64_t s, uint64_t e, uint32_t sh) {
    // lines of 2^sh four-byte elements touched by elements [s, e), e > s
    return ((e - 1) >> sh) - (s >> sh) + 1;
}

// ------------------------------------------------------------ reductions / scans
__device__ __forceinline__ uint64_t wave_sum(uint64_t x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Exclusive prefix sum over the wave; *total gets the wave's sum.
__device__ __forceinline__ uint64_t wave_exclusive_sum(uint64_t x, uint64_t* total) {
    const int lane = threadIdx.x & 63;
    uint64_t v = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t y = __shfl_up(v, d, 64);
        if (lane >= d) v += y;
    }
    *total = __shfl(v, 63, 64);
    return v - x;
}

// Exclusive prefix maximum over the wave (0 for lane 0); *total gets the wave's maximum.
__device__ __forceinline__ uint64_t wave_exclusive_max(uint64_t x, uint64_t* total) {
    const int lane = threadIdx.x & 63;
    uint64_t v = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t y = __shfl_up(v, d, 64);
        if (lane >= d) v = v > y ? v : y;
    }
    *total = __shfl(v, 63, 64);
    const uint64_t ex = __shfl_up(v, 1, 64);
    return lane ? ex : 0;
}

// ------------------------------------------------------------- engine selection
// Sec. 5.1 with RTT = 1 and every comparison cleared of denominators:
//   Tef = ceil(E*d1 / L), Tec = ceil((Ea*d1 + nA*d2) / L), Q = ceil(Rq / MR),
//   Tiz = Q * (gn*E + (gd-gn)*Ea) / (gd*E)
//   compaction iff ad*Tec < an*Tef  and  bd*gd*E*Tec < bn*Q*(gn*E + (gd-gn)*Ea);
//   else zero-copy iff Q*(gn*E + (gd-gn)*Ea) < gd*E*Tef; else filter.
__device__ __forceinline__ uint8_t select_engine(uint64_t E, uint64_t nA, uint64_t Ea, uint64_t Rq,
                                                 const SelParams& sp) {
    const uint64_t tef = (E * sp.d1 + sp.L - 1) / sp.L;
    uint64_t tec = (Ea * sp.d1 + nA * sp.d2 + sp.L - 1) / sp.L;
    if (sp.gn_c) {
        // the host gather runs as a pipeline with the copy: the slower of the two counts
        const u128 den = (u128)sp.L * sp.gd_c;
        const uint64_t tgc = (uint64_t)(((u128)Ea * sp.d1 * sp.gn_c + den - 1) / den);
        if (tgc > tec) tec = tgc;
    }
    const uint64_t q = (Rq + sp.MR - 1) / sp.MR;
    const u128 zfac = (u128)sp.gn * E + (u128)(sp.gd - sp.gn) * Ea;
    const bool c1 = (u128)sp.ad * tec < (u128)sp.an * tef;
    const bool c2 = (u128)sp.bd * sp.gd * E * tec < (u128)sp.bn * q * zfac;
    if (c1 && c2 && sp.allow_compact) return P_COMPACT;
    const u128 zl = (u128)q * zfac, zr = (u128)sp.gd * E * tef;
    if (zl < zr || (sp.zc_tie && zl == zr)) return P_ZC;
    return sp.allow_filter ? P_FILTER : P_ZC;
}

// ------------------------------------------------------------------- stats
// One wave per unit (four units per workgroup, no workgroup barriers): a unit is a run of at
// most 64 aligned windows of 64 vertices of one partition, so a partition of many vertices
// (they are cut by edges: R-MAT's low-degree tail puts up to 0.5M vertices into one) is
// walked by many waves.  Lane l loads the active bits of window l, a wave scan counts them,
// and then the unit's active vertices are dealt out in order, one per lane, in batches of 64
// (SEL_B batches with their offset loads in flight together).  Lanes are busy whatever the
// density, and where the frontier is dense consecutive lanes hold consecutive vertices, so
// the offset loads coalesce.  A partition of one unit is finished here; the units of a larger
// one leave records that k_part_combine joins.
// Bound by the offset gathers of scattered frontiers, by latency on small ones.  One wave per
// partition took, all vertices active, 1.68 + 1.49 ms (statistics + lists) on R-MAT 24 and
// 0.73 + 0.62 ms on symmetrized R-MAT 21.
constexpr int SEL_B = 4;

// Active bits of window q (vertices 64 q .. 64 q + 63) restricted to [vb, ve).
__device__ __forceinline__ uint64_t window_bits(const uint32_t* __restrict__ bm, uint32_t q, uint32_t vb,
                                                uint32_t ve) {
    const uint32_t lo = q << 6;
    // word 2q+1 may lie past the bitmap when 64q + 32 >= ve; then its bits are masked off
    // below, and the load reads the partition's last word instead
    const uint32_t hi = min(2 * q + 1, (ve - 1) >> 5);
    uint64_t bits = bm[2 * q] | ((uint64_t)bm[hi] << 32);
    if (lo < vb) bits &= ~0ull << (vb - lo);
    if (ve - lo < 64) bits &= (1ull << (ve - lo)) - 1ull;
    return bits;
}

// Position of the r-th (from 0) set bit of x; r < popcount(x).
__device__ __forceinline__ uint32_t select_bit(uint64_t x, uint32_t r) {
    uint32_t pos = 0, c;
    c = __popc((uint32_t)x);
    if (r >= c) { r -= c; x >>= 32; pos += 32; }
    c = __popc((uint32_t)x & 0xFFFFu);
    if (r >= c) { r -= c; x >>= 16; pos += 16; }
    c = __popc((uint32_t)x & 0xFFu);
    if (r >= c) { r -= c; x >>= 8; pos += 8; }
    c = __popc((uint32_t)x & 0xFu);
    if (r >= c) { r -= c; x >>= 4; pos += 4; }
    c = __popc((uint32_t)x & 0x3u);
    if (r >= c) { r -= c; x >>= 2; pos += 2; }
    if (r >= ((uint32_t)x & 1u)) pos += 1;
    return pos;
}

// Inclusive prefix sum over the wave.
__device__ __forceinline__ uint32_t wave_inclusive_sum_u32(uint32_t x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// The vertex holding the k-th (from 0) active bit of the round: windows q0 + j, with
// incl the inclusive count of active bits over windows 0..lane; k < the round's total.
__device__ __forceinline__ uint32_t round_vertex(uint32_t k, uint32_t incl, uint32_t cnt, uint64_t wbits,
                                                 uint32_t q0) {
    uint32_t j = 0;
#pragma unroll
    for (uint32_t step = 32; step; step >>= 1)
        if (__shfl(incl, j + step - 1, 64) <= k) j += step;
    const uint64_t bj = __shfl(wbits, j, 64);
    const uint32_t before = __shfl(incl - cnt, j, 64);
    return ((q0 + j) << 6) + select_bit(bj, k - before);
}

// Running sums of a partition's statistics in one lane: active lists, their edges, request
// lines per list and distinct (Eq. 3), kernel lines; with a byte weight array its request
// lines are counted apart (a list of D edges spans D bytes there).  carry / carry_w: (line + 1)
// of the latest list's last line in each array, 0 = none.
// lm: the lanes active at the vertices seen (batched runs).
struct SelAcc {
    uint64_t c = 0, ea = 0, rq = 0, kl = 0, rqd = 0, carry = 0;
    uint64_t rqw = 0, rqdw = 0, carry_w = 0;
    uint64_t first = 0, first_w = 0;  // (line + 1) of the unit's first list's first line
    uint64_t lm = 0;
};

// The lines of a list [s, e) in an array whose lines hold 2^sh entries: (first + 1, last + 1).
__device__ __forceinline__ void list_lines(uint64_t s, uint64_t e, uint32_t sh, uint64_t& fl, uint64_t& ll) {
    fl = (s >> sh) + 1;
    ll = ((e - 1) >> sh) + 1;
}

// Batches [b0, b0 + 64 G) of a round's active vertices: every lane loads (a lane past the
// round's end the round's last vertex), so the loads of all G batches are issued before the
// first is used.
template <int G>
__device__ __forceinline__ void stats_batches(uint32_t b0, uint32_t T, uint32_t incl, uint32_t cnt, uint64_t wbits,
                                              uint32_t q0, const uint64_t* __restrict__ off, const SelParams& sp,
                                              const uint64_t* __restrict__ mcur, bool lines, SelAcc& a) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t sh = sp.cost_shift, shw = sp.cost_shift + 2;  // byte weights: 4x the entries per line
    const bool bytew = sp.wbytes == 1;
    uint64_t s[G], e[G];
#pragma unroll
    for (int g = 0; g < G; g++) {
        const uint32_t k = b0 + 64 * g + lane;
        const uint32_t v = round_vertex(k < T ? k : T - 1, incl, cnt, wbits, q0);
        s[g] = off[v];
        e[g] = off[v + 1];
        if (mcur) a.lm |= mcur[v];
    }
#pragma unroll
    for (int g = 0; g < G; g++) {
        if (b0 + 64 * g >= T) break;
        const bool has = b0 + 64 * g + lane < T && e[g] > s[g];
        uint64_t fl = 0, ll = 0, flw = 0, llw = 0;
        if (has) {
            a.c += 1;
            a.ea += e[g] - s[g];
        }
        if (!lines) continue;  // uniform: a resident partition, or one whose engine is forced
        if (has) {
            a.rq += lines_of(s[g], e[g], sh);
            a.kl += lines_of(s[g], e[g], ZC_LINE_SHIFT);
            list_lines(s[g], e[g], sh, fl, ll);
            if (bytew) {
                a.rqw += lines_of(s[g], e[g], shw);
                list_lines(s[g], e[g], shw, flw, llw);
            }
        }
        // the last line of the latest earlier list (lists are in vertex order)
        uint64_t tot;
        const uint64_t ex = wave_exclusive_max(ll, &tot);
        const uint64_t prev = a.carry > ex ? a.carry : ex;
        if (!a.first) {  // uniform: the first list of the unit holds its smallest line
            const uint64_t A = __ballot(has);
            if (A) {
                const int l0 = (int)__ffsll((unsigned long long)A) - 1;
                a.first = __shfl(fl, l0, 64);
                a.first_w = __shfl(flw, l0, 64);
            }
        }
        if (has) a.rqd += ll - fl + 1 - (prev == fl ? 1 : 0);
        a.carry = a.carry > tot ? a.carry : tot;
        if (bytew) {  // uniform
            const uint64_t exw = wave_exclusive_max(llw, &tot);
            const uint64_t prevw = a.carry_w > exw ? a.carry_w : exw;
            if (has) a.rqdw += llw - flw + 1 - (prevw == flw ? 1 : 0);
            a.carry_w = a.carry_w > tot ? a.carry_w : tot;
        }
    }
}

// Engine of a partition from its statistics.
__device__ __forceinline__ uint8_t engine_of(uint32_t i, uint64_t E, uint64_t c, uint64_t ea, uint64_t rq,
                                             const SelParams& sp) {
    if (ea == 0) return P_NONE;
    if (i < sp.nres) return P_RES;
    if (sp.force) return (uint8_t)sp.force;
    return select_engine(E, c, ea, rq, sp);
}

typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// The bytes of a word that equal `tag`, one bit each.
__device__ __forceinline__ uint64_t bytes_equal(uint64_t w, uint64_t tag) {
    const uint64_t t = w ^ (tag * 0x0101010101010101ull), low = 0x7F7F7F7F7F7F7F7Full;
    const uint64_t z = ~(((t & low) + low) | t | low);  // 0x80 in every zero byte of t
    return ((z >> 7) * 0x0102040810204080ull) >> 56;
}

// Window q0 + lane of a unit's windows [q0, qe), its vertices of [vb, ve), as a wide iteration
// left it (LevelScan).  Whole windows go into the frontier and visited bitmaps; a window that
// two partitions share is written by the waves of both, with the same words.
__device__ __forceinline__ uint64_t level_bits(const LevelScan& ls, uint32_t q0, uint32_t qe, uint32_t vb,
                                               uint32_t ve, uint32_t nwords) {
    constexpr uint32_t G = 16;  // windows with their loads in flight together
    const uint32_t lane = threadIdx.x & 63;
    uint64_t bits = 0;
    if (ls.lvl) {  // uniform
        for (uint32_t q = q0; q < qe; q += G) {
            uint32_t x[G];
#pragma unroll
            for (uint32_t r = 0; r < G; r++) {
                const uint64_t v = ((uint64_t)(q + r) << 6) + lane;
                x[r] = q + r < qe && v < ls.n ? ls.lvl[v] : UNREACHED;
            }
#pragma unroll
            for (uint32_t r = 0; r < G; r++) {
                const uint64_t b = __ballot(x[r] == ls.level);
                if (q + r - q0 == lane) bits = b;
            }
        }
    } else if (q0 + lane < qe) {
        const u64x2* m = (const u64x2*)(ls.marks + ((uint64_t)(q0 + lane) << 6));
        u64x2 x[4];
#pragma unroll
        for (int r = 0; r < 4; r++) x[r] = m[r];
#pragma unroll
        for (int r = 0; r < 4; r++)
            bits |= (bytes_equal(x[r].x, ls.level) | bytes_equal(x[r].y, ls.level) << 8) << (16 * r);
    }
    if (q0 + lane >= qe) return 0;
    const uint32_t w = 2 * (q0 + lane), lo = (uint32_t)bits, hi = (uint32_t)(bits >> 32);
    ls.cur[w] = lo;
    if (w + 1 < nwords) ls.cur[w + 1] = hi;
    if (ls.visited) {
        if (lo) ls.visited[w] |= lo;
        if (hi) ls.visited[w + 1] |= hi;
    }
    const uint32_t v0 = (q0 + lane) << 6;
    if (v0 < vb) bits &= ~0ull << (vb - v0);
    if (ve - v0 < 64) bits &= (1ull << (ve - v0)) - 1ull;
    return bits;
}

// The record of unit u, taken by a whole wave (the same in every lane).  clear (or null): a
// bitmap of nwords words zeroed along the way (the frontier after next).  mcur (or null): *lm
// gains the lane masks of the active vertices.
// SCAN: the frontier is not in cur yet but the vertices at level ls.level (ls).
template <bool SCAN>
__device__ __forceinline__ UnitRec unit_record(const Units& un, uint32_t u, const uint32_t* __restrict__ pv,
                                               const uint64_t* __restrict__ off, const uint32_t* __restrict__ cur,
                                               uint32_t* __restrict__ clear, uint32_t nwords,
                                               const uint64_t* __restrict__ mcur, const SelParams& sp,
                                               const LevelScan& ls, uint64_t* lm) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t i = un.part[u], q0 = un.q[u];
    const uint32_t vb = pv[i], ve = pv[i + 1];
    const uint32_t qe = min(q0 + un.windows, (ve + 63) >> 6);
    // request lines matter where the cost model decides, kernel lines to zero-copy
    const bool lines = i >= sp.nres && (!sp.force || sp.force == P_ZC);
    SelAcc a;
    uint64_t wbits;
    if constexpr (SCAN)
        wbits = level_bits(ls, q0, qe, vb, ve, nwords);
    else
        wbits = q0 + lane < qe ? window_bits(cur, q0 + lane, vb, ve) : 0ull;
    if (clear && q0 + lane < qe) {  // windows shared by two partitions are zeroed by both
        const uint32_t w = 2 * (q0 + lane);
        clear[w] = 0;
        if (w + 1 < nwords) clear[w + 1] = 0;
    }
    UnitRec r{};
    if (!__ballot(wbits != 0)) return r;
    const uint32_t cnt = __popcll(wbits);
    const uint32_t incl = wave_inclusive_sum_u32(cnt);
    const uint32_t T = __shfl(incl, 63, 64);
    r.f = T;
    // at most 64 active vertices take one batch, more SEL_B at a time
    if (T <= 64)
        stats_batches<1>(0, T, incl, cnt, wbits, q0, off, sp, mcur, lines, a);
    else
        for (uint32_t b0 = 0; b0 < T; b0 += 64 * SEL_B)
            stats_batches<SEL_B>(b0, T, incl, cnt, wbits, q0, off, sp, mcur, lines, a);
    r.c = (uint32_t)wave_sum(a.c);
    r.ea = wave_sum(a.ea);
    if (lines) {
        // request lines: the neighbour array, and the weight array beside it (Eq. 3)
        r.rq = wave_sum(sp.rq_distinct ? a.rqd : a.rq);
        if (sp.wbytes == 1)
            r.rq += wave_sum(sp.rq_distinct ? a.rqdw : a.rqw);
        else if (sp.wbytes)
            r.rq *= 2;  // 4-byte weights: the neighbour array's lines again
        r.kl = wave_sum(a.kl);
        r.first = a.first;
        r.last = a.carry;
        r.first_w = a.first_w;
        r.last_w = a.carry_w;
    }
    if (mcur) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) a.lm |= __shfl_xor(a.lm, d, 64);
        *lm |= a.lm;
    }
    return r;
}

// lanes: *lanes |= the lane masks of the active vertices (with mcur).
template <bool SCAN>
__global__ __launch_bounds__(256) void k_unit_stats(Units un, const uint32_t* __restrict__ pv,
                                                    const uint64_t* __restrict__ off,
                                                    const uint32_t* __restrict__ cur, uint32_t* __restrict__ clear,
                                                    uint32_t nwords, const uint64_t* __restrict__ mcur,
                                                    unsigned long long* __restrict__ lanes, SelParams sp,
                                                    uint8_t* __restrict__ mode, uint32_t* __restrict__ nA,
                                                    uint32_t* __restrict__ nF, uint64_t* __restrict__ Ea,
                                                    uint64_t* __restrict__ K, LevelScan ls) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wpb = blockDim.x >> 6, waves = gridDim.x * wpb;
    for (uint32_t u = blockIdx.x * wpb + (threadIdx.x >> 6); u < un.count; u += waves) {
        uint64_t lm = 0;
        const UnitRec r = unit_record<SCAN>(un, u, pv, off, cur, clear, nwords, mcur, sp, ls, &lm);
        if (lane != 0) continue;
        if (lm && (lm & ~(uint64_t)*lanes)) atomicOr(lanes, (unsigned long long)lm);
        const uint32_t i = un.part[u];
        if (un.first[i + 1] - un.first[i] == 1) {
            mode[i] = engine_of(i, off[pv[i + 1]] - off[pv[i]], r.c, r.ea, r.rq, sp);
            nA[i] = r.c;
            nF[i] = r.f;
            Ea[i] = r.ea;
            K[i] = r.kl;
        } else {
            un.rec[u] = r;
        }
    }
}

// The records rec[u0, u1) of a partition's units joined by a wave (a line that one unit's last
// list ends and the next one's first list starts in counts once where distinct lines are
// counted); every record becomes the list entries, edges and lines of the partition's
// earlier units, where the unit's part of the lists starts.
__device__ __forceinline__ UnitRec join_units(UnitRec* rec, uint32_t u0, uint32_t u1, const SelParams& sp) {
    const uint32_t lane = threadIdx.x & 63;
    uint64_t c = 0, f = 0, ea = 0, kl = 0, rq = 0, dup = 0, last = 0, last_w = 0;
    const uint64_t twice = sp.wbytes == 4 ? 2 : 1;
    for (uint32_t b = u0; b < u1; b += 64) {
        const bool in = b + lane < u1;
        UnitRec r{};
        if (in) r = rec[b + lane];
        uint64_t tc, te, tk, tot, totw;
        const uint64_t xc = wave_exclusive_sum(r.c, &tc);
        const uint64_t xe = wave_exclusive_sum(r.ea, &te);
        const uint64_t xk = wave_exclusive_sum(r.kl, &tk);
        f += wave_sum(r.f);
        rq += wave_sum(r.rq);
        // the last line of the latest earlier list (lines never decrease along the units)
        uint64_t pl = wave_exclusive_max(r.last, &tot), plw = wave_exclusive_max(r.last_w, &totw);
        if (last > pl) pl = last;
        if (last_w > plw) plw = last_w;
        uint64_t d = r.first && pl == r.first ? twice : 0;
        if (r.first_w && plw == r.first_w) d += 1;
        dup += wave_sum(d);
        if (in) {
            UnitRec o = r;
            o.c = (uint32_t)(c + xc);
            o.ea = ea + xe;
            o.kl = kl + xk;
            rec[b + lane] = o;
        }
        c += tc;
        ea += te;
        kl += tk;
        last = last > tot ? last : tot;
        last_w = last_w > totw ? last_w : totw;
    }
    UnitRec r{};
    r.c = (uint32_t)c;
    r.f = (uint32_t)f;
    r.ea = ea;
    r.kl = kl;
    r.rq = sp.rq_distinct ? rq - dup : rq;
    return r;
}

// Partitions of several units, one wave each: their records joined and the engine chosen.
__global__ __launch_bounds__(256) void k_part_combine(Units un, const uint32_t* __restrict__ pv,
                                                      const uint64_t* __restrict__ off, SelParams sp,
                                                      uint8_t* __restrict__ mode, uint32_t* __restrict__ nA,
                                                      uint32_t* __restrict__ nF, uint64_t* __restrict__ Ea,
                                                      uint64_t* __restrict__ K) {
    const uint32_t k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= un.multis) return;  // the same for the whole wave
    const uint32_t i = un.multi[k];
    const UnitRec r = join_units(un.rec, un.first[i], un.first[i + 1], sp);
    if ((threadIdx.x & 63) == 0) {
        mode[i] = engine_of(i, off[pv[i + 1]] - off[pv[i]], r.c, r.ea, r.rq, sp);
        nA[i] = r.c;
        nF[i] = r.f;
        Ea[i] = r.ea;
        K[i] = r.kl;
    }
}

__global__ void k_select_only(uint64_t npart, const uint64_t* __restrict__ E, const uint64_t* __restrict__ nA,
                              const uint64_t* __restrict__ Ea, const uint64_t* __restrict__ Rq, SelParams sp,
                              uint8_t* __restrict__ p) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < npart;
         i += (uint64_t)gridDim.x * blockDim.x) {
        uint8_t r;
        if (Ea[i] == 0)
            r = P_NONE;
        else if (i < sp.nres)
            r = P_RES;
        else if (sp.force)
            r = (uint8_t)sp.force;
        else
            r = select_engine(E[i], nA[i], Ea[i], Rq[i], sp);
        p[i] = r;
    }
}

// -------------------------------------------------------------------- scan
// The engine segments' list and work offsets and the selection header.  Up to SCAN_ONE_MAX
// partitions one workgroup does it (k_scan_one below); past that, three launches: per tile of
// SCAN_TILE partitions the totals of every value (one workgroup per tile), then the segment
// starts and each tile's bases from the tile totals (one small workgroup), then per tile the
// offsets of each partition (one workgroup per tile).  Every thread takes a contiguous run of
// partitions, so a workgroup needs one barrier per pass.
constexpr int SCAN_NV = 4 * NSEG + 1;  // cnt[4], work[4], parts[4], edges[4], frontier
constexpr int SCAN_NB = 2 * NSEG;      // scanned per segment: list entries, work items
constexpr int SCAN_NW = SCAN_THREADS / 64;

// The values of partitions [i0, i1) summed into val[0, NV).
template <int NV>
__device__ __forceinline__ void scan_run_sums(uint32_t i0, uint32_t i1, const uint8_t* __restrict__ mode,
                                              const uint32_t* __restrict__ nA, const uint32_t* __restrict__ nF,
                                              const uint64_t* __restrict__ Ea,
                                              const uint64_t* __restrict__ K, uint64_t (&val)[NV]) {
#pragma unroll
    for (int k = 0; k < NV; k++) val[k] = 0;
    for (uint32_t i = i0; i < i1; i++) {
        if constexpr (NV == SCAN_NV) val[SCAN_NV - 1] += nF[i];
        const uint8_t m = mode[i];
        if (m == P_NONE) continue;
        const uint64_t ea = Ea[i], w = (m == P_ZC) ? K[i] : ea, na = nA[i];
#pragma unroll
        for (int sg = 0; sg < NSEG; sg++) {
            if (m != sg + 1) continue;
            val[sg] += na;
            val[NSEG + sg] += w;
            if (NV == SCAN_NV) {
                val[2 * NSEG + sg] += 1;
                val[3 * NSEG + sg] += ea;
            }
        }
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_tot(uint32_t npart, const uint8_t* __restrict__ mode,
                                                   const uint32_t* __restrict__ nA, const uint32_t* __restrict__ nF,
                                                   const uint64_t* __restrict__ Ea, const uint64_t* __restrict__ K,
                                                   uint64_t* __restrict__ tile_tot) {
    __shared__ uint64_t s_tot[SCAN_NW][SCAN_NV];
    const uint32_t i0 = min(blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_PER, npart), i1 = min(i0 + SCAN_PER, npart);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint64_t val[SCAN_NV];
    scan_run_sums<SCAN_NV>(i0, i1, mode, nA, nF, Ea, K, val);
#pragma unroll
    for (int k = 0; k < SCAN_NV; k++) {
        const uint64_t v = wave_sum(val[k]);
        if (lane == 0) s_tot[wid][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < SCAN_NV) {
        uint64_t t = 0;
        for (int w = 0; w < SCAN_NW; w++) t += s_tot[w][threadIdx.x];
        tile_tot[(uint64_t)blockIdx.x * SCAN_NV + threadIdx.x] = t;
    }
}

// The header's words besides the scan's: the lanes met (their word is cleared for the next
// selection) and the overflow lanes.
__device__ __forceinline__ void scan_extra(Header* hdr, const ScanExtra& x) {
    hdr->lanes = x.lanes ? *x.lanes : 0;
    if (x.lanes) *x.lanes = 0;
    hdr->overflow = x.overflow ? x.overflow[0] | ((uint64_t)x.overflow[1] << 32) : 0;
}

// One workgroup for up to 1024 * PER partitions, each thread a run of PER held in registers;
// segments without partitions (three of four when everything is resident) are skipped.  The
// header goes straight to pinned host memory, and after it (and the partitions' bases and
// modes, where the host asks for them) its number, which the host polls: no copy and no
// synchronisation between the selection and the pushes, and the list kernel overlaps the
// host's launches.  Bound by latency.  Measured per selection on R-MAT 22 (2,036 partitions):
// the three launches took 25 us of kernels, this one 8 us.
template <int PER>
__global__ __launch_bounds__(1024) void k_scan_one(uint32_t npart, const uint8_t* __restrict__ mode,
                                                   const uint32_t* __restrict__ nA, const uint32_t* __restrict__ nF,
                                                   const uint64_t* __restrict__ Ea, const uint64_t* __restrict__ K,
                                                   uint32_t* lbase, uint64_t* wbase,
                                                   uint64_t* __restrict__ wpre, ScanExtra x, ScanHost host) {
    constexpr int NW = 16;
    // per segment and wave: list entries, work, partitions, edges; then the waves' bases
    __shared__ uint64_t s_t[NSEG][4][NW];
    __shared__ uint64_t s_f[NW];
    __shared__ uint64_t s_tot[NSEG][4];
    const uint32_t t = threadIdx.x, lane = t & 63, wid = t >> 6, i0 = t * PER;
    uint32_t na[PER];
    uint8_t m[PER];
    uint64_t wk[PER], ze = 0, f = 0;  // ze: edges of the zero-copy partitions, whose work is lines
    uint32_t has = 0;
#pragma unroll
    for (int r = 0; r < PER; r++) {
        const uint32_t i = i0 + r;
        const bool in = i < npart;
        m[r] = in ? mode[i] : (uint8_t)P_NONE;
        na[r] = in ? nA[i] : 0u;
        wk[r] = in ? Ea[i] : 0ull;
        const uint64_t k = in ? K[i] : 0ull;
        f += in ? nF[i] : 0u;
        has |= 1u << m[r];
        if (m[r] == P_ZC) {
            ze += wk[r];
            wk[r] = k;
        }
    }
    for (uint32_t q = t; q < NSEG * 4 * NW; q += 1024) (&s_t[0][0][0])[q] = 0;
    f = wave_sum(f);
    if (lane == 0) s_f[wid] = f;
    __syncthreads();
    uint64_t xc[NSEG], xw[NSEG];
#pragma unroll
    for (int sg = 0; sg < NSEG; sg++) {
        xc[sg] = xw[sg] = 0;
        if (!__ballot((has >> (sg + 1)) & 1)) continue;  // uniform across the wave
        uint64_t c = 0, w = 0;
        uint32_t p = 0;
#pragma unroll
        for (int r = 0; r < PER; r++)
            if (m[r] == sg + 1) {
                c += na[r];
                w += wk[r];
                p += 1;
            }
        uint64_t tc, tw;
        xc[sg] = wave_exclusive_sum(c, &tc);
        xw[sg] = wave_exclusive_sum(w, &tw);
        const uint64_t tp = wave_sum(p), te = sg == SEG_Z ? wave_sum(ze) : tw;
        if (lane == 0) {
            s_t[sg][0][wid] = tc;
            s_t[sg][1][wid] = tw;
            s_t[sg][2][wid] = tp;
            s_t[sg][3][wid] = te;
        }
    }
    __syncthreads();
    if (t < NSEG * 4) {
        const int sg = t >> 2, k = t & 3;
        uint64_t run = 0;
        for (int w = 0; w < NW; w++) {
            const uint64_t y = s_t[sg][k][w];
            s_t[sg][k][w] = run;
            run += y;
        }
        s_tot[sg][k] = run;
    }
    __syncthreads();
    uint64_t la = 0, wa = 0, bc[NSEG], bw[NSEG];
#pragma unroll
    for (int sg = 0; sg < NSEG; sg++) {
        bc[sg] = la + s_t[sg][0][wid] + xc[sg];
        bw[sg] = wa + s_t[sg][1][wid] + xw[sg];
        la += s_tot[sg][0];
        wa += s_tot[sg][1];
    }
#pragma unroll
    for (int r = 0; r < PER; r++) {
        const uint32_t i = i0 + r;
        if (i >= npart) break;
        uint32_t lb = 0xFFFFFFFFu;
        uint64_t wb = ~0ull;
#pragma unroll
        for (int sg = 0; sg < NSEG; sg++)
            if (m[r] == sg + 1) {
                lb = (uint32_t)bc[sg];
                wb = bw[sg];
                bc[sg] += na[r];
                bw[sg] += wk[r];
            }
        lbase[i] = lb;
        wbase[i] = wb;
    }
    if (t == 0) {
        Header* hdr = host.hdr;
        uint64_t l = 0, w = 0, fr = 0;
#pragma unroll
        for (int sg = 0; sg < NSEG; sg++) {
            hdr->seg_parts[sg] = (uint32_t)s_tot[sg][2];
            hdr->seg_list_start[sg] = (uint32_t)l;
            hdr->seg_list_count[sg] = (uint32_t)s_tot[sg][0];
            hdr->seg_work_start[sg] = w;
            hdr->seg_work_total[sg] = s_tot[sg][1];
            hdr->seg_edges[sg] = s_tot[sg][3];
            l += s_tot[sg][0];
            w += s_tot[sg][1];
        }
        for (int q = 0; q < NW; q++) fr += s_f[q];
        hdr->total_active = l;
        hdr->frontier = fr;
        scan_extra(hdr, x);
        wpre[l] = w;
    }
    if (host.mode) {
        // across the link in whole lines: a thread's own run of entries took a transaction each
        __syncthreads();
        for (uint32_t i = t; i < npart; i += 1024) {
            host.wbase[i] = wbase[i];
            host.lbase[i] = lbase[i];
            host.mode[i] = mode[i];
        }
    }
    __threadfence_system();
    __syncthreads();
    if (t == 0) __hip_atomic_store(&host.hdr->seq, host.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One workgroup of 64 threads: grand totals, segment starts (segments lie one after another:
// RESIDENT, FILTER, ZEROCOPY, COMPACT), each tile's bases, the header, and the work prefix's
// closing entry.
__global__ __launch_bounds__(64) void k_scan_base(uint32_t ntiles, const uint64_t* __restrict__ tile_tot,
                                                  uint64_t* __restrict__ tile_base, Header* __restrict__ hdr,
                                                  uint64_t* __restrict__ wpre, ScanExtra x) {
    __shared__ uint64_t s_g[SCAN_NV];
    const uint32_t k = threadIdx.x;
    if (k < SCAN_NV) {
        uint64_t t = 0;
        for (uint32_t i = 0; i < ntiles; i++) t += tile_tot[(uint64_t)i * SCAN_NV + k];
        s_g[k] = t;
    }
    __syncthreads();
    if (k < SCAN_NB) {
        const uint32_t sg = k % NSEG, first = k - sg;  // first: 0 (list entries) or NSEG (work)
        uint64_t run = 0;
        for (uint32_t s2 = 0; s2 < sg; s2++) run += s_g[first + s2];
        for (uint32_t i = 0; i < ntiles; i++) {
            tile_base[(uint64_t)i * SCAN_NB + k] = run;
            run += tile_tot[(uint64_t)i * SCAN_NV + k];
        }
    }
    if (k == 0) {
        uint64_t la = 0, wa = 0;
#pragma unroll
        for (int sg = 0; sg < NSEG; sg++) {
            hdr->seg_parts[sg] = (uint32_t)s_g[2 * NSEG + sg];
            hdr->seg_list_start[sg] = (uint32_t)la;
            hdr->seg_list_count[sg] = (uint32_t)s_g[sg];
            hdr->seg_work_start[sg] = wa;
            hdr->seg_work_total[sg] = s_g[NSEG + sg];
            hdr->seg_edges[sg] = s_g[3 * NSEG + sg];
            la += s_g[sg];
            wa += s_g[NSEG + sg];
        }
        hdr->total_active = la;
        hdr->frontier = s_g[SCAN_NV - 1];
        scan_extra(hdr, x);
        wpre[la] = wa;
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_write(uint32_t npart, const uint8_t* __restrict__ mode,
                                                     const uint32_t* __restrict__ nA, const uint64_t* __restrict__ Ea,
                                                     const uint64_t* __restrict__ K,
                                                     const uint64_t* __restrict__ tile_base,
                                                     uint32_t* __restrict__ lbase, uint64_t* __restrict__ wbase) {
    __shared__ uint64_t s_tot[SCAN_NW][SCAN_NB];
    const uint32_t i0 = min(blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_PER, npart), i1 = min(i0 + SCAN_PER, npart);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint64_t val[SCAN_NB];
    scan_run_sums<SCAN_NB>(i0, i1, mode, nA, nullptr, Ea, K, val);
    uint64_t ex[SCAN_NB];
#pragma unroll
    for (int k = 0; k < SCAN_NB; k++) {
        uint64_t v = val[k];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t y = __shfl_up(v, d, 64);
            if (lane >= d) v += y;
        }
        ex[k] = v - val[k];
        if (lane == 63) s_tot[wid][k] = v;
    }
    __syncthreads();
    uint64_t run[SCAN_NB];
#pragma unroll
    for (int k = 0; k < SCAN_NB; k++) {
        uint64_t before = 0;
        for (int w = 0; w < wid; w++) before += s_tot[w][k];
        run[k] = tile_base[(uint64_t)blockIdx.x * SCAN_NB + k] + before + ex[k];
    }
    for (uint32_t i = i0; i < i1; i++) {
        const uint8_t m = mode[i];
        uint32_t lb = 0xFFFFFFFFu;
        uint64_t wb = ~0ull;
#pragma unroll
        for (int sg = 0; sg < NSEG; sg++) {
            if (m != sg + 1) continue;
            lb = (uint32_t)run[sg];
            wb = run[NSEG + sg];
            run[sg] += nA[i];
            run[NSEG + sg] += (m == P_ZC) ? K[i] : Ea[i];
        }
        lbase[i] = lb;
        wbase[i] = wb;
    }
}

// ------------------------------------------------------------------ lists
// One wave per unit of the scheduled partitions, dealing out its active vertices as in
// k_unit_stats; a batch's entries are written in lane order, so the stores coalesce.
// Batches [b0, b0 + 64 G) of a round's active vertices, loaded as in stats_batches; the
// entries of vertices with edges go to list[pos...) in lane order with their work prefix.
template <int G>
__device__ __forceinline__ void list_batches(uint32_t b0, uint32_t T, uint32_t incl, uint32_t cnt, uint64_t wbits,
                                             uint32_t q0, const uint64_t* __restrict__ off, bool by_lines,
                                             uint32_t* __restrict__ list, uint64_t* __restrict__ wpre,
                                             uint32_t* __restrict__ tile, uint64_t& pos, uint64_t& wp) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    uint64_t s[G], e[G];
    uint32_t vv[G];
#pragma unroll
    for (int g = 0; g < G; g++) {
        const uint32_t k = b0 + 64 * g + lane;
        vv[g] = round_vertex(k < T ? k : T - 1, incl, cnt, wbits, q0);
        s[g] = off[vv[g]];
        e[g] = off[vv[g] + 1];
    }
#pragma unroll
    for (int g = 0; g < G; g++) {
        if (b0 + 64 * g >= T) break;
        const bool has = b0 + 64 * g + lane < T && e[g] > s[g];
        const uint64_t A = __ballot(has);
        const uint64_t wk = has ? (by_lines ? lines_of(s[g], e[g], ZC_LINE_SHIFT) : e[g] - s[g]) : 0;
        uint64_t tw;
        const uint64_t ew = wave_exclusive_sum(wk, &tw);
        if (has) {
            const uint64_t at = pos + __popcll(A & below);
            list[at] = vv[g];
            const uint64_t w0 = wp + ew;
            wpre[at] = w0;
            // the tiles whose first item is this entry's
            const uint32_t sh = by_lines ? LINE_TILE_SHIFT : EDGE_TILE_SHIFT;
            const uint64_t t1 = (w0 + wk - 1) >> sh;
            for (uint64_t t = (w0 + (1u << sh) - 1) >> sh; t <= t1; t++) tile[t] = (uint32_t)at;
        }
        pos += __popcll(A);
        wp += tw;
    }
}

// The list entries of unit u (of a partition with engine m), from list position pos and work
// position wp on.
__device__ __forceinline__ void unit_list(const Units& un, uint32_t u, uint32_t m, uint64_t pos, uint64_t wp,
                                          const uint32_t* __restrict__ pv, const uint64_t* __restrict__ off,
                                          const uint32_t* __restrict__ cur, uint32_t* __restrict__ list,
                                          uint64_t* __restrict__ wpre, uint32_t* __restrict__ tile_e,
                                          uint32_t* __restrict__ tile_l) {
    const uint32_t lane = threadIdx.x & 63;
    const bool by_lines = m == P_ZC;
    const uint32_t i = un.part[u], q0 = un.q[u];
    const uint32_t vb = pv[i], ve = pv[i + 1];
    const uint32_t qe = min(q0 + un.windows, (ve + 63) >> 6);
    const uint64_t wbits = q0 + lane < qe ? window_bits(cur, q0 + lane, vb, ve) : 0ull;
    if (!__ballot(wbits != 0)) return;
    const uint32_t cnt = __popcll(wbits);
    const uint32_t incl = wave_inclusive_sum_u32(cnt);
    const uint32_t T = __shfl(incl, 63, 64);
    uint32_t* tile = by_lines ? tile_l : tile_e;
    if (T <= 64)
        list_batches<1>(0, T, incl, cnt, wbits, q0, off, by_lines, list, wpre, tile, pos, wp);
    else
        for (uint32_t b0 = 0; b0 < T; b0 += 64 * SEL_B)
            list_batches<SEL_B>(b0, T, incl, cnt, wbits, q0, off, by_lines, list, wpre, tile, pos, wp);
}

__global__ __launch_bounds__(256) void k_build_lists(Units un, const uint32_t* __restrict__ pv,
                                                     const uint64_t* __restrict__ off,
                                                     const uint32_t* __restrict__ cur,
                                                     const uint8_t* __restrict__ mode,
                                                     const uint32_t* __restrict__ lbase,
                                                     const uint64_t* __restrict__ wbase,
                                                     uint32_t* __restrict__ list, uint64_t* __restrict__ wpre,
                                                     uint32_t* __restrict__ tile_e, uint32_t* __restrict__ tile_l) {
    const uint32_t wpb = blockDim.x >> 6, waves = gridDim.x * wpb;
    for (uint32_t u = blockIdx.x * wpb + (threadIdx.x >> 6); u < un.count; u += waves) {
        const uint32_t i = un.part[u];
        const uint8_t m = mode[i];
        if (m == P_NONE) continue;  // uniform across the wave
        uint64_t pos = lbase[i], wp = wbase[i];
        if (un.first[i + 1] - un.first[i] > 1) {  // after the partition's earlier units
            pos += un.rec[u].c;
            wp += m == P_ZC ? un.rec[u].kl : un.rec[u].ea;
        }
        unit_list(un, u, m, pos, wp, pv, off, cur, list, wpre, tile_e, tile_l);
    }
}

// The whole selection of a small graph (at most SMALL_UNITS units) in one workgroup: the units'
// records (in LDS), their partitions joined and their engines chosen, the segments laid out
// by one wave with the header reported to the host, and the lists written while the host
// reads it.  Four launches, whose gaps are as long as their work on such a graph, become one.
__global__ __launch_bounds__(1024) void k_select_small(uint32_t npart, Units un, const uint32_t* __restrict__ pv,
                                                       const uint64_t* __restrict__ off,
                                                       const uint32_t* __restrict__ cur,
                                                       uint32_t* __restrict__ clear, uint32_t nwords,
                                                       const uint64_t* __restrict__ mcur, SelParams sp,
                                                       uint8_t* __restrict__ mode, uint32_t* __restrict__ list,
                                                       uint64_t* __restrict__ wpre, uint32_t* __restrict__ tile_e,
                                                       uint32_t* __restrict__ tile_l, bool lists, ScanExtra x,
                                                       ScanHost host) {
    __shared__ UnitRec s_rec[SMALL_UNITS];  // per unit
    __shared__ UnitRec s_part[SMALL_UNITS];  // per partition: joined
    __shared__ uint32_t s_mode[SMALL_UNITS], s_lb[SMALL_UNITS];
    __shared__ uint64_t s_wb[SMALL_UNITS];
    __shared__ unsigned long long s_lanes;
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_lanes = 0;
    __syncthreads();
    for (uint32_t u = wid; u < un.count; u += 16) {
        uint64_t lm = 0;
        const UnitRec r = unit_record<false>(un, u, pv, off, cur, clear, nwords, mcur, sp, LevelScan{}, &lm);
        if (lane == 0) {
            s_rec[u] = r;
            if (lm) atomicOr(&s_lanes, (unsigned long long)lm);
        }
    }
    __syncthreads();
    for (uint32_t i = wid; i < npart; i += 16) {
        const UnitRec r = join_units(s_rec, un.first[i], un.first[i + 1], sp);
        if (lane == 0) {
            s_part[i] = r;
            s_mode[i] = engine_of(i, off[pv[i + 1]] - off[pv[i]], r.c, r.ea, r.rq, sp);
        }
    }
    __syncthreads();
    if (wid == 0) {  // npart <= un.count: lane i holds partition i
        const bool in = lane < npart;
        UnitRec r{};
        if (in) r = s_part[lane];
        const uint32_t m = in ? s_mode[lane] : (uint32_t)P_NONE;
        const uint64_t wk = m == P_ZC ? r.kl : r.ea;
        Header* hdr = host.hdr;
        uint64_t l = 0, w = 0;
        uint32_t lb = 0xFFFFFFFFu;
        uint64_t wb = ~0ull;
        for (int sg = 0; sg < NSEG; sg++) {
            const bool mine = m == (uint32_t)sg + 1;
            const uint64_t who = __ballot(mine);
            uint64_t tc = 0, tw = 0, te = 0;
            if (who) {  // uniform
                const uint64_t xc = wave_exclusive_sum(mine ? r.c : 0u, &tc);
                const uint64_t xw = wave_exclusive_sum(mine ? wk : 0ull, &tw);
                te = sg == SEG_Z ? wave_sum(mine ? r.ea : 0ull) : tw;
                if (mine) {
                    lb = (uint32_t)(l + xc);
                    wb = w + xw;
                }
            }
            if (lane == 0) {
                hdr->seg_parts[sg] = (uint32_t)__popcll(who);
                hdr->seg_list_start[sg] = (uint32_t)l;
                hdr->seg_list_count[sg] = (uint32_t)tc;
                hdr->seg_work_start[sg] = w;
                hdr->seg_work_total[sg] = tw;
                hdr->seg_edges[sg] = te;
            }
            l += tc;
            w += tw;
        }
        const uint64_t fr = wave_sum(r.f);
        if (in) {
            s_lb[lane] = lb;
            s_wb[lane] = wb;
            mode[lane] = (uint8_t)m;
            if (host.mode) {
                host.lbase[lane] = lb;
                host.wbase[lane] = wb;
                host.mode[lane] = (uint8_t)m;
            }
        }
        if (lane == 0) {
            hdr->total_active = l;
            hdr->frontier = fr;
            scan_extra(hdr, x);
            hdr->lanes = s_lanes;
            wpre[l] = w;
        }
        __threadfence_system();
        if (lane == 0) __hip_atomic_store(&hdr->seq, host.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (!lists) return;
    __syncthreads();
    for (uint32_t u = wid; u < un.count; u += 16) {
        const uint32_t i = un.part[u], m = s_mode[i];
        if (m == P_NONE) continue;  // uniform across the wave
        unit_list(un, u, m, s_lb[i] + (uint64_t)s_rec[u].c, s_wb[i] + (m == P_ZC ? s_rec[u].kl : s_rec[u].ea), pv, off,
                  cur, list, wpre, tile_e, tile_l);
    }
}

// --------------------------------------------------------------- operators
// src(u): the value u pushes (read when the workgroup stages its vertices; it may
// already reflect updates made earlier in the same iteration, which only helps the
// monotone operators).  Relaxing edge (u, v) with weight w is split into steps that a thread
// takes for several edges side by side (push_batch), so that each step's accesses are in
// flight together: probe(v) reads the target's state, want(value, p, w) decides from it
// whether the edge may improve it, update(...) makes the atomic update and returns the old
// state, and mark(...) records an improvement.  Probes are ordinary loads that may return a
// value of earlier in the kernel: states only move one way, so an old one lets at most an
// unneeded update through, and the update's own result decides.
// mark_next sets v's bit in a bitmap unless it is seen there already.
__device__ __forceinline__ void mark_next(uint32_t* map, uint32_t v) {
    const uint32_t bit = 1u << (v & 31);
    if (!(map[v >> 5] & bit)) atomicOr(map + (v >> 5), bit);
}

// An operator that relaxes a thread's edges in its own way: push_many(ok, val, v).
struct BatchOp {};

struct OpBfs {
    static constexpr bool steps = true;
    static constexpr bool weighted = false;
    uint32_t* visited;
    uint32_t* next;
    uint32_t* lvl;
    uint32_t level_next;
    __device__ __forceinline__ uint32_t src(uint32_t) const { return 0; }
    __device__ __forceinline__ uint32_t probe(uint32_t v) const { return visited[v >> 5]; }
    __device__ __forceinline__ bool want(uint32_t, uint32_t v, uint32_t, uint32_t p) const { return !((p >> (v & 31)) & 1); }
    __device__ __forceinline__ uint32_t update(uint32_t, uint32_t v, uint32_t) const {
        return atomicOr(visited + (v >> 5), 1u << (v & 31));
    }
    __device__ __forceinline__ void mark(uint32_t, uint32_t v, uint32_t, uint32_t old) const {
        if ((old >> (v & 31)) & 1) return;  // exactly one thread discovers v
        lvl[v] = level_next;
        atomicOr(next + (v >> 5), 1u << (v & 31));
    }
};

// A wide iteration's BFS: discoveries are plain stores of the level (every thread that finds v
// undiscovered stores the same one), and the next selection takes the frontier from the
// levels.  OpBfs is bound by its two atomics per discovery, which go past the L2 to bitmaps
// with few hot lines, about 10 G/s (random ones 27): R-MAT 22, 14M and 49M active edges with
// 2.4M and 1.4M atomic requests, 324 and 518 us; the whole traversal 1.55 -> 1.06 ms.
struct OpBfsWide {
    static constexpr bool steps = true;
    static constexpr bool weighted = false;
    const uint32_t* visited;  // as of the iteration's start
    uint32_t* lvl;
    uint32_t level_next;
    __device__ __forceinline__ uint32_t src(uint32_t) const { return 0; }
    __device__ __forceinline__ uint32_t probe(uint32_t v) const { return visited[v >> 5]; }
    __device__ __forceinline__ bool want(uint32_t, uint32_t v, uint32_t, uint32_t p) const { return !((p >> (v & 31)) & 1); }
    __device__ __forceinline__ uint32_t update(uint32_t, uint32_t v, uint32_t) const {
        lvl[v] = level_next;
        return 0;
    }
    __device__ __forceinline__ void mark(uint32_t, uint32_t, uint32_t, uint32_t) const {}
};

struct OpSssp {
    static constexpr bool steps = true;
    static constexpr bool weighted = true;
    uint32_t* dist;
    uint32_t* next;
    uint32_t* overflow;
    uint32_t* far;   // improved vertices at or above `bound` wait here (bound 0xFFFFFFFF: never)
    uint32_t bound;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return dist[u]; }
    __device__ __forceinline__ uint32_t probe(uint32_t v) const { return dist[v]; }
    __device__ __forceinline__ bool want(uint32_t du, uint32_t, uint32_t w, uint32_t p) const {
        const uint64_t nd = (uint64_t)du + w;
        if (nd >= UNREACHED) {
            *overflow = 1u;
            return false;
        }
        return (uint32_t)nd < p;
    }
    __device__ __forceinline__ uint32_t update(uint32_t du, uint32_t v, uint32_t w) const {
        return atomicMin(dist + v, du + w);
    }
    __device__ __forceinline__ void mark(uint32_t du, uint32_t v, uint32_t w, uint32_t old) const {
        const uint32_t nd = du + w;
        if (nd < old) mark_next(nd < bound ? next : far, v);
    }
};

// A wide iteration's SSSP: improved vertices are marked by plain byte stores.
struct OpSsspWide : OpSssp {
    uint8_t* marks;
    uint8_t tag;
    __device__ __forceinline__ void mark(uint32_t du, uint32_t v, uint32_t w, uint32_t old) const {
        if (du + w < old) marks[v] = tag;
    }
};

struct OpBfsRelax {
    static constexpr bool steps = true;
    static constexpr bool weighted = false;
    uint32_t* lvl;
    uint32_t* next;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return lvl[u]; }
    __device__ __forceinline__ uint32_t probe(uint32_t v) const { return lvl[v]; }
    __device__ __forceinline__ bool want(uint32_t lu, uint32_t, uint32_t, uint32_t p) const { return lu + 1 < p; }
    __device__ __forceinline__ uint32_t update(uint32_t lu, uint32_t v, uint32_t) const {
        return atomicMin(lvl + v, lu + 1);
    }
    __device__ __forceinline__ void mark(uint32_t lu, uint32_t v, uint32_t, uint32_t old) const {
        if (lu + 1 < old) mark_next(next, v);
    }
};

struct OpCc {
    static constexpr bool steps = true;
    static constexpr bool weighted = false;
    uint32_t* lab;
    uint32_t* next;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return lab[u]; }
    __device__ __forceinline__ uint32_t probe(uint32_t v) const { return lab[v]; }
    __device__ __forceinline__ bool want(uint32_t lu, uint32_t, uint32_t, uint32_t p) const { return lu < p; }
    __device__ __forceinline__ uint32_t update(uint32_t lu, uint32_t v, uint32_t) const { return atomicMin(lab + v, lu); }
    __device__ __forceinline__ void mark(uint32_t lu, uint32_t v, uint32_t, uint32_t old) const {
        if (lu < old) mark_next(next, v);
    }
};

struct OpCcWide : OpCc {
    uint8_t* marks;
    uint8_t tag;
    __device__ __forceinline__ void mark(uint32_t lu, uint32_t v, uint32_t, uint32_t old) const {
        if (lu < old) marks[v] = tag;
    }
};

// Join the trees of u and v in a parent forest whose parents are smaller ids: the larger of the
// two walked-to ids climbs to its parent, or, a root, is hooked below the smaller one.  Every
// step lowers the larger id (a failed hook returns the parent someone else set), so it ends
// whatever the loads return; a root stays the smallest id of its tree.
__device__ __forceinline__ void link_trees(uint32_t* par, uint32_t u, uint32_t v) {
    uint32_t a = __hip_atomic_load(par + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t b = __hip_atomic_load(par + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (a != b) {
        if (a < b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        uint32_t p = __hip_atomic_load(par + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (p == a) {
            p = atomicCAS(par + a, a, b);
            if (p == a) return;
        }
        a = p;
    }
}

// Components over a parent forest: every edge joins its ends' trees.
struct OpLink {
    static constexpr bool wave = false, steps = false;
    static constexpr bool weighted = false;
    uint32_t* par;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return u; }
    __device__ __forceinline__ void push(uint32_t u, uint32_t v, uint32_t) const { link_trees(par, u, v); }
};

// Accumulator copy of the XCD (accelerator complex die) the wave runs on, masked to the
// copies in use.  Any value in [0, copies) would be correct -- the adds are device-scope
// atomics and the copies are summed afterwards -- the die id just keeps each copy's lines in
// few dies' L2 and splits the adds aimed at one hub vertex `copies` ways.
__device__ __forceinline__ uint32_t acc_copy(uint32_t cmask) {
    uint32_t x;
    asm("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(x));
    return x & cmask;
}

struct OpPr {
    static constexpr bool wave = false, steps = false;
    static constexpr bool weighted = false;
    float* acc;
    uint64_t stride;  // floats per accumulator copy
    const float* contrib;
    uint32_t cmask;   // copies in use - 1
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return __float_as_uint(contrib[u]); }
    __device__ __forceinline__ void push(uint32_t c, uint32_t v, uint32_t) const {
        unsafeAtomicAdd(acc + acc_copy(cmask) * stride + acc_slot(v), __uint_as_float(c));
    }
};

// Batched BFS: lanes of u's mask that have not reached v yet reach it now (one 64-bit
// atomicOr decides, per lane, which edge discovers v first).  The staged value is u.
struct OpMBfs {
    static constexpr bool wave = false, steps = false;
    static constexpr bool weighted = false;
    const uint64_t* mcur;
    uint64_t* mnext;
    uint64_t* mvisited;
    uint32_t* lvl;   // n rows of 2^lshift lanes
    uint32_t* next;  // union of the next frontier
    uint32_t level_next;
    uint32_t lshift;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return u; }
    __device__ __forceinline__ void push(uint32_t u, uint32_t v, uint32_t) const {
        const uint64_t want = mcur[u] & ~mvisited[v];
        if (!want) return;
        const uint64_t old = atomicOr((unsigned long long*)(mvisited + v), (unsigned long long)want);
        uint64_t gained = want & ~old;
        if (!gained) return;
        atomicOr((unsigned long long*)(mnext + v), (unsigned long long)gained);
        mark_next(next, v);
        uint32_t* row = lvl + ((uint64_t)v << lshift);
        while (gained) {
            row[__ffsll((unsigned long long)gained) - 1] = level_next;
            gained &= gained - 1;
        }
    }
};

// A wide iteration's batched BFS: the lanes an edge may improve are added to mnext only; the
// lanes reached, the levels and the frontier bitmap follow from it at the iteration's end
// (k_settle_lanes).  OpMBfs updates a second mask and the bitmap atomically and stores a
// target's levels one lane after another: R-MAT 20, 64 lanes, resident pushes of two wide
// iterations 547 and 413 us alone, 228 us and (beside a stream) 531 us here with 40 us each
// to settle, the call 9.56 -> 9.42 ms of which the host link takes 7.7.
struct OpMBfsWide : BatchOp {
    static constexpr bool steps = false;
    static constexpr bool weighted = false;
    const uint64_t* mcur;
    uint64_t* mnext;
    const uint64_t* mvisited;  // as of the iteration's start
    explicit OpMBfsWide(const AlgoState& s) : mcur(s.mcur), mnext(s.mnext), mvisited(s.mvisited) {}
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return u; }
    template <int N>
    __device__ __forceinline__ void push_many(const bool (&ok)[N], const uint32_t (&u)[N],
                                              const uint32_t (&v)[N]) const {
        uint64_t m[N], seen[N];
#pragma unroll
        for (int r = 0; r < N; r++) {
            m[r] = ok[r] ? mcur[u[r]] : 0ull;
            seen[r] = ok[r] ? mvisited[v[r]] | mnext[v[r]] : 0ull;
        }
#pragma unroll
        for (int r = 0; r < N; r++)
            if (m[r] & ~seen[r]) atomicOr((unsigned long long*)(mnext + v[r]), (unsigned long long)(m[r] & ~seen[r]));
    }
};

// Batched SSSP: every lane active at u relaxes (u, v) in its own distance row.  WU: edges that a
// thread of the wave form takes side by side.
template <int WU>
struct OpMSssp {
    static constexpr bool wave = true, steps = false;
    static constexpr bool weighted = true;
    const uint64_t* mcur;
    uint64_t* mnext;
    uint32_t* dist;      // n rows of 2^lshift lanes
    uint32_t* next;      // union of the next frontier
    uint32_t* overflow;  // two words of lane bits: lanes whose distance would overflow
    uint32_t lshift;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return u; }
    __device__ __forceinline__ void push(uint32_t u, uint32_t v, uint32_t w) const {
        uint64_t m = mcur[u], gained = 0;
        const uint32_t* du = dist + ((uint64_t)u << lshift);
        uint32_t* dv = dist + ((uint64_t)v << lshift);
        while (m) {
            const uint32_t l = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            const uint64_t nd = (uint64_t)du[l] + w;
            if (nd >= UNREACHED) {
                atomicOr(overflow + (l >> 5), 1u << (l & 31));
                continue;
            }
            if ((uint32_t)nd < dv[l]) {
                const uint32_t old = atomicMin(dv + l, (uint32_t)nd);
                if ((uint32_t)nd < old) gained |= 1ull << l;
            }
        }
        if (gained) {
            atomicOr((unsigned long long*)(mnext + v), (unsigned long long)gained);
            mark_next(next, v);
        }
    }
    // Wave form (see OpMPpr::push_wave): each pass gives 64 >> lshift of the wave's edges one
    // thread per lane, so an edge's relaxations are one atomicMin instruction over its
    // contiguous distance row; the lanes that improved are collected by ballot and one
    // thread per edge marks them.  The wave's edges are first moved to its front, and WU of
    // them per thread go through each step together, so that their rows are in flight at once
    // (one at a time, 262K vertices with 37 lanes: 0.93 ms of the widest iteration's 4M edges).
    // It pays when the rows are dense (a batch started together); when the wave's edges
    // carry fewer than a quarter row of active lanes on average (queries at different stages)
    // each thread relaxes its own edge's lanes.  Called by every thread of the wave.
    __device__ __forceinline__ void push_wave(bool ok, uint32_t u, uint32_t v, uint32_t w) const {
        uint32_t active = ok ? (uint32_t)__popcll(mcur[u]) : 0u;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) active += __shfl_xor(active, d, 64);
        const uint64_t act = __ballot(ok);
        const uint32_t cnt = __popcll(act);
        if (lshift < 3 || active * 4 < (cnt << lshift)) {
            if (ok) push(u, v, w);
            return;
        }
        const uint32_t me = __lane_id();
        const uint32_t slot = me >> lshift, ln = me & ((1u << lshift) - 1);
        const uint32_t per = 64u >> lshift;
        const uint64_t rowmask = lshift >= 6 ? ~0ull : ((1ull << (1u << lshift)) - 1);
        const uint64_t below = (1ull << me) - 1ull;
        const int to = (int)((ok ? __popcll(act & below) : cnt + __popcll(~act & below)) << 2);
        const int uc = __builtin_amdgcn_ds_permute(to, (int)u), vc = __builtin_amdgcn_ds_permute(to, (int)v);
        const int wc = __builtin_amdgcn_ds_permute(to, (int)w);
        for (uint32_t j = 0; j < cnt; j += WU * per) {
            uint32_t vv[WU], nd[WU], dv[WU];
            bool go[WU];
#pragma unroll
            for (int r = 0; r < WU; r++) {
                const uint32_t q = j + r * per + slot;
                const int from = (int)(q & 63);
                const uint32_t uu = (uint32_t)__shfl(uc, from, 64), ww = (uint32_t)__shfl(wc, from, 64);
                vv[r] = (uint32_t)__shfl(vc, from, 64);
                go[r] = q < cnt && ((mcur[uu] >> ln) & 1);
                const uint64_t x = go[r] ? (uint64_t)dist[((uint64_t)uu << lshift) + ln] + ww : 0ull;
                dv[r] = go[r] ? dist[((uint64_t)vv[r] << lshift) + ln] : 0u;
                if (x >= UNREACHED) {
                    atomicOr(overflow + (ln >> 5), 1u << (ln & 31));
                    go[r] = false;
                }
                nd[r] = (uint32_t)x;
            }
#pragma unroll
            for (int r = 0; r < WU; r++) {
                go[r] = go[r] && nd[r] < dv[r];
                if (go[r]) dv[r] = atomicMin(dist + ((uint64_t)vv[r] << lshift) + ln, nd[r]);
            }
#pragma unroll
            for (int r = 0; r < WU; r++) {
                const uint64_t g = (__ballot(go[r] && nd[r] < dv[r]) >> (slot << lshift)) & rowmask;
                if (ln == 0 && g) {
                    atomicOr((unsigned long long*)(mnext + vv[r]), (unsigned long long)g);
                    mark_next(next, vv[r]);
                }
            }
        }
    }
};

// Batched personalized PageRank: every lane active at u adds its share x_u / D_o(u)
// (prepared in place in u's row, FP32) into v's accumulator row (FP64: a hub's value is a
// sum of up to ~10^5 shares per step, which FP32 adds in atomic order would carry ~1e-4
// relative error; in FP64 only the FP32 rounding of x and of the shares remains).
struct OpMPpr {
    static constexpr bool wave = true, steps = false;
    static constexpr bool weighted = false;
    const uint64_t* mcur;
    uint64_t* mnext;
    const float* share;  // n rows of 2^lshift lanes
    double* acc;         // n rows of 2^lshift lanes
    uint32_t* next;      // union of the next frontier
    uint32_t lshift;
    __device__ __forceinline__ uint32_t src(uint32_t u) const { return u; }
    __device__ __forceinline__ void push(uint32_t u, uint32_t v, uint32_t) const {
        const uint64_t m = mcur[u];
        if (!m) return;
        const float* su = share + ((uint64_t)u << lshift);
        double* av = acc + ((uint64_t)v << lshift);
        uint64_t b = m;
        while (b) {
            const uint32_t l = __ffsll((unsigned long long)b) - 1;
            b &= b - 1;
            unsafeAtomicAdd(av + l, (double)su[l]);
        }
        mark(m, v);
    }
    __device__ __forceinline__ void mark(uint64_t m, uint32_t v) const {
        if ((__builtin_nontemporal_load(mnext + v) & m) != m) atomicOr((unsigned long long*)(mnext + v), (unsigned long long)m);
        const uint32_t bit = 1u << (v & 31);
        if (!(__builtin_nontemporal_load(next + (v >> 5)) & bit)) atomicOr(next + (v >> 5), bit);
    }
    // The wave's edges (threads with ok) spread over the wave: each pass gives 64 >> lshift
    // edges one thread per lane, so the adds of one edge are one instruction over a
    // contiguous accumulator row instead of one instruction per lane.  Called by every
    // thread of the wave.
    __device__ __forceinline__ void push_wave(bool ok, uint32_t u, uint32_t v, uint32_t) const {
        if (lshift < 3) {  // rows of 1..4 lanes: one thread per edge
            if (ok) push(u, v, 0);
            return;
        }
        const uint32_t me = __lane_id();
        const uint32_t slot = me >> lshift, ln = me & ((1u << lshift) - 1);
        const uint32_t per = 64u >> lshift;
        uint64_t act = __ballot(ok);
        while (act) {
            uint64_t a = act;
            for (uint32_t k = 0; k < slot; k++) a &= a - 1;
            const int from = a ? (int)__ffsll((unsigned long long)a) - 1 : 0;
            const uint32_t uu = __shfl(u, from, 64), vv = __shfl(v, from, 64);
            if (a && ((mcur[uu] >> ln) & 1))
                unsafeAtomicAdd(acc + ((uint64_t)vv << lshift) + ln, (double)share[((uint64_t)uu << lshift) + ln]);
            for (uint32_t k = 0; k < per && act; k++) act &= act - 1;
        }
        if (ok) {
            const uint64_t m = mcur[u];
            if (m) mark(m, v);
        }
    }
};

// Relax N edges per thread where ok holds, called by every thread of the wave together:
// operators in steps take each step for all N, those with a wave form (Op::wave) share an
// edge's work across the wave.
// On R-MAT 22 BFS's widest iteration (49M edges) one edge after another, with probes past the
// caches, took 1.45 ms.
template <int N, class Op>
__device__ __forceinline__ void push_batch(const Op& op, const bool (&ok)[N], const uint32_t (&val)[N],
                                           const uint32_t (&v)[N], const uint32_t (&w)[N]) {
    if constexpr (std::is_base_of<BatchOp, Op>::value) {
        op.push_many(ok, val, v);
    } else if constexpr (Op::steps) {
        uint32_t p[N];
        bool go[N];
#pragma unroll
        for (int r = 0; r < N; r++) p[r] = op.probe(ok[r] ? v[r] : 0u);
#pragma unroll
        for (int r = 0; r < N; r++) go[r] = ok[r] && op.want(val[r], v[r], w[r], p[r]);
#pragma unroll
        for (int r = 0; r < N; r++)
            if (go[r]) p[r] = op.update(val[r], v[r], w[r]);
#pragma unroll
        for (int r = 0; r < N; r++)
            if (go[r]) op.mark(val[r], v[r], w[r], p[r]);
    } else {
#pragma unroll
        for (int r = 0; r < N; r++) {
            if constexpr (Op::wave)
                op.push_wave(ok[r], val[r], v[r], w[r]);
            else if (ok[r])
                op.push(val[r], v[r], w[r]);
        }
    }
}

// Largest j in [lo, hi) with pred(j) true, for a predicate that is true on a prefix of
// [lo, hi) and true at lo.  The whole workgroup searches together: each round every
// thread probes one of blockDim.x evenly spaced positions, so a range of N entries takes
// about log(N)/log(blockDim.x) rounds of independent loads instead of log2(N) dependent
// ones.  Every thread of the block must call it with the same arguments.
template <class Pred>
__device__ __forceinline__ uint32_t block_search_last(uint32_t lo, uint32_t hi, Pred pred, uint32_t* s_tmp) {
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + blockDim.x - 1) / blockDim.x;
        const uint32_t p = lo + threadIdx.x * step;
        const bool ok = p < hi && (threadIdx.x == 0 || pred(p));
        if (threadIdx.x == 0) *s_tmp = 0;
        __syncthreads();
        if (ok && threadIdx.x) atomicMax(s_tmp, threadIdx.x);
        __syncthreads();
        const uint32_t t = *s_tmp;
        __syncthreads();
        lo = lo + t * step;
        hi = min(lo + step, hi);
    }
    return lo;
}

// Inclusive prefix maximum of a[0 .. count) in LDS, count <= PER * blockDim.x, blockDim.x
// a multiple of 64 and at most 1024.  s_wave holds blockDim.x / 64 entries.
template <int PER = 4>
__device__ __forceinline__ void block_prefix_max_u16(uint16_t* a, uint32_t count, uint32_t* s_wave) {
    const uint32_t t = threadIdx.x, lane = t & 63, wid = t >> 6, nw = blockDim.x >> 6;
    uint32_t v[PER], m = 0;
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const uint32_t i = PER * t + q;
        v[q] = i < count ? a[i] : 0u;
        m = max(m, v[q]);
        v[q] = m;
    }
    uint32_t x = m;  // inclusive scan of thread maxima across the wave
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= (uint32_t)d) x = max(x, y);
    }
    if (lane == 63) s_wave[wid] = x;
    __syncthreads();
    uint32_t before = __shfl_up(x, 1, 64);
    if (lane == 0) before = 0;
    for (uint32_t w = 0; w < wid; w++) before = max(before, s_wave[w]);
    (void)nw;
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const uint32_t i = PER * t + q;
        if (i < count) a[i] = (uint16_t)max(v[q], before);
    }
    __syncthreads();
}

// ------------------------------------------------------------- edge push
// Decode an edge word (see Pack): the neighbour, and the weight from the word or from w.
__device__ __forceinline__ uint32_t pk_v(uint32_t c, const Pack& pk) { return c & pk.mask; }
__device__ __forceinline__ uint32_t pk_w(uint32_t c, uint32_t wraw, const Pack& pk) {
    return pk.shift < 32 ? (c >> pk.shift) + pk.wmin : wraw;
}
// A weight kept apart from the neighbour words: a uint32, or one byte holding w - wmin.
__device__ __forceinline__ uint32_t load_w(const uint32_t* __restrict__ w, uint64_t e, const Pack& pk) {
    return pk.wbytes == 1 ? (uint32_t)((const uint8_t*)w)[e] + pk.wmin : w[e];
}

constexpr int EDGE_THREADS = 256;
constexpr int EDGE_IPB = 1 << EDGE_TILE_SHIFT;  // edge items per workgroup pass
constexpr int EDGE_PER = EDGE_IPB / EDGE_THREADS;

// A pass covers the items of one tile (EDGE_IPB items, aligned) that lie in [item_lo,
// item_hi).  The list entries it meets come from the tile table that k_build_lists wrote
// (tile[t] = the entry holding item t * EDGE_IPB), so a pass waits for one load instead of two
// searches of the list; a compaction chunk, which may start inside an entry, searches.
template <class Op, bool COMPACTED>
__global__ __launch_bounds__(EDGE_THREADS) void k_push_edges(const uint32_t* __restrict__ list,
                                                             const uint64_t* __restrict__ wpre,
                                                             const uint32_t* __restrict__ tile, uint32_t ja,
                                                             uint32_t jb, uint64_t item_lo, uint64_t item_hi,
                                                             const uint64_t* __restrict__ off,
                                                             const uint32_t* __restrict__ col,
                                                             const uint32_t* __restrict__ w, uint64_t shift,
                                                             Op op, Pack pk) {
    __shared__ uint64_t s_at[EDGE_IPB];     // staged vertex: edge index of item x is s_at + x
    __shared__ uint32_t s_val[EDGE_IPB];
    __shared__ uint16_t s_owner[EDGE_IPB];  // item -> staged vertex
    __shared__ uint32_t s_tmp, s_wave[EDGE_THREADS / 64];
    for (uint64_t t = (item_lo >> EDGE_TILE_SHIFT) + blockIdx.x;; t += gridDim.x) {
        const uint64_t i0 = max(t << EDGE_TILE_SHIFT, item_lo);
        if (i0 >= item_hi) break;
        const uint64_t i1 = min((t + 1) << EDGE_TILE_SHIFT, item_hi);
        // list entries whose items meet [i0, i1): every one has at least one item there,
        // so there are at most EDGE_IPB of them
        uint32_t j0, j1;
        if constexpr (COMPACTED) {
            j0 = block_search_last(ja, jb, [&](uint32_t j) { return wpre[j] <= i0; }, &s_tmp);
            j1 = block_search_last(j0, jb, [&](uint32_t j) { return wpre[j] < i1; }, &s_tmp);
        } else {
            j0 = i0 == item_lo ? ja : tile[t];
            j1 = jb - 1;
            if (i1 < item_hi) {
                j1 = tile[t + 1];
                if (wpre[j1] == i1) j1--;
            }
        }
        const uint32_t nv = j1 - j0 + 1;
        const uint32_t cnt = (uint32_t)(i1 - i0);
        for (uint32_t q = threadIdx.x; q < cnt; q += EDGE_THREADS) s_owner[q] = 0;
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < nv; k += EDGE_THREADS) {
            const uint32_t v = list[j0 + k];
            const uint64_t pre = wpre[j0 + k];
            s_at[k] = (COMPACTED ? 0 : off[v] - pre) - shift;
            s_val[k] = op.src(v);
            if (k) s_owner[pre - i0] = (uint16_t)k;  // first item of every later vertex
        }
        __syncthreads();
        block_prefix_max_u16<EDGE_PER>(s_owner, cnt, s_wave);
        uint32_t val[EDGE_PER], v[EDGE_PER], wt[EDGE_PER];
        bool ok[EDGE_PER];
#pragma unroll
        for (int r = 0; r < EDGE_PER; r++) {
            const uint32_t q = r * EDGE_THREADS + threadIdx.x;
            ok[r] = q < cnt;
            val[r] = v[r] = wt[r] = 0;
            if (ok[r]) {
                const uint32_t k = s_owner[q];
                const uint64_t e = s_at[k] + (i0 + q);
                v[r] = col[e];
                if (Op::weighted && pk.shift == 32) wt[r] = load_w(w, e, pk);
                val[r] = s_val[k];
            }
        }
#pragma unroll
        for (int r = 0; r < EDGE_PER; r++) {
            if (Op::weighted) wt[r] = pk_w(v[r], wt[r], pk);
            v[r] = pk_v(v[r], pk);
        }
        push_batch<EDGE_PER>(op, ok, val, v, wt);
        __syncthreads();
    }
}

// ------------------------------------------------------------- line push
constexpr int LINE_THREADS = 256;
constexpr int LINE_HALVES = LINE_THREADS / 32;  // half waves per workgroup
constexpr int LINE_UNROLL = 8;                  // lines per half wave per pass
constexpr int LINE_IPB = LINE_HALVES * LINE_UNROLL;
static_assert(LINE_IPB == 1 << LINE_TILE_SHIFT, "the tile table's lines per pass");

// A pass waits for its lines behind all that are queued on the link (up to 0.2 ms), while the
// values that its vertices push may have improved.  Operators in steps, whose states only improve,
// read them once the lines are there: components of 2^20 uniform vertices, a quarter resident, zero-copy
// 3.7 -> 2.9 ms (values of the start of the pass made the third iteration push 12M edges again, 1.7M
// so), 3M vertices 9.5 -> 9.4; nothing else became slower.  (The streaming filter's chunks are one
// per workgroup at a time either way; there it gained nothing.)
template <class Op>
__global__ __launch_bounds__(LINE_THREADS) void k_push_lines(const uint32_t* __restrict__ list,
                                                             const uint64_t* __restrict__ wpre,
                                                             const uint32_t* __restrict__ tile, uint32_t ja,
                                                             uint32_t jb, uint64_t item_lo, uint64_t item_hi,
                                                             const uint64_t* __restrict__ off,
                                                             const uint32_t* __restrict__ col,
                                                             const uint32_t* __restrict__ w, Op op,
                                                             unsigned long long* __restrict__ distinct, Pack pk) {
    __shared__ uint64_t s_pre[LINE_IPB];
    __shared__ uint64_t s_s[LINE_IPB];
    __shared__ uint64_t s_e[LINE_IPB];
    __shared__ uint32_t s_val[LINE_IPB];  // the pushed value; operators in steps: the vertex
    __shared__ uint64_t s_prev_end;  // end offset of the list entry before the staged ones
    __shared__ uint32_t s_cnt;
    uint32_t my_lines = 0;  // distinct lines of the items this half wave loaded
    const uint32_t half = threadIdx.x >> 5, lane = threadIdx.x & 31;
    for (uint64_t t = (item_lo >> LINE_TILE_SHIFT) + blockIdx.x;; t += gridDim.x) {
        const uint64_t i0 = max(t << LINE_TILE_SHIFT, item_lo);
        if (i0 >= item_hi) break;
        const uint64_t i1 = min((t + 1) << LINE_TILE_SHIFT, item_hi);
        // the entries met, from the tile table as in k_push_edges
        const uint32_t j0 = i0 == item_lo ? ja : tile[t];
        uint32_t j1 = jb - 1;
        if (i1 < item_hi) {
            j1 = tile[t + 1];
            if (wpre[j1] == i1) j1--;
        }
        const uint32_t nv = j1 - j0 + 1;
        for (uint32_t k = threadIdx.x; k < nv; k += LINE_THREADS) {
            const uint32_t v = list[j0 + k];
            s_pre[k] = wpre[j0 + k];
            s_s[k] = off[v];
            s_e[k] = off[v + 1];
            s_val[k] = Op::steps ? v : op.src(v);
        }
        if (distinct && threadIdx.x == 0) s_prev_end = j0 > ja ? off[list[j0 - 1] + 1] : UINT64_MAX;
        __syncthreads();
        uint32_t cv[LINE_UNROLL], wv[LINE_UNROLL], kk[LINE_UNROLL];
        bool ok[LINE_UNROLL];
#pragma unroll
        for (int r = 0; r < LINE_UNROLL; r++) {
            const uint64_t i = i0 + half + (uint64_t)LINE_HALVES * r;
            ok[r] = false;
            kk[r] = 0;
            cv[r] = 0;
            wv[r] = 0;
            if (i < i1) {
                uint32_t lo = 0, hi = nv;
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (s_pre[mid] <= i)
                        lo = mid;
                    else
                        hi = mid;
                }
                const uint64_t s = s_s[lo];
                const uint64_t e = ((s >> ZC_LINE_SHIFT) << ZC_LINE_SHIFT) + ((i - s_pre[lo]) << ZC_LINE_SHIFT) + lane;
                if (distinct && lane == 0) {
                    // the first line of a vertex repeats when the previous active vertex
                    // (list order is CSR order) ends in it: count each line once
                    const uint64_t pe = lo ? s_e[lo - 1] : s_prev_end;
                    const bool dup = i == s_pre[lo] && pe != UINT64_MAX && pe > 0 &&
                                     ((pe - 1) >> ZC_LINE_SHIFT) == (s >> ZC_LINE_SHIFT);
                    my_lines += dup ? 0u : 1u;
                }
                if (e >= s && e < s_e[lo]) {
                    ok[r] = true;
                    kk[r] = lo;
                    cv[r] = col[e];
                    if (Op::weighted && pk.shift == 32) wv[r] = load_w(w, e, pk);
                }
            }
        }
        if constexpr (Op::steps) {  // the loads below stay behind the lines' arrival
#pragma unroll
            for (int r = 0; r < LINE_UNROLL; r++) asm volatile("" : "+v"(cv[r]), "+v"(wv[r]) : : "memory");
        }
#pragma unroll
        for (int r = 0; r < LINE_UNROLL; r++) {
            kk[r] = s_val[kk[r]];
            if constexpr (Op::steps) kk[r] = ok[r] ? op.src(kk[r]) : 0u;
            if (Op::weighted) wv[r] = pk_w(cv[r], wv[r], pk);
            cv[r] = pk_v(cv[r], pk);
        }
        push_batch<LINE_UNROLL>(op, ok, kk, cv, wv);
        __syncthreads();
    }
    if (distinct) {
        if (threadIdx.x == 0) s_cnt = 0;
        __syncthreads();
        if (lane == 0 && my_lines) atomicAdd(&s_cnt, my_lines);
        __syncthreads();
        if (threadIdx.x == 0 && s_cnt) atomicAdd(distinct, (unsigned long long)s_cnt);
    }
}

// ------------------------------------------------------------- init etc.
__global__ void k_init(AlgoState s, uint64_t n, uint32_t source, float x0, float* __restrict__ x,
                       uint32_t* __restrict__ cur, uint32_t nwords) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += stride) {
        if (s.algo == ALGO_PR)
            x[v] = s.inv_n ? s.inv_n[v] : x0;
        else if (s.algo == ALGO_CC)
            s.val[v] = (uint32_t)v;
        else
            s.val[v] = v == source ? 0u : UNREACHED;
    }
    for (uint64_t wi = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; wi < nwords; wi += stride) {
        uint32_t c;
        if (s.algo == ALGO_BFS || s.algo == ALGO_SSSP || s.algo == ALGO_BFS_RELAX) {
            c = (wi == (source >> 5)) ? (1u << (source & 31)) : 0u;
        } else {
            const uint64_t lo = wi << 5;
            c = lo + 32 <= n ? ~0u : (lo < n ? (1u << (uint32_t)(n - lo)) - 1u : 0u);
        }
        cur[wi] = c;
        if (s.next) s.next[wi] = 0;
        if (s.visited) s.visited[wi] = s.algo == ALGO_BFS ? c : 0u;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && s.overflow) *s.overflow = 0;
}

// Batched runs: value rows to UNREACHED except each lane's own source, lane masks with
// each lane's bit at its source, the union frontier holding every source.
__global__ void k_init_lanes(AlgoState s, LaneSources src, uint32_t* __restrict__ cur, uint32_t nwords) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t cells = s.n << s.lshift;
    const uint32_t lmask = (1u << s.lshift) - 1;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < cells; i += stride) {
        const uint32_t v = (uint32_t)(i >> s.lshift), l = (uint32_t)i & lmask;
        const bool at_src = l < src.count && src.src[l] == v;
        if (s.algo == ALGO_MPPR) {
            s.lx[i] = at_src ? 1.0f : 0.0f;
            s.lacc[i] = 0.0;
        } else {
            s.lval[i] = at_src ? 0u : UNREACHED;
        }
    }
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < s.n; v += stride) {
        uint64_t m = 0;
        for (uint32_t l = 0; l < src.count; l++)
            if (src.src[l] == v) m |= 1ull << l;
        ((uint64_t*)s.mcur)[v] = m;
        s.mnext[v] = 0;
        if (s.mvisited) s.mvisited[v] = m;
    }
    for (uint64_t wi = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; wi < nwords; wi += stride) {
        uint32_t c = 0;
        for (uint32_t l = 0; l < src.count; l++)
            if ((src.src[l] >> 5) == wi) c |= 1u << (src.src[l] & 31);
        cur[wi] = c;
        s.next[wi] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && s.overflow) s.overflow[0] = s.overflow[1] = 0;
}

// The end of a wide iteration of a batched BFS, from the lanes each vertex gained (mnext): they
// are reached, at the level, and the vertices that gained any are the next frontier.  One wave
// per window of 64 vertices; a row of levels is stored by one thread per lane.
__global__ __launch_bounds__(256) void k_settle_lanes(AlgoState s, uint32_t nwords) {
    const uint32_t lane = threadIdx.x & 63, ln = lane & ((1u << s.lshift) - 1), slot = lane >> s.lshift;
    const uint32_t per = 64u >> s.lshift;  // rows per store
    const uint64_t some = per == 64 ? ~0ull : (1ull << per) - 1;
    const uint64_t windows = (s.n + 63) >> 6, waves = (uint64_t)gridDim.x * 4;
    for (uint64_t q = blockIdx.x * 4ull + (threadIdx.x >> 6); q < windows; q += waves) {
        const uint64_t v = (q << 6) + lane;
        const uint64_t x = v < s.n ? s.mnext[v] : 0ull;
        const uint64_t any = __ballot(x != 0);
        if (lane < 2 && 2 * q + lane < nwords) s.next[2 * q + lane] = (uint32_t)(any >> (32 * lane));
        if (x) s.mvisited[v] |= x;
        for (uint32_t j = 0; j < 64; j += per) {
            if (!((any >> j) & some)) continue;  // uniform
            const uint64_t y = __shfl(x, (int)(j + slot), 64);
            if ((y >> ln) & 1) s.lval[(((q << 6) + j + slot) << s.lshift) + ln] = s.level_next;
        }
    }
}

// Lane extraction through LDS: a workgroup loads the rows of V vertices with coalesced
// reads (row pitch padded by one word against bank conflicts), then writes each requested
// lane as a contiguous run of V values.  Into host memory the link bounds it: 64 lanes of
// 2^20 vertices in 4.81 ms, 55.8 GB/s, where extracting eight lanes at a time into device
// rows and copying those took 5.3 ms.  Rows of an odd length start in the middle of a
// write: runs of 64 values then reach 49.2 GB/s, of 256 values 52.6; below EX_WIDE vertices
// runs of 64 give the chip more workgroups (1,000 vertices: 13 us, 24 us in runs of 256).
// Into device rows the reads bound it, and runs of 64, whose 16 KB of LDS leave eight workgroups
// to a CU, read 64 lanes of 2^21 vertices in 0.17 ms where runs of 256 took 0.49.
constexpr uint64_t EX_WIDE = 1ull << 15;
template <uint32_t V>
__global__ __launch_bounds__(256) void k_extract_lanes(const uint32_t* __restrict__ vals, uint64_t n,
                                                       uint32_t lshift, LaneSet set, uint32_t nsel, bool sub_base,
                                                       const uint32_t* __restrict__ rank, LaneRows out) {
    extern __shared__ uint32_t ex_tile[];  // V rows of pitch words
    __shared__ uint8_t s_lane[MAX_LANES];
    __shared__ uint32_t s_base[MAX_LANES];
    __shared__ uint32_t* s_out[MAX_LANES];
    const uint32_t S = 1u << lshift, pitch = S + 1;
    if (threadIdx.x < MAX_LANES) {
        // k-th set lane of the mask, k = threadIdx.x
        uint64_t m = set.mask;
        for (uint32_t k = 0; k < threadIdx.x && m; k++) m &= m - 1;
        if (m) {
            const uint32_t l = __ffsll((unsigned long long)m) - 1;
            s_lane[threadIdx.x] = (uint8_t)l;
            s_base[threadIdx.x] = set.base[l];
            s_out[threadIdx.x] = out.row[threadIdx.x];
        }
    }
    for (uint64_t v0 = (uint64_t)blockIdx.x * V; v0 < n; v0 += (uint64_t)gridDim.x * V) {
        const uint32_t nv = (uint32_t)(n - v0 < V ? n - v0 : V);
        __syncthreads();
        const uint32_t cells = nv << lshift;
        for (uint32_t c = threadIdx.x; c < cells; c += blockDim.x) {
            const uint32_t i = c >> lshift;
            const uint64_t r = rank ? rank[v0 + i] : v0 + i;
            ex_tile[i * pitch + (c & (S - 1))] = vals[(r << lshift) + (c & (S - 1))];
        }
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < nsel * V; q += blockDim.x) {
            const uint32_t k = q / V, i = q % V;
            if (i >= nv) continue;
            uint32_t x = ex_tile[i * pitch + s_lane[k]];
            if (sub_base && x != UNREACHED) x -= s_base[k];
            s_out[k][v0 + i] = x;
        }
    }
}

__global__ __launch_bounds__(256) void k_loaded_frontier(uint32_t npart, const uint32_t* __restrict__ pv,
                                                         const uint8_t* __restrict__ mode, uint32_t mode_mask,
                                                         const uint32_t* __restrict__ next, uint32_t* __restrict__ cur2) {
    for (uint32_t p = blockIdx.x; p < npart; p += gridDim.x) {
        if (!((mode_mask >> mode[p]) & 1)) continue;  // uniform across the workgroup
        for (uint32_t v = pv[p] + threadIdx.x; v < pv[p + 1]; v += blockDim.x)
            if ((next[v >> 5] >> (v & 31)) & 1) atomicOr(cur2 + (v >> 5), 1u << (v & 31));
    }
}

__global__ __launch_bounds__(256) void k_dpr_fold(uint32_t npart, const uint32_t* __restrict__ pv, uint64_t n,
                                                  float* __restrict__ acc, uint32_t copies,
                                                  float* __restrict__ delta, double* __restrict__ psum) {
    __shared__ double s_w[4];
    const uint64_t slots = acc_slots(n);
    for (uint32_t p = blockIdx.x; p < npart; p += gridDim.x) {
        double sum = 0.0;
        for (uint32_t v = pv[p] + threadIdx.x; v < pv[p + 1]; v += blockDim.x) {
            const uint32_t sl = acc_slot(v);
            float d = delta[v];
            for (uint32_t c = 0; c < copies; c++) {
                d += acc[c * slots + sl];
                acc[c * slots + sl] = 0.0f;
            }
            delta[v] = d;
            sum += (double)d;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0) psum[p] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_dpr_activate(uint32_t npart, const uint32_t* __restrict__ pv,
                                                      const uint64_t* __restrict__ off,
                                                      const uint8_t* __restrict__ sched, float* __restrict__ delta,
                                                      float* __restrict__ x, float* __restrict__ contrib,
                                                      uint32_t* __restrict__ cur, float damping) {
    for (uint32_t p = blockIdx.x; p < npart; p += gridDim.x) {
        if (!sched[p]) continue;  // uniform across the workgroup
        for (uint32_t v = pv[p] + threadIdx.x; v < pv[p + 1]; v += blockDim.x) {
            const float d = delta[v];
            if (!(d > 0.0f)) continue;
            x[v] += d;
            delta[v] = 0.0f;
            const uint64_t deg = off[v + 1] - off[v];
            if (deg) {
                contrib[v] = damping * d / (float)deg;
                atomicOr(cur + (v >> 5), 1u << (v & 31));
            }
        }
    }
}

__global__ void k_dpr_init(uint64_t n, float* __restrict__ delta, const float* __restrict__ inv_n, float restart,
                           float uniform) {
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += (uint64_t)gridDim.x * blockDim.x)
        delta[v] = inv_n ? restart * inv_n[v] : uniform;
}

__global__ void k_dpr_finish(uint64_t n, float* __restrict__ x, const float* __restrict__ delta) {
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += (uint64_t)gridDim.x * blockDim.x)
        x[v] += delta[v];
}

__global__ void k_gather_u32(const uint32_t* __restrict__ src, const uint32_t* __restrict__ rank, uint64_t n,
                             uint32_t* __restrict__ dst) {
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += (uint64_t)gridDim.x * blockDim.x)
        dst[v] = src[rank[v]];
}

// minold[label] = the smallest original id among the vertices holding that label.  Nearly
// every vertex of a graph with a giant component holds the same label, so one word would
// take an atomic per vertex: lanes holding the label of the wave's first lane fold their ids
// into one atomic, and no atomic is made when the slot already holds a smaller id (slots
// only decrease, so a stale read can only let an unneeded atomic through).
__global__ void k_cc_min_old(const uint32_t* __restrict__ lab, const uint32_t* __restrict__ order, uint64_t n,
                             uint32_t* minold) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n; base += stride) {  // uniform per block
        const uint64_t v = base + threadIdx.x;
        const bool ok = v < n;
        const uint32_t l = ok ? lab[v] : UNREACHED;
        const uint32_t o = ok ? order[v] : UNREACHED;
        const uint32_t l0 = __shfl(l, 0, 64);  // lane 0 holds the wave's smallest v
        const bool same = ok && l == l0;
        uint32_t m = same ? o : UNREACHED;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = min(m, (uint32_t)__shfl_xor(m, d, 64));
        if (__lane_id() == 0 && m != UNREACHED && m < minold[l0]) atomicMin(minold + l0, m);
        if (ok && !same && o < minold[l]) atomicMin(minold + l, o);
    }
}

__global__ void k_cc_canon(const uint32_t* __restrict__ lab, const uint32_t* __restrict__ minold,
                           const uint32_t* __restrict__ rank, uint64_t n, uint32_t* __restrict__ dst) {
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += (uint64_t)gridDim.x * blockDim.x)
        dst[v] = minold[lab[rank[v]]];
}

// ----------------------------------------- components of a resident graph
// The r-th edge of every vertex joined (par = a parent forest, at first every vertex its own).
__global__ __launch_bounds__(256) void k_cc_link(uint64_t n, const uint64_t* __restrict__ off,
                                                 const uint32_t* __restrict__ col, uint32_t vmask, uint32_t r,
                                                 uint32_t* par) {
    for (uint64_t v = blockIdx.x * 256ull + threadIdx.x; v < n; v += (uint64_t)gridDim.x * 256) {
        const uint64_t e = off[v] + r;
        if (e < off[v + 1]) link_trees(par, (uint32_t)v, col[e] & vmask);
    }
}

// Every vertex moved below its root.  Only roots' entries stay as they are, so a value read
// before or after another vertex's move is an ancestor either way.
__global__ __launch_bounds__(256) void k_cc_compress(uint64_t n, uint32_t* par) {
    for (uint64_t v = blockIdx.x * 256ull + threadIdx.x; v < n; v += (uint64_t)gridDim.x * 256) {
        const uint32_t p = par[v];
        uint32_t r = p;
        for (uint32_t q = par[r]; q != r; q = par[r]) r = q;
        if (r != p) par[v] = r;
    }
}

// The most frequent root among 4,096 sampled vertices (one workgroup; counted in an LDS table
// where colliding roots share a counter of whoever came first, so the answer may be off, which
// costs time only).
__global__ __launch_bounds__(1024) void k_cc_giant(uint64_t n, const uint32_t* __restrict__ par,
                                                   uint32_t* __restrict__ giant) {
    constexpr uint32_t T = 2048;
    __shared__ uint32_t s_key[T], s_cnt[T];
    __shared__ unsigned long long s_best;
    for (uint32_t q = threadIdx.x; q < T; q += 1024) {
        s_key[q] = UNREACHED;
        s_cnt[q] = 0;
    }
    if (threadIdx.x == 0) s_best = 0;
    __syncthreads();
    for (uint32_t k = 0; k < 4; k++) {
        const uint64_t i = k * 1024 + threadIdx.x;
        const uint32_t l = par[(i * 0x9E3779B97F4A7C15ull >> 11) % n];
        const uint32_t slot = (l * 0x9E3779B1u) >> 21;
        const uint32_t was = atomicCAS(&s_key[slot], UNREACHED, l);
        if (was == UNREACHED || was == l) atomicAdd(&s_cnt[slot], 1u);
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < T; q += 1024)
        if (s_cnt[q]) atomicMax(&s_best, (unsigned long long)s_cnt[q] << 32 | s_key[q]);
    __syncthreads();
    if (threadIdx.x == 0) *giant = (uint32_t)s_best;
}

// rest = the vertices outside the giant's tree with more than `done` edges (one wave per two
// words of the bitmap).
__global__ __launch_bounds__(256) void k_cc_rest(uint64_t n, const uint64_t* __restrict__ off, uint32_t done,
                                                 const uint32_t* __restrict__ par,
                                                 const uint32_t* __restrict__ giant, uint32_t* __restrict__ rest,
                                                 uint32_t nwords) {
    const uint32_t g = *giant;
    for (uint64_t v = blockIdx.x * 256ull + threadIdx.x; (v & ~63ull) < n; v += (uint64_t)gridDim.x * 256) {
        const uint64_t b = __ballot(v < n && par[v] != g && off[v + 1] - off[v] > done);
        const uint32_t w = (uint32_t)(v >> 6) * 2;
        if ((v & 63) == 0) {
            rest[w] = (uint32_t)b;
            if (w + 1 < nwords) rest[w + 1] = (uint32_t)(b >> 32);
        }
    }
}

// Smallest distance among the far vertices: one word of the far bitmap per thread, a wave
// minimum, one atomic per wave that holds any.
__global__ void k_far_min(const uint32_t* __restrict__ far, const uint32_t* __restrict__ dist, uint32_t nwords,
                          uint32_t* out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < nwords; base += stride) {  // uniform per block
        const uint64_t wd = base + threadIdx.x;
        uint32_t bits = wd < nwords ? far[wd] : 0u, m = UNREACHED;
        while (bits) {
            const uint32_t b = __ffs(bits) - 1;
            bits &= bits - 1;
            m = min(m, dist[wd * 32 + b]);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = min(m, (uint32_t)__shfl_xor(m, d, 64));
        if (__lane_id() == 0 && m != UNREACHED) atomicMin(out, m);
    }
}

// Far vertices with distance below `bound` leave the far set and join the frontier; each
// thread owns one word of both bitmaps.
__global__ void k_far_move(uint32_t* __restrict__ far, const uint32_t* __restrict__ dist, uint32_t* __restrict__ cur,
                           uint32_t nwords, uint32_t bound) {
    for (uint64_t wd = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; wd < nwords;
         wd += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t f = far[wd];
        if (!f) continue;
        uint32_t bits = f, moved = 0;
        while (bits) {
            const uint32_t b = __ffs(bits) - 1;
            bits &= bits - 1;
            if (dist[wd * 32 + b] < bound) moved |= 1u << b;
        }
        if (moved) {
            far[wd] = f & ~moved;
            cur[wd] |= moved;
        }
    }
}

// SSSP overflow, decided after convergence.  A relaxation whose candidate reaches 2^32-1 is
// skipped and only raises a lane's flag; whether that lane's shortest distances really
// overflow is decided here.  After convergence every vertex whose shortest distance fits
// below 2^32-1 holds it, so a lane overflows exactly when some edge leads from a vertex it
// reached to one it did not.  One wave per vertex u (grid-stride): the lanes of `mask`
// that reached u read u's out-edges from the mapped host array `col` and check their
// targets; lanes that find an unreached target are ORed into *out.  dist: n rows of
// 2^lshift lanes (lshift 0: one distance per vertex).
__global__ __launch_bounds__(256) void k_sssp_ovf_check(const uint64_t* __restrict__ off,
                                                        const uint32_t* __restrict__ col, Pack pk,
                                                        const uint32_t* __restrict__ dist, uint32_t lshift,
                                                        uint64_t mask, uint64_t n, unsigned long long* out) {
    const uint32_t lane = __lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / 64);
    uint64_t found = 0;
    for (uint64_t u = blockIdx.x * (uint64_t)(blockDim.x / 64) + threadIdx.x / 64; u < n; u += waves) {
        const bool mine = lane < (1u << lshift) && ((mask >> lane) & 1) && dist[(u << lshift) + lane] != UNREACHED;
        const uint64_t reached = __ballot(mine);
        if (!reached) continue;
        const uint64_t e1 = off[u + 1];
        for (uint64_t e = off[u] + lane; e < e1; e += 64) {
            const uint32_t* dv = dist + ((uint64_t)pk_v(col[e], pk) << lshift);
            for (uint64_t r = reached; r; r &= r - 1) {
                const uint32_t l = __ffsll((unsigned long long)r) - 1;
                if (dv[l] == UNREACHED) found |= 1ull << l;
            }
        }
    }
    if (found) atomicOr(out, (unsigned long long)found);
}

__global__ void k_admit_lanes(AlgoState s, LaneSet set, uint32_t* __restrict__ cur) {
    const uint32_t l = threadIdx.x;
    if (l >= MAX_LANES || !((set.mask >> l) & 1)) return;
    const uint32_t v = set.src[l];
    const uint64_t cell = ((uint64_t)v << s.lshift) + l;
    if (s.algo == ALGO_MPPR)
        s.lx[cell] = 1.0f;
    else
        s.lval[cell] = s.algo == ALGO_MBFS ? set.base[l] : 0u;
    atomicOr((unsigned long long*)(s.mcur + v), 1ull << l);
    if (s.mvisited) atomicOr((unsigned long long*)(s.mvisited + v), 1ull << l);
    atomicOr(cur + (v >> 5), 1u << (v & 31));
}

__global__ void k_reset_lanes(AlgoState s, uint64_t mask) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t lmask = (1u << s.lshift) - 1;
    const uint64_t cells = s.n << s.lshift;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < cells; i += stride) {
        if (!((mask >> ((uint32_t)i & lmask)) & 1)) continue;
        if (s.algo == ALGO_MPPR) {
            s.lx[i] = 0.0f;
            s.lacc[i] = 0.0;
        } else {
            s.lval[i] = UNREACHED;
        }
    }
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < s.n; v += stride) {
        ((uint64_t*)s.mcur)[v] &= ~mask;
        s.mnext[v] &= ~mask;
        if (s.mvisited) s.mvisited[v] &= ~mask;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && s.overflow) {
        s.overflow[0] &= ~(uint32_t)mask;
        s.overflow[1] &= ~(uint32_t)(mask >> 32);
    }
}

// The steps of personalized PageRank over its values, at the (vertex, lane) cells whose bits
// are set in cell_mask.  A wave takes windows of `rows` vertices (a power of two, at most 64, whole
// accesses): it loads their masks, passes over the rows without a set bit (of few active vertices
// almost all) and takes the others 64 cells at a time, contiguous, PPR_ROWS of these accesses in
// flight.  Bound by the rows' bytes where the frontier is dense, by the masks' where it is sparse:
// whole calls, one thread per cell and this, 12 lanes of 2^25 uniform vertices with 2 edges each 39.8
// -> 34.6 ms (a thread per vertex 36.1, but 0.54 ms a pass of 1M dense rows of 64), 64 lanes of R-MAT
// 20 18.7 -> 18.2.
constexpr int PPR_ROWS = 4;
template <class Op>
__device__ __forceinline__ void ppr_cells(const AlgoState& s, uint32_t rows, const Op& op) {
    const uint32_t lane = threadIdx.x & 63, ln = lane & ((1u << s.lshift) - 1), slot = lane >> s.lshift;
    const uint32_t per = 64u >> s.lshift;  // rows per access
    const uint64_t some = per == 64 ? ~0ull : (1ull << per) - 1;
    const uint64_t step = (uint64_t)gridDim.x * 4 * rows;
    for (uint64_t v0 = (blockIdx.x * 4ull + (threadIdx.x >> 6)) * rows; v0 < s.n; v0 += step) {
        const uint64_t m = lane < rows && v0 + lane < s.n ? op.cell_mask(v0 + lane) : 0ull;
        uint64_t left = __ballot(m != 0);  // vertices whose rows are to come
        while (left) {                     // uniform
            uint64_t v[PPR_ROWS];
            bool on[PPR_ROWS];
            typename Op::Reg x[PPR_ROWS];
#pragma unroll
            for (int r = 0; r < PPR_ROWS; r++) {
                const uint32_t j = left ? ((uint32_t)__ffsll((unsigned long long)left) - 1) & ~(per - 1) : 0u;
                const uint64_t y = __shfl(m, (int)(j + slot), 64);
                on[r] = left && ((y >> ln) & 1);
                v[r] = v0 + j + slot;
                if (on[r]) x[r] = op.load(v[r], (v[r] << s.lshift) + ln);
                left &= ~(some << j);
            }
#pragma unroll
            for (int r = 0; r < PPR_ROWS; r++)
                if (on[r]) op.store(v[r], (v[r] << s.lshift) + ln, ln, x[r]);
        }
    }
}

// x of each active cell scaled to x / D_o.
struct PprPrepare {
    struct Reg {
        float x;
        uint64_t d;
    };
    const AlgoState& s;
    const uint64_t* __restrict__ off;
    __device__ __forceinline__ uint64_t cell_mask(uint64_t v) const { return s.mcur[v]; }
    __device__ __forceinline__ Reg load(uint64_t v, uint64_t i) const { return Reg{s.lx[i], off[v + 1] - off[v]}; }
    __device__ __forceinline__ void store(uint64_t, uint64_t i, uint32_t, const Reg& r) const {
        if (r.d) s.lx[i] = r.x / (float)r.d;
    }
};
__global__ __launch_bounds__(256) void k_ppr_prepare(AlgoState s, uint32_t rows, const uint64_t* __restrict__ off) {
    ppr_cells(s, rows, PprPrepare{s, off});
}

struct PprApply {
    typedef double Reg;
    const AlgoState& s;
    float damping;
    __device__ __forceinline__ uint64_t cell_mask(uint64_t v) const { return s.mcur[v] | s.mnext[v]; }
    __device__ __forceinline__ Reg load(uint64_t, uint64_t i) const { return s.lacc[i]; }
    __device__ __forceinline__ void store(uint64_t, uint64_t i, uint32_t, Reg a) const {
        s.lx[i] = (float)((double)damping * a);
        s.lacc[i] = 0.0;
    }
};
__global__ __launch_bounds__(256) void k_ppr_apply(AlgoState s, uint32_t rows, float damping) {
    ppr_cells(s, rows, PprApply{s, damping});
}

// k_ppr_apply and the next step's k_ppr_prepare in one pass, for lanes that all step on: the
// values after the restart of each lane's source (active in every step, so among the cells),
// scaled by 1 / D_o where there are out-edges.
struct PprApplyNext : PprApply {
    struct Reg {
        double a;
        uint64_t d;
    };
    const uint64_t* __restrict__ off;
    const uint32_t* src;  // per lane (LDS)
    float restart;
    __device__ __forceinline__ Reg load(uint64_t v, uint64_t i) const { return Reg{s.lacc[i], off[v + 1] - off[v]}; }
    __device__ __forceinline__ void store(uint64_t v, uint64_t i, uint32_t l, const Reg& r) const {
        float x = (float)((double)damping * r.a);
        if (src[l] == v) x += restart;
        s.lx[i] = r.d ? x / (float)r.d : x;
        s.lacc[i] = 0.0;
    }
};
__global__ __launch_bounds__(256) void k_ppr_apply_next(AlgoState s, uint32_t rows, const uint64_t* __restrict__ off,
                                                        LaneSet set, float damping, float restart) {
    __shared__ uint32_t s_src[MAX_LANES];
    if (threadIdx.x < MAX_LANES) s_src[threadIdx.x] = (set.mask >> threadIdx.x) & 1 ? set.src[threadIdx.x] : UNREACHED;
    __syncthreads();
    ppr_cells(s, rows, PprApplyNext{{s, damping}, off, s_src, restart});
}

__global__ void k_ppr_restart(AlgoState s, LaneSet set, float restart) {
    const uint32_t l = threadIdx.x;
    if (l >= MAX_LANES || !((set.mask >> l) & 1)) return;
    const uint32_t v = set.src[l];
    if (restart != 0.0f) s.lx[((uint64_t)v << s.lshift) + l] += restart;
    atomicOr((unsigned long long*)(s.mnext + v), 1ull << l);
    atomicOr(s.next + (v >> 5), 1u << (v & 31));
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint64_t count, uint32_t value) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

__global__ __launch_bounds__(256) void k_fill2_u32(uint32_t* __restrict__ p, uint64_t np, uint32_t* __restrict__ q,
                                                   uint64_t nq, uint32_t value) {
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < np + nq; i += (uint64_t)gridDim.x * 256) {
        if (i < np)
            p[i] = value;
        else
            q[i - np] = value;
    }
}

__global__ void k_pr_prepare(uint64_t n, const uint64_t* __restrict__ off, const float* __restrict__ x,
                             float* __restrict__ contrib, float* __restrict__ acc, uint32_t copies) {
    const uint64_t slots = acc_slots(n);
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < slots;
         v += (uint64_t)gridDim.x * blockDim.x) {
        if (v < n) {
            const uint64_t d = off[v + 1] - off[v];
            contrib[v] = d ? x[v] / (float)d : 0.0f;
        }
        for (uint32_t c = 0; c < copies; c++) acc[c * slots + v] = 0.0f;
    }
}

__global__ void k_pr_apply(uint64_t n, float* __restrict__ x, const float* __restrict__ acc, uint32_t copies,
                           float base, float damping, const float* __restrict__ inv_n, float restart) {
    const uint64_t slots = acc_slots(n);
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n;
         v += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t s = acc_slot((uint32_t)v);
        float sum = 0.0f;
        for (uint32_t c = 0; c < copies; c++) sum += acc[c * slots + s];
        x[v] = (inv_n ? restart * inv_n[v] : base) + damping * sum;
    }
}

// ---------------------------------------------------- propagation blocking
constexpr int PB_THREADS = 256;
constexpr int PB_PLAN_THREADS = 1024;
constexpr uint32_t PB_TILE = 2048;   // pairs per scatter tile, 8 per thread
constexpr uint32_t PB_LOCAL = PB_LOCAL_BINS;

// Exclusive sum of one value per thread over the workgroup (a multiple of 64 threads);
// *total = the sum of all.  s_w holds blockDim.x / 64 + 1 entries.  Every thread calls it.
__device__ __forceinline__ uint32_t block_excl_sum(uint32_t x, uint32_t* s_w, uint32_t* total) {
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t inc = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, 64);
        if (lane >= (uint32_t)d) inc += y;
    }
    if (lane == 63) s_w[wid] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t a = 0;
        for (uint32_t w = 0; w < nw; w++) {
            const uint32_t t = s_w[w];
            s_w[w] = a;
            a += t;
        }
        s_w[nw] = a;
    }
    __syncthreads();
    const uint32_t r = s_w[wid] + inc - x;
    *total = s_w[nw];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(PB_THREADS) void k_pb_hist(const uint32_t* __restrict__ pv, uint32_t vmask, uint64_t cnt,
                                                        uint32_t fshift, uint32_t nfine, uint32_t* __restrict__ hist,
                                                        uint32_t* __restrict__ err) {
    __shared__ uint32_t s_h[PB_MAX_FINE];
    for (uint32_t f = threadIdx.x; f < nfine; f += PB_THREADS) s_h[f] = 0;
    __syncthreads();
    bool bad = false;
    for (uint64_t i = blockIdx.x * (uint64_t)PB_THREADS + threadIdx.x; i < cnt;
         i += (uint64_t)gridDim.x * PB_THREADS) {
        const uint32_t f = (pv[i] & vmask) >> fshift;
        if (f < nfine)
            atomicAdd(&s_h[f], 1u);
        else
            bad = true;
    }
    if (bad) atomicOr(err, 1u);
    __syncthreads();
    for (uint32_t f = threadIdx.x; f < nfine; f += PB_THREADS)
        if (s_h[f]) atomicAdd(hist + f, s_h[f]);
}

// One workgroup: bin starts and the accumulation segments of every non-empty bin.
__global__ __launch_bounds__(PB_PLAN_THREADS) void k_pb_plan(const uint32_t* __restrict__ hist, uint32_t nfine,
                                                             uint32_t seg, uint32_t* __restrict__ foff,
                                                             uint32_t* __restrict__ segs,
                                                             uint32_t* __restrict__ nsegs) {
    constexpr uint32_t PER = PB_MAX_FINE / PB_PLAN_THREADS;
    __shared__ uint32_t s_w[PB_PLAN_THREADS / 64 + 1];
    const uint32_t f0 = threadIdx.x * PER;
    uint32_t c[PER], sum = 0, ns = 0;
#pragma unroll
    for (uint32_t q = 0; q < PER; q++) {
        c[q] = f0 + q < nfine ? hist[f0 + q] : 0u;
        sum += c[q];
        ns += (c[q] + seg - 1) / seg;
    }
    uint32_t total, stotal;
    uint32_t base = block_excl_sum(sum, s_w, &total);
    uint32_t sb = block_excl_sum(ns, s_w, &stotal);
    for (uint32_t q = 0; q < PER; q++) {
        const uint32_t f = f0 + q;
        if (f >= nfine) break;
        foff[f] = base;
        base += c[q];
        for (uint32_t j = 0; (uint64_t)j * seg < c[q]; j++, sb++) {
            segs[2 * sb] = f;
            segs[2 * sb + 1] = j;
        }
    }
    if (threadIdx.x == 0) {
        foff[nfine] = total;
        *nsegs = stotal;
    }
}

// A tile whose keys span fewer than PB_LOCAL bins is counting-sorted in LDS: one cursor
// reservation per bin present, then the tile's pairs leave bin by bin in runs.  A tile
// spanning more (a stretch of nearly empty bins) reserves a position per pair.
__global__ __launch_bounds__(PB_THREADS) void k_pb_scatter(const uint32_t* __restrict__ in_v,
                                                           const float* __restrict__ in_c, uint64_t cnt,
                                                           uint32_t kshift, uint32_t stride, uint32_t nfine,
                                                           const uint32_t* __restrict__ foff,
                                                           uint32_t* __restrict__ cursor, uint32_t* __restrict__ out_v,
                                                           float* __restrict__ out_c, uint32_t* __restrict__ err) {
    constexpr uint32_t PER = PB_TILE / PB_THREADS;
    constexpr uint32_t LPER = PB_LOCAL / PB_THREADS;
    __shared__ uint32_t s_v[PB_TILE];
    __shared__ float s_c[PB_TILE];
    __shared__ uint16_t s_k[PB_TILE];
    __shared__ uint32_t s_cnt[PB_LOCAL], s_ofs[PB_LOCAL], s_g[PB_LOCAL], s_end[PB_LOCAL];
    __shared__ uint32_t s_kmin, s_kmax, s_w[PB_THREADS / 64 + 1];
    const uint32_t nkeys = (nfine + stride - 1) / stride;
    const uint32_t lane = threadIdx.x & 63;
    bool bad = false;
    // each workgroup walks tiles blockIdx.x, + gridDim.x, ...; the next tile's loads are
    // issued before the current tile is sorted
    const uint64_t step = (uint64_t)gridDim.x * PB_TILE;
    uint32_t v[PER], key[PER], rank[PER];
    float c[PER];
    {
        const uint64_t t0 = blockIdx.x * (uint64_t)PB_TILE;
        const uint32_t tc = (uint32_t)min((uint64_t)PB_TILE, cnt - t0);
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            const uint32_t i = r * PB_THREADS + threadIdx.x;
            v[r] = i < tc ? in_v[t0 + i] : 0u;
            c[r] = i < tc ? in_c[t0 + i] : 0.0f;
        }
    }
    for (uint64_t t0 = blockIdx.x * (uint64_t)PB_TILE; t0 < cnt; t0 += step) {
        const uint32_t tc = (uint32_t)min((uint64_t)PB_TILE, cnt - t0);
        uint32_t nv[PER];
        float nc[PER];
        {
            const uint64_t t1 = t0 + step;
            const uint32_t tc1 = t1 < cnt ? (uint32_t)min((uint64_t)PB_TILE, cnt - t1) : 0u;
#pragma unroll
            for (uint32_t r = 0; r < PER; r++) {
                const uint32_t i = r * PB_THREADS + threadIdx.x;
                nv[r] = i < tc1 ? in_v[t1 + i] : 0u;
                nc[r] = i < tc1 ? in_c[t1 + i] : 0.0f;
            }
        }
        uint32_t kmin = UINT32_MAX, kmax = 0;
        if (threadIdx.x == 0) {
            s_kmin = UINT32_MAX;
            s_kmax = 0;
        }
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            key[r] = 0;
            rank[r] = 0;
            if (r * PB_THREADS + threadIdx.x < tc) {
                key[r] = v[r] >> kshift;
                kmin = min(kmin, key[r]);
                kmax = max(kmax, key[r]);
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            kmin = min(kmin, (uint32_t)__shfl_xor(kmin, d, 64));
            kmax = max(kmax, (uint32_t)__shfl_xor(kmax, d, 64));
        }
        __syncthreads();
        if (lane == 0) {
            atomicMin(&s_kmin, kmin);
            atomicMax(&s_kmax, kmax);
        }
        __syncthreads();
        const uint32_t k0 = s_kmin, k1 = s_kmax;
        if (k1 < nkeys && k1 - k0 < PB_LOCAL) {  // uniform across the workgroup
#pragma unroll
            for (uint32_t q = 0; q < LPER; q++) s_cnt[LPER * threadIdx.x + q] = 0;
            __syncthreads();
#pragma unroll
            for (uint32_t r = 0; r < PER; r++)
                if (r * PB_THREADS + threadIdx.x < tc) rank[r] = atomicAdd(&s_cnt[key[r] - k0], 1u);
            __syncthreads();
            uint32_t loc[LPER], sum = 0, tot;
#pragma unroll
            for (uint32_t q = 0; q < LPER; q++) {
                loc[q] = s_cnt[LPER * threadIdx.x + q];
                sum += loc[q];
            }
            uint32_t base = block_excl_sum(sum, s_w, &tot);
#pragma unroll
            for (uint32_t q = 0; q < LPER; q++) {
                const uint32_t b = LPER * threadIdx.x + q;
                s_ofs[b] = base;
                base += loc[q];
                if (loc[q]) {
                    const uint32_t k = k0 + b;
                    s_g[b] = atomicAdd(cursor + k, loc[q]);
                    s_end[b] = foff[min((k + 1) * stride, nfine)];
                }
            }
            __syncthreads();
#pragma unroll
            for (uint32_t r = 0; r < PER; r++)
                if (r * PB_THREADS + threadIdx.x < tc) {
                    const uint32_t lk = key[r] - k0;
                    const uint32_t p = s_ofs[lk] + rank[r];
                    s_v[p] = v[r];
                    s_c[p] = c[r];
                    s_k[p] = (uint16_t)lk;
                }
            __syncthreads();
            for (uint32_t p = threadIdx.x; p < tc; p += PB_THREADS) {
                const uint32_t lk = s_k[p];
                const uint32_t gpos = s_g[lk] + (p - s_ofs[lk]);
                if (gpos < s_end[lk]) {
                    out_v[gpos] = s_v[p];
                    out_c[gpos] = s_c[p];
                } else {
                    bad = true;
                }
            }
        } else {
#pragma unroll
            for (uint32_t r = 0; r < PER; r++)
                if (r * PB_THREADS + threadIdx.x < tc) {
                    const uint32_t k = key[r];
                    if (k >= nkeys) {
                        bad = true;
                        continue;
                    }
                    const uint32_t gpos = atomicAdd(cursor + k, 1u);
                    if (gpos < foff[min((k + 1) * stride, nfine)]) {
                        out_v[gpos] = v[r];
                        out_c[gpos] = c[r];
                    } else {
                        bad = true;
                    }
                }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            v[r] = nv[r];
            c[r] = nc[r];
        }
    }
    if (bad) atomicOr(err, 1u);
}

// Resident push of a piece (every vertex active): slot t of [0, cnt) gets the contribution
// of its edge's source, the list entry j in [ja, jb) whose work range holds wa + t.
// tj[k] = the last entry whose range starts at or before tile k's first slot (computed
// once per piece by k_pb_tiles); a workgroup marks, in an LDS owner map, where each later
// entry of its tile starts, takes prefix maxima, and writes the tile with coalesced stores.
constexpr uint32_t PB_EXP_TILE = 4096;

__global__ void k_pb_tiles(const uint64_t* __restrict__ wpre, uint32_t ja, uint32_t jb, uint64_t wa, uint64_t cnt,
                           uint32_t* __restrict__ tj) {
    const uint64_t ntiles = (cnt + PB_EXP_TILE - 1) / PB_EXP_TILE;
    for (uint64_t k = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; k < ntiles;
         k += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t t = wa + k * PB_EXP_TILE;
        uint32_t lo = ja, hi = jb;  // wpre[ja] <= t < wpre[jb]
        while (hi - lo > 1) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if (wpre[mid] <= t)
                lo = mid;
            else
                hi = mid;
        }
        tj[k] = lo;
    }
}

// IDS: the slot gets the source itself instead of its contribution.
template <bool IDS>
__global__ __launch_bounds__(256) void k_pb_expand(const uint32_t* __restrict__ list,
                                                   const uint64_t* __restrict__ wpre, uint32_t jb, uint64_t wa,
                                                   uint64_t cnt, const uint32_t* __restrict__ tj,
                                                   const float* __restrict__ contrib, float* __restrict__ pc) {
    constexpr uint32_t PER = PB_EXP_TILE / 256;
    __shared__ uint16_t s_owner[PB_EXP_TILE];
    __shared__ float s_val[PB_EXP_TILE + 1];
    __shared__ uint32_t s_wave[4];
    const uint64_t ntiles = (cnt + PB_EXP_TILE - 1) / PB_EXP_TILE;
    for (uint64_t k = blockIdx.x; k < ntiles; k += gridDim.x) {
        const uint64_t t0 = k * PB_EXP_TILE;
        const uint32_t tc = (uint32_t)min((uint64_t)PB_EXP_TILE, cnt - t0);
        const uint32_t j0 = tj[k];
        // entries that start inside the tile: j0 + 1 .. (the next tile's first entry), each
        // at most one per slot
        const uint32_t jl = k + 1 < ntiles ? tj[k + 1] : jb - 1;
        const uint32_t nv = jl - j0 + 1;  // <= PB_EXP_TILE + 1
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) s_owner[r * 256 + threadIdx.x] = 0;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < nv; i += 256) {
            const uint32_t j = j0 + i;
            const uint32_t u = list[j];
            s_val[i] = IDS ? __uint_as_float(u) : contrib[u];
            if (i) {
                const uint64_t st = wpre[j] - wa;
                if (st < t0 + tc) s_owner[st - t0] = (uint16_t)i;
            }
        }
        __syncthreads();
        block_prefix_max_u16<PER>(s_owner, tc, s_wave);
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            const uint32_t q = r * 256 + threadIdx.x;
            if (q < tc) pc[t0 + q] = s_val[s_owner[q]];
        }
        __syncthreads();
    }
}

// First sort pass with fixed output places: workgroup w of the pass takes input slice
// [w * range, (w + 1) * range), and the pairs of that slice in bin k go to
// offA[w * nkeys + k] onwards (the slice's pairs and their bins are the same in every
// PageRank iteration, so the places are counted once).  No global atomics.
__global__ __launch_bounds__(PB_THREADS) void k_pb_count_a(const uint32_t* __restrict__ in_v, uint32_t vmask,
                                                           uint64_t cnt, uint64_t range, uint32_t kshift,
                                                           uint32_t nkeys, uint32_t* __restrict__ cntA,
                                                           uint32_t* __restrict__ err) {
    __shared__ uint32_t s_cnt[PB_LOCAL];
    for (uint32_t b = threadIdx.x; b < nkeys; b += PB_THREADS) s_cnt[b] = 0;
    __syncthreads();
    const uint64_t lo = blockIdx.x * range, hi = min(cnt, lo + range);
    bool bad = false;
    for (uint64_t i = lo + threadIdx.x; i < hi; i += PB_THREADS) {
        const uint32_t k = (in_v[i] & vmask) >> kshift;
        if (k < nkeys)
            atomicAdd(&s_cnt[k], 1u);
        else
            bad = true;
    }
    if (bad) atomicOr(err, 1u);
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nkeys; b += PB_THREADS) cntA[(uint64_t)blockIdx.x * nkeys + b] = s_cnt[b];
}

// offA[w][k] = start of bin k + pairs of bin k in slices before w (in place over cntA).
// One workgroup of PB_A_WG threads per bin k, thread w holding slice w.
__global__ __launch_bounds__(PB_A_WG) void k_pb_scan_a(uint32_t* __restrict__ cntA, uint32_t nwg, uint32_t nkeys,
                                                       uint32_t stride, const uint32_t* __restrict__ foff) {
    __shared__ uint32_t s_w[PB_A_WG / 64 + 1];
    const uint32_t k = blockIdx.x, w = threadIdx.x;
    const uint64_t at = (uint64_t)w * nkeys + k;
    const uint32_t c = w < nwg ? cntA[at] : 0u;
    uint32_t tot;
    const uint32_t before = block_excl_sum(c, s_w, &tot);
    if (w < nwg) cntA[at] = foff[k * stride] + before;
}

__global__ __launch_bounds__(PB_THREADS) void k_pb_scatter_a(const uint32_t* __restrict__ in_v, uint32_t vmask,
                                                             const float* __restrict__ in_c, uint64_t cnt,
                                                             uint64_t range, uint32_t kshift, uint32_t stride,
                                                             uint32_t nfine, const uint32_t* __restrict__ foff,
                                                             const uint32_t* __restrict__ offA,
                                                             uint32_t* __restrict__ out_v, float* __restrict__ out_c,
                                                             uint32_t* __restrict__ fcur, uint32_t* __restrict__ err) {
    constexpr uint32_t PER = PB_TILE / PB_THREADS;
    constexpr uint32_t LPER = PB_LOCAL / PB_THREADS;
    __shared__ uint32_t s_v[PB_TILE];
    __shared__ float s_c[PB_TILE];
    __shared__ uint16_t s_k[PB_TILE];
    __shared__ uint32_t s_cnt[PB_LOCAL], s_ofs[PB_LOCAL], s_run[PB_LOCAL], s_end[PB_LOCAL];
    __shared__ uint32_t s_w[PB_THREADS / 64 + 1];
    const uint32_t nkeys = (nfine + stride - 1) / stride;
    // the second pass's cursors start at the fine bins' starts
    if (fcur)
        for (uint32_t f = blockIdx.x * PB_THREADS + threadIdx.x; f < nfine; f += gridDim.x * PB_THREADS)
            fcur[f] = foff[f];
    for (uint32_t b = threadIdx.x; b < PB_LOCAL; b += PB_THREADS) {
        s_run[b] = b < nkeys ? offA[(uint64_t)blockIdx.x * nkeys + b] : 0u;
        s_end[b] = b < nkeys ? foff[min((b + 1) * stride, nfine)] : 0u;
    }
    bool bad = false;
    const uint64_t lo = blockIdx.x * range, hi = min(cnt, lo + range);
    uint32_t v[PER], key[PER], rank[PER];
    float c[PER];
    // every load of a tile in flight before any is used; the next tile's loads are issued
    // before the current tile is sorted
#pragma unroll
    for (uint32_t r = 0; r < PER; r++) {
        const uint64_t i = lo + r * PB_THREADS + threadIdx.x;
        v[r] = i < hi ? in_v[i] & vmask : 0u;
        c[r] = i < hi ? in_c[i] : 0.0f;
    }
    for (uint64_t t0 = lo; t0 < hi; t0 += PB_TILE) {
        const uint32_t tc = (uint32_t)min((uint64_t)PB_TILE, hi - t0);
        uint32_t nv[PER];
        float nc[PER];
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            const uint64_t i = t0 + PB_TILE + r * PB_THREADS + threadIdx.x;
            nv[r] = i < hi ? in_v[i] & vmask : 0u;
            nc[r] = i < hi ? in_c[i] : 0.0f;
        }
#pragma unroll
        for (uint32_t q = 0; q < LPER; q++) s_cnt[LPER * threadIdx.x + q] = 0;
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            key[r] = PB_LOCAL;
            rank[r] = 0;
            if (r * PB_THREADS + threadIdx.x < tc) {
                const uint32_t k = v[r] >> kshift;
                if (k < nkeys) {
                    key[r] = k;
                    rank[r] = atomicAdd(&s_cnt[k], 1u);
                } else {
                    bad = true;
                }
            }
        }
        __syncthreads();
        uint32_t loc[LPER], sum = 0, tot;
#pragma unroll
        for (uint32_t q = 0; q < LPER; q++) {
            loc[q] = s_cnt[LPER * threadIdx.x + q];
            sum += loc[q];
        }
        uint32_t base = block_excl_sum(sum, s_w, &tot);
#pragma unroll
        for (uint32_t q = 0; q < LPER; q++) {
            s_ofs[LPER * threadIdx.x + q] = base;
            base += loc[q];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < PER; r++)
            if (key[r] < PB_LOCAL) {
                const uint32_t p = s_ofs[key[r]] + rank[r];
                s_v[p] = v[r];
                s_c[p] = c[r];
                s_k[p] = (uint16_t)key[r];
            }
        __syncthreads();
        for (uint32_t p = threadIdx.x; p < tot; p += PB_THREADS) {
            const uint32_t k = s_k[p];
            const uint32_t gpos = s_run[k] + (p - s_ofs[k]);
            if (gpos < s_end[k]) {
                out_v[gpos] = s_v[p];
                out_c[gpos] = s_c[p];
            } else {
                bad = true;
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < LPER; q++) s_run[LPER * threadIdx.x + q] += loc[q];
        // the next tile's count reset follows this update (barrier after the reset)
#pragma unroll
        for (uint32_t r = 0; r < PER; r++) {
            v[r] = nv[r];
            c[r] = nc[r];
        }
    }
    if (bad) atomicOr(err, 1u);
}

constexpr int PB_ACC_THREADS = 512;
constexpr uint32_t PB_ACC_BATCH = 8;  // pairs per thread with loads in flight together

// FP32 sums, although the LDS adds FP64 ones ten times faster (k_pg_gather): a bin's FP64 sums
// take 128 KB of LDS, and workgroups of that size wait for a CU that the edge streams beside
// them have left (R-MAT 28 under 8 GB, 160 pieces: 2,709 ms with FP32 sums, 3,395 ms with FP64,
// and the streams 3% slower).
__global__ __launch_bounds__(PB_ACC_THREADS) void k_pb_accum(const uint32_t* __restrict__ pv,
                                                             const float* __restrict__ pc,
                                                             const uint32_t* __restrict__ foff,
                                                             const uint32_t* __restrict__ segs,
                                                             const uint32_t* __restrict__ nsegs, uint32_t seg,
                                                             uint64_t n, float* __restrict__ acc,
                                                             uint32_t* __restrict__ err) {
    constexpr uint32_t Q4 = PB_FINE / 4 / PB_ACC_THREADS;  // float4 slots per thread
    __shared__ float4 s_a4[PB_FINE / 4];
    float* s_a = (float*)s_a4;
    const uint32_t s = blockIdx.x;
    if (s >= *nsegs) return;  // the same for every thread of the workgroup
    const uint32_t f = segs[2 * s], j = segs[2 * s + 1];
    const uint32_t b0 = foff[f], b1 = foff[f + 1];
    const uint32_t start = b0 + j * seg;
    const uint32_t end = min(b1, start + seg);
    const bool multi = b1 - b0 > seg;
#pragma unroll
    for (uint32_t q = 0; q < Q4; q++) s_a4[q * PB_ACC_THREADS + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    bool bad = false;
    for (uint32_t i0 = start; i0 < end; i0 += PB_ACC_BATCH * PB_ACC_THREADS) {
        uint32_t v[PB_ACC_BATCH];
        float c[PB_ACC_BATCH];
#pragma unroll
        for (uint32_t r = 0; r < PB_ACC_BATCH; r++) {
            const uint32_t i = i0 + r * PB_ACC_THREADS + threadIdx.x;
            v[r] = i < end ? pv[i] : UINT32_MAX;
            c[r] = i < end ? pc[i] : 0.0f;
        }
#pragma unroll
        for (uint32_t r = 0; r < PB_ACC_BATCH; r++) {
            if (i0 + r * PB_ACC_THREADS + threadIdx.x >= end) continue;
            if ((v[r] >> PB_FINE_SHIFT) == f && v[r] < n)
                atomicAdd(&s_a[acc_slot(v[r]) & (PB_FINE - 1)], c[r]);
            else
                bad = true;
        }
    }
    if (bad) atomicOr(err, 1u);
    __syncthreads();
    // the bin's accumulator slots: [base, base + lim), lim a multiple of 4096
    const uint64_t base = (uint64_t)f << PB_FINE_SHIFT;
    const uint32_t lim4 = (uint32_t)min((uint64_t)PB_FINE, acc_slots(n) - base) / 4;
    if (!multi) {
        float4* a4 = (float4*)(acc + base);
        float4 x[Q4];
#pragma unroll
        for (uint32_t q = 0; q < Q4; q++) {
            const uint32_t k = q * PB_ACC_THREADS + threadIdx.x;
            if (k < lim4) x[q] = a4[k];
        }
#pragma unroll
        for (uint32_t q = 0; q < Q4; q++) {
            const uint32_t k = q * PB_ACC_THREADS + threadIdx.x;
            if (k < lim4) {
                const float4 y = s_a4[k];
                x[q].x += y.x;
                x[q].y += y.y;
                x[q].z += y.z;
                x[q].w += y.w;
                a4[k] = x[q];
            }
        }
    } else {
        for (uint32_t q = threadIdx.x; q < lim4 * 4; q += PB_ACC_THREADS)
            if (s_a[q] != 0.0f) unsafeAtomicAdd(acc + base + q, s_a[q]);
    }
}

// ----------------------------------------------------------- in-edge lists
// In-degrees, then their prefix sums (edges, and segments of IN_SEG edges per vertex), then
// the sources placed by atomic cursors; a list's order is of no account.
__global__ __launch_bounds__(256) void k_in_count(const uint32_t* __restrict__ col, uint32_t vmask, uint64_t m,
                                                  uint64_t n, uint32_t* __restrict__ cnt) {
    for (uint64_t e = blockIdx.x * 256ull + threadIdx.x; e < m; e += (uint64_t)gridDim.x * 256) {
        const uint32_t v = col[e] & vmask;
        if (v < n) atomicAdd(cnt + v, 1u);
    }
}

constexpr uint32_t IN_TILE = 4096;  // vertices per workgroup of the prefix sums, 16 per thread

__device__ __forceinline__ uint32_t in_segs(uint32_t c) { return (c + IN_SEG - 1) / IN_SEG; }

// tot[2 k], tot[2 k + 1] = edges and segments of tile k.
__global__ __launch_bounds__(256) void k_in_tot(const uint32_t* __restrict__ cnt, uint64_t n,
                                                uint64_t* __restrict__ tot) {
    __shared__ uint64_t s_t[4][2];
    uint64_t a = 0, b = 0;
    for (uint32_t q = threadIdx.x; q < IN_TILE; q += 256) {
        const uint64_t v = (uint64_t)blockIdx.x * IN_TILE + q;
        const uint32_t c = v < n ? cnt[v] : 0u;
        a += c;
        b += in_segs(c);
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if ((threadIdx.x & 63) == 0) {
        s_t[threadIdx.x >> 6][0] = a;
        s_t[threadIdx.x >> 6][1] = b;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        tot[2 * (uint64_t)blockIdx.x + threadIdx.x] =
            s_t[0][threadIdx.x] + s_t[1][threadIdx.x] + s_t[2][threadIdx.x] + s_t[3][threadIdx.x];
}

// One wave: the tiles' totals become their bases; toff[n] and soff[n] the grand totals.
__global__ __launch_bounds__(64) void k_in_base(uint64_t tiles, uint64_t* __restrict__ tot, uint64_t n,
                                                uint64_t* __restrict__ toff, uint32_t* __restrict__ soff) {
    uint64_t ra = 0, rb = 0;
    for (uint64_t k0 = 0; k0 < tiles; k0 += 64) {
        const uint64_t k = k0 + threadIdx.x;
        uint64_t ta, tb;
        const uint64_t a = wave_exclusive_sum(k < tiles ? tot[2 * k] : 0, &ta);
        const uint64_t b = wave_exclusive_sum(k < tiles ? tot[2 * k + 1] : 0, &tb);
        if (k < tiles) {
            tot[2 * k] = ra + a;
            tot[2 * k + 1] = rb + b;
        }
        ra += ta;
        rb += tb;
    }
    if (threadIdx.x == 0) {
        toff[n] = ra;
        if (soff) soff[n] = (uint32_t)rb;
    }
}

__global__ __launch_bounds__(256) void k_in_write(uint32_t* __restrict__ cnt, uint64_t n,
                                                  const uint64_t* __restrict__ tot, uint64_t* __restrict__ toff,
                                                  uint32_t* __restrict__ soff, uint32_t* __restrict__ seg_v) {
    constexpr uint32_t PER = IN_TILE / 256;
    __shared__ uint64_t s_t[4][2];
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint64_t v0 = (uint64_t)blockIdx.x * IN_TILE + threadIdx.x * PER;
    uint32_t c[PER];
    uint64_t a = 0, b = 0;
#pragma unroll
    for (uint32_t q = 0; q < PER; q++) {
        c[q] = v0 + q < n ? cnt[v0 + q] : 0u;
        a += c[q];
        b += in_segs(c[q]);
    }
    uint64_t ta, tb;
    uint64_t ea = wave_exclusive_sum(a, &ta), eb = wave_exclusive_sum(b, &tb);
    if (lane == 0) {
        s_t[wid][0] = ta;
        s_t[wid][1] = tb;
    }
    __syncthreads();
    ea += tot[2 * (uint64_t)blockIdx.x];
    eb += tot[2 * (uint64_t)blockIdx.x + 1];
    for (uint32_t w = 0; w < wid; w++) {
        ea += s_t[w][0];
        eb += s_t[w][1];
    }
#pragma unroll
    for (uint32_t q = 0; q < PER; q++) {
        const uint64_t v = v0 + q;
        if (v >= n) break;
        toff[v] = ea;
        if (soff) {  // else only the edges are wanted
            soff[v] = (uint32_t)eb;
            const uint32_t sg = in_segs(c[q]);
            for (uint32_t k = 0; k < sg; k++) seg_v[eb + k] = (uint32_t)v;
            eb += sg;
        }
        ea += c[q];
        cnt[v] = 0;  // the scatter's cursors
    }
}

// Largest u in [lo, hi) with off[u] <= e (off[lo] <= e): the source of edge e.
__device__ __forceinline__ uint64_t source_of(const uint64_t* __restrict__ off, uint64_t lo, uint64_t hi, uint64_t e) {
    while (hi - lo > 1) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (off[mid] <= e)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// A wave takes 64 consecutive edges: it finds the sources of the first and the last, and each
// lane its own between them.
__global__ __launch_bounds__(256) void k_in_scatter(const uint64_t* __restrict__ off, const uint32_t* __restrict__ col,
                                                    const uint32_t* __restrict__ w, Pack pk, uint64_t m, uint64_t n,
                                                    const uint64_t* __restrict__ toff, uint32_t* __restrict__ cur,
                                                    uint32_t* __restrict__ tsrc, uint32_t* __restrict__ tdst,
                                                    uint32_t* __restrict__ tw) {
    for (uint64_t e0 = (blockIdx.x * 256ull + threadIdx.x) & ~63ull; e0 < m; e0 += (uint64_t)gridDim.x * 256) {
        const uint64_t e = e0 + (threadIdx.x & 63);
        const uint64_t u0 = source_of(off, 0, n, e0);
        const uint64_t u1 = source_of(off, u0, n, min(e0 + 63, m - 1));
        if (e >= m) continue;
        const uint64_t u = source_of(off, u0, u1 + 1, e);
        const uint32_t c = col[e], v = pk_v(c, pk);
        if (v < n) {
            const uint64_t at = toff[v] + atomicAdd(cur + v, 1u);
            tsrc[at] = (uint32_t)u;
            tdst[at] = v;
            if (tw) tw[at] = pk_w(c, pk.shift == 32 ? load_w(w, e, pk) : 0u, pk);
        }
    }
}

// Lane rows over in-edges: a step of personalized PageRank (the active sources' shares summed)
// or of batched SSSP (the least distance over the active sources).  Two forms by the width
// of a row, S = 2^LSH:
//
// Rows of 16 lanes and more (k_pull_runs): S threads take a run of `run` consecutive
// in-edges, S of them at a time: each thread loads one edge's source, destination and lane
// mask, then all of them take the sources' rows, one lane per thread, IN_UNROLL rows in
// flight, and hand the result over whenever the destination changes.  A destination inside
// the run is written with plain stores (no other run holds its edges); the run's first and
// last one may continue in the neighbouring runs and are updated atomically.
//
// Narrower rows, PPR's only (k_pull_segs): 16 threads take a segment of one vertex's in-list, 16 / S of
// its edges at once.
//
// Bound by the gathered rows (a wave per vertex waited through six dependent loads for the
// few edges of an average in-list).  Measured on R-MAT 20 with 64 PPR lanes: 16M rows of 256
// bytes in 1.3 ms, 3.3 TB/s; the push's FP64 atomic adds took 10 ms.
//
// Four rows in flight per wave suffice with 8 waves on a SIMD, and more registers cost waves:
// 37 lanes of SSSP on R-MAT 18 3.65 ms with eight, 3.34 with four.  Long runs cut fewer lists
// (atomics), short ones give small graphs enough waves: with runs of 64 / 128 / 256 / 512 edges,
// R-MAT 20 PPR 26.8 / 20.4 / 18.4 / 18.6 ms, uniform 2^18 with 64 SSSP lanes 12.6 / 8.2 / 7.3 / 7.0,
// R-MAT 18 with 37 4.2 / 3.34 / 3.40 / 4.05, R-MAT 16 PPR 2.60 / 2.12 / 2.55 / 3.40, 70K vertices
// with 17 lanes 1.38 / 1.59 / 2.26 / 3.52: a run is the longest power of two that gives
// PULL_WAVES waves, at most IN_RUN_MAX and at least 64 and two rounds of its S threads.
constexpr int IN_UNROLL = 4;
constexpr uint32_t IN_RUN_MAX = 256, PULL_WAVES = 12288;

// What a destination gathers: PPR sums in FP64 and the lanes that received a share, SSSP the
// least candidate distance.
struct PullPpr {
    typedef double Acc;
    static constexpr bool weighted = false;
    static __device__ __forceinline__ Acc none() { return 0.0; }
    static __device__ __forceinline__ Acc join(Acc a, Acc b) { return a + b; }
    // value of lane ln of source u's row, for an edge of weight w whose source has the lanes mu active
    template <int LSH>
    static __device__ __forceinline__ float take(const AlgoState& s, uint32_t u, uint64_t mu, uint32_t ln) {
        return mu ? s.lx[((uint64_t)u << LSH) + ln] : 0.0f;
    }
    static __device__ __forceinline__ Acc value(const AlgoState&, float x, uint32_t, uint64_t, uint32_t) { return x; }
    // the result of destination v, handed over by the S threads of its row
    template <int LSH>
    static __device__ __forceinline__ void hand_over(const AlgoState& s, uint32_t v, uint32_t ln, Acc acc, uint64_t m,
                                                     bool shared) {
        if (!m) return;
        double* av = s.lacc + ((uint64_t)v << LSH);
        if (shared) {
            if ((m >> ln) & 1) unsafeAtomicAdd(av + ln, acc);
            if (ln == 0) atomicOr((unsigned long long*)(s.mnext + v), (unsigned long long)m);
        } else {
            av[ln] = acc;  // the sums are zero before
            if (ln == 0) s.mnext[v] = m;
        }
        if (ln == 0) mark_next(s.next, v);
    }
};

struct PullSssp {
    typedef uint32_t Acc;
    static constexpr bool weighted = true;
    static __device__ __forceinline__ Acc none() { return UNREACHED; }
    static __device__ __forceinline__ Acc join(Acc a, Acc b) { return a < b ? a : b; }
    template <int LSH>
    static __device__ __forceinline__ uint32_t take(const AlgoState& s, uint32_t u, uint64_t mu, uint32_t ln) {
        return (mu >> ln) & 1 ? s.lval[((uint64_t)u << LSH) + ln] : 0u;
    }
    static __device__ __forceinline__ Acc value(const AlgoState& s, uint32_t x, uint32_t w, uint64_t mu, uint32_t ln) {
        if (!((mu >> ln) & 1)) return UNREACHED;
        const uint64_t nd = (uint64_t)x + w;
        if (nd >= UNREACHED) {
            atomicOr(s.overflow + (ln >> 5), 1u << (ln & 31));
            return UNREACHED;
        }
        return (uint32_t)nd;
    }
    template <int LSH>
    static __device__ __forceinline__ void hand_over(const AlgoState& s, uint32_t v, uint32_t ln, Acc acc, uint64_t m,
                                                     bool shared) {
        if (!m) return;
        uint32_t* dv = s.lval + ((uint64_t)v << LSH) + ln;
        bool better = acc < *dv;
        if (better) {
            if (shared)
                better = acc < atomicMin(dv, acc);
            else
                *dv = acc;
        }
        const uint64_t rowmask = LSH >= 6 ? ~0ull : ((1ull << (1u << LSH)) - 1);
        const uint64_t g = (__ballot(better) >> (__lane_id() & ~((1u << LSH) - 1))) & rowmask;
        if (ln == 0 && g) {
            if (shared)
                atomicOr((unsigned long long*)(s.mnext + v), (unsigned long long)g);
            else
                s.mnext[v] = g;
            mark_next(s.next, v);
        }
    }
};

template <int LSH, class P>
__global__ __launch_bounds__(256) void k_pull_runs(AlgoState s, InLists in, uint32_t run_len) {
    constexpr uint32_t S = 1u << LSH;
    const uint32_t lane = threadIdx.x & 63, ln = lane & (S - 1), g0 = lane & ~(S - 1);
    const uint64_t groups = (uint64_t)gridDim.x * (256u >> LSH);
    const uint64_t runs = (in.m + run_len - 1) / run_len;
    const uint64_t first = (blockIdx.x * 256ull + threadIdx.x) >> LSH;
    // whole waves stay together: a group past the last run goes through the loop with no edges
    for (uint64_t w0 = first - (lane >> LSH); w0 < runs; w0 += groups) {
        const uint64_t run = w0 + (lane >> LSH);
        const uint64_t b = min(run * run_len, in.m), e = min(b + run_len, in.m);
        uint32_t cur = UNREACHED;
        bool head = b > 0 && b < e && in.tdst[b - 1] == in.tdst[b];  // the first destination began earlier
        typename P::Acc acc = P::none();
        uint64_t got = 0;
        for (uint32_t k = 0; k < run_len; k += S) {
            const uint64_t i = b + k + ln;
            const bool ok = i < e;
            const uint32_t u = ok ? in.tsrc[i] : 0u, d = ok ? in.tdst[i] : UNREACHED;
            const uint32_t w = P::weighted && ok ? in.tw[i] : 0u;
            const uint64_t mu = ok ? s.mcur[u] : 0ull;
#pragma unroll 1
            for (uint32_t t = 0; t < S; t += IN_UNROLL) {
                decltype(P::template take<LSH>(s, 0u, 0ull, 0u)) x[IN_UNROLL];
                uint32_t dd[IN_UNROLL], ww[IN_UNROLL];
                uint64_t mm[IN_UNROLL];
#pragma unroll
                for (int r = 0; r < IN_UNROLL; r++) {
                    uint32_t uu;
                    ww[r] = 0;
                    if constexpr (LSH == 6) {
                        uu = __builtin_amdgcn_readlane(u, t + r);
                        dd[r] = __builtin_amdgcn_readlane(d, t + r);
                        if (P::weighted) ww[r] = __builtin_amdgcn_readlane(w, t + r);
                        mm[r] = (uint32_t)__builtin_amdgcn_readlane((uint32_t)mu, t + r) |
                                (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(mu >> 32), t + r) << 32;
                    } else {
                        uu = __shfl(u, g0 + t + r, 64);
                        dd[r] = __shfl(d, g0 + t + r, 64);
                        if (P::weighted) ww[r] = __shfl(w, g0 + t + r, 64);
                        mm[r] = __shfl((uint32_t)mu, g0 + t + r, 64);
                    }
                    x[r] = P::template take<LSH>(s, uu, mm[r], ln);
                }
#pragma unroll
                for (int r = 0; r < IN_UNROLL; r++) {
                    if (dd[r] != cur) {
                        if (cur != UNREACHED) {
                            P::template hand_over<LSH>(s, cur, ln, acc, got, head);
                            head = false;
                        }
                        cur = dd[r];
                        acc = P::none();
                        got = 0;
                    }
                    acc = P::join(acc, P::value(s, x[r], ww[r], mm[r], ln));
                    got |= mm[r];
                }
            }
        }
        // the last destination: past a short run's end it has been handed over already
        if (cur != UNREACHED)
            P::template hand_over<LSH>(s, cur, ln, acc, got, head || (e < in.m && in.tdst[e] == cur));
    }
}

template <int LSH>
__global__ __launch_bounds__(256) void k_pull_segs(AlgoState s, InLists in) {
    constexpr uint32_t S = 1u << LSH, W = 16, E = W / S;
    const uint32_t sl = threadIdx.x & (W - 1), grp = sl >> LSH, ln = sl & (S - 1);
    const uint64_t groups = gridDim.x * (256ull / W);
    for (uint64_t sg = (blockIdx.x * 256ull + threadIdx.x) / W; sg < in.nseg; sg += groups) {  // uniform over 16 threads
        const uint32_t v = in.seg_v[sg];
        const uint32_t s0 = in.soff[v];
        const bool multi = in.soff[v + 1] - s0 > 1;
        const uint64_t b = in.toff[v] + (sg - s0) * IN_SEG;
        const uint64_t e = min(b + IN_SEG, in.toff[v + 1]);
        double acc = 0.0;
        uint32_t m = 0;  // S <= 8 lanes
        for (uint64_t i = b; i < e; i += W) {
            const bool ok = i + sl < e;
            const uint32_t u = ok ? in.tsrc[i + sl] : 0u;
            const uint32_t mu = ok ? (uint32_t)s.mcur[u] : 0u;
            m |= mu;
            float x[S];
#pragma unroll
            for (uint32_t t = 0; t < S; t++) {
                const uint32_t q = t * E + grp;
                x[t] = PullPpr::take<LSH>(s, __shfl(u, q, W), __shfl(mu, q, W), ln);
            }
#pragma unroll
            for (uint32_t t = 0; t < S; t++) acc += x[t];
        }
#pragma unroll
        for (uint32_t d = W / 2; d >= 1; d >>= 1) m |= __shfl_xor(m, d, W);
#pragma unroll
        for (uint32_t d = S; d < W; d <<= 1) acc += __shfl_xor(acc, (int)d, W);
        if (grp == 0) PullPpr::hand_over<LSH>(s, v, ln, acc, m, multi);
    }
}

// ------------------------------------------------- PageRank gather plan
// The pairs of a piece, kept sorted by destination bin between iterations: the source id
// and the 16-bit place of the destination in its bin's LDS sums.  An iteration then reads 6
// bytes per edge and the source's contribution, instead of writing, sorting and reading
// back (destination, contribution) pairs.

// Place of a bin's k-th vertex in its LDS sums: the low 6 bits are XORed with a hash of the
// rest (a bijection on each aligned run of 64), so that hub ids, which share many zero low
// bits, spread over the banks.
__device__ __forceinline__ uint32_t pg_place(uint32_t k) { return k ^ (((k >> 6) * 0x9E3779B1u) >> 26); }

__global__ __launch_bounds__(256) void k_pg_pack(const uint32_t* __restrict__ v, uint64_t cnt, uint32_t shift,
                                                 uint64_t n, uint16_t* __restrict__ slot,
                                                 uint32_t* __restrict__ err) {
    const uint32_t mask = (1u << shift) - 1;
    bool bad = false;
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < cnt; i += (uint64_t)gridDim.x * 256) {
        const uint32_t d = v[i];
        if (d >= n) bad = true;
        slot[i] = (uint16_t)pg_place(d & mask);
    }
    if (bad) atomicOr(err, 1u);
}


typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One workgroup per accumulation segment (as k_pb_accum): the segment's pairs are read eight
// to a thread with 16-byte loads, each source's contribution is gathered and added into the
// bin's sums in LDS, and the sums are added to acc (plain read-modify-write when the bin is
// one segment, atomic adds of the non-zero sums when it spans several).  The pairs of the
// piece start at e0 of src / slot, which are padded to a multiple of eight.
// The sums are FP64: an LDS add of 64 lanes takes 193 cycles of a CU in FP32 whatever the
// places (3 per lane), 20 in FP64 at random places, 9 in order.
// Measured on R-MAT 24 (263M pairs, 20 iterations), against 135 ms for expanding, sorting and
// summing the pairs: FP32 sums 32.6 ms (32.2 without the gathers, 21.8 without the adds), FP64
// 22.1, with the next pairs loaded ahead 20.6 ms, 0.26 T edges/s.  Bound by the gathers then
// (contributions without the gaps of vertices that have no out-edges fetch fewer lines and take
// as long).  Bins of 2^11 / 2^12 / 2^13 / 2^14 sums 22.0 / 21.6 / 20.6 / 21.8 ms; pieces of 3n /
// 4n pairs 21.4 / 20.6 ms, of 8n at 2^12 24.7 against 22.9 ms (each piece adds every vertex's
// sum once more, larger ones spread their sources over more of the L2).
__global__ __launch_bounds__(512) void k_pg_gather(const uint32_t* __restrict__ src,
                                                          const uint16_t* __restrict__ slot, uint64_t e0,
                                                          const uint32_t* __restrict__ foff,
                                                          const uint32_t* __restrict__ segs, uint32_t seg,
                                                          uint32_t shift, uint64_t n,
                                                          const float* __restrict__ contrib,
                                                          float* __restrict__ acc) {
    extern __shared__ double s_a[];
    const uint32_t f = segs[2 * blockIdx.x], j = segs[2 * blockIdx.x + 1];
    const uint32_t b0 = foff[f], b1 = foff[f + 1];
    const bool multi = b1 - b0 > seg;
    const uint64_t a0 = e0 + b0 + (uint64_t)j * seg, a1 = min(e0 + b1, a0 + seg);
    const uint32_t fine = 1u << shift;
    for (uint32_t k = threadIdx.x; k < fine; k += blockDim.x) s_a[k] = 0.0;
    __syncthreads();
    const u32x4* src4 = (const u32x4*)src;
    const u32x4* slot8 = (const u32x4*)slot;
    // the next group's pairs are on their way while the present one's contributions are gathered
    uint64_t g = (a0 >> 3) + threadIdx.x;
    u32x4 p{}, q{}, z{};
    if ((g << 3) < a1) {
        p = __builtin_nontemporal_load(src4 + 2 * g);
        q = __builtin_nontemporal_load(src4 + 2 * g + 1);
        z = __builtin_nontemporal_load(slot8 + g);
    }
    while ((g << 3) < a1) {
        const uint32_t u[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
        const uint32_t zz[4] = {z.x, z.y, z.z, z.w};
        const uint64_t i0 = g << 3;
        const bool whole = i0 >= a0 && i0 + 8 <= a1;
        float c[8];
        if (whole) {
#pragma unroll
            for (int r = 0; r < 8; r++) c[r] = contrib[u[r]];
        }
        g += blockDim.x;
        if ((g << 3) < a1) {
            p = __builtin_nontemporal_load(src4 + 2 * g);
            q = __builtin_nontemporal_load(src4 + 2 * g + 1);
            z = __builtin_nontemporal_load(slot8 + g);
        }
        if (whole) {
#pragma unroll
            for (int r = 0; r < 8; r++)
                unsafeAtomicAdd(&s_a[(zz[r >> 1] >> (16 * (r & 1))) & 0xFFFFu], (double)c[r]);
        } else {  // the segment's first or last group: its pairs only
#pragma unroll
            for (int r = 0; r < 8; r++)
                if (i0 + r >= a0 && i0 + r < a1)
                    unsafeAtomicAdd(&s_a[(zz[r >> 1] >> (16 * (r & 1))) & 0xFFFFu], (double)contrib[u[r]]);
        }
    }
    __syncthreads();
    const uint64_t base = (uint64_t)f << shift;
    const uint32_t lim = (uint32_t)min((uint64_t)fine, n - base);
    if (!multi) {
        for (uint32_t k = threadIdx.x; k < lim; k += blockDim.x) acc[base + k] += (float)s_a[pg_place(k)];
    } else {
        for (uint32_t k = threadIdx.x; k < lim; k += blockDim.x) {
            const float y = (float)s_a[pg_place(k)];
            if (y != 0.0f) unsafeAtomicAdd(acc + base + k, y);
        }
    }
}

// The compact plan of a budgeted graph's resident edges: a pair is one word, the low 16 bits of
// the source under the destination's place in its bin, and pairs are sorted by bin and within
// it by block of 2^16 sources; start[f * blocks + p] = the first pair of bin f from block p.
// A workgroup takes chunks of RG_CHUNK consecutive edges and of each its source blocks one by
// one: the bins' pairs are counted in LDS and added to cnt, one atomic per bin (an atomic per
// pair took 25 ms of 16M pairs on R-MAT 22, whose hub bin takes one pair in twenty); SCATTER
// takes the places so reserved and deals them out in LDS.
constexpr uint32_t RG_CHUNK = 1u << 15;
template <bool SCATTER>
__global__ __launch_bounds__(512) void k_rg_sort(const uint64_t* __restrict__ off, const uint32_t* __restrict__ col,
                                                 uint32_t vmask, uint64_t m, uint64_t nv, uint64_t n, uint32_t shift,
                                                 uint32_t nfine, uint32_t blocks, const uint64_t* __restrict__ start,
                                                 uint32_t* __restrict__ cnt, uint32_t* __restrict__ pairs,
                                                 uint32_t* __restrict__ err) {
    extern __shared__ uint32_t s_h[];
    __shared__ uint64_t s_u[2];
    const uint32_t mask = (1u << shift) - 1, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    bool bad = false;
    for (uint64_t e0 = (uint64_t)blockIdx.x * RG_CHUNK; e0 < m; e0 += (uint64_t)gridDim.x * RG_CHUNK) {
        const uint64_t e1 = min(e0 + RG_CHUNK, m);
        if (threadIdx.x < 2) s_u[threadIdx.x] = source_of(off, 0, nv, threadIdx.x ? e1 - 1 : e0);
        __syncthreads();
        const uint64_t ua = s_u[0], ub = s_u[1];
        for (uint64_t p = ua >> 16; p <= ub >> 16; p++) {  // uniform across the workgroup
            const uint64_t ea = max(e0, off[min(p << 16, nv)]), eb = min(e1, off[min((p + 1) << 16, nv)]);
            if (ea >= eb) continue;
            for (uint32_t f = threadIdx.x; f < nfine; f += 512) s_h[f] = 0;
            __syncthreads();
            for (uint64_t e = ea + threadIdx.x; e < eb; e += 512) {
                const uint32_t v = col[e] & vmask;
                if (v < n)
                    atomicAdd(&s_h[v >> shift], 1u);
                else
                    bad = true;
            }
            __syncthreads();
            for (uint32_t f = threadIdx.x; f < nfine; f += 512) {
                if (!s_h[f]) continue;
                const uint64_t key = (uint64_t)f * blocks + p;
                const uint32_t base = atomicAdd(cnt + key, s_h[f]);
                if (SCATTER) s_h[f] = (uint32_t)start[key] + base;
            }
            __syncthreads();
            if (SCATTER) {
                const uint64_t ul = max(ua, p << 16), uh = min(ub, (p << 16) | 0xFFFF);
                for (uint64_t w0 = ea + wid * 64; w0 < eb; w0 += 512) {  // uniform across the wave
                    const uint64_t e = w0 + lane;
                    const uint64_t u0 = source_of(off, ul, uh + 1, w0);
                    const uint64_t u1 = source_of(off, u0, uh + 1, min(w0 + 63, eb - 1));
                    if (e >= eb) continue;
                    const uint64_t u = source_of(off, u0, u1 + 1, e);
                    const uint32_t v = col[e] & vmask;
                    if (v < n)
                        pairs[atomicAdd(&s_h[v >> shift], 1u)] = (uint32_t)(u & 0xFFFFu) | pg_place(v & mask) << 16;
                }
                __syncthreads();
            }
        }
        __syncthreads();  // s_u is written again
    }
    if (bad) atomicOr(err, 1u);
}

__global__ void k_rg_hist(const uint64_t* __restrict__ start, uint32_t nfine, uint32_t blocks,
                          uint32_t* __restrict__ hist) {
    const uint32_t f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f < nfine) hist[f] = (uint32_t)(start[(uint64_t)(f + 1) * blocks] - start[(uint64_t)f * blocks]);
}

// As k_pg_gather over the compact plan: eight pairs to a thread, whose source block is found
// among the bin's block starts (in LDS) for the first pair and followed from there.  The sums go
// to the accumulator copy of the blocked adds (acc_slot order) beside the streamed atomic adds.
__global__ __launch_bounds__(256) void k_rg_gather(const uint32_t* __restrict__ pairs,
                                                   const uint64_t* __restrict__ start, uint32_t blocks,
                                                   const uint32_t* __restrict__ foff,
                                                   const uint32_t* __restrict__ segs, uint32_t seg, uint32_t shift,
                                                   uint64_t n, const float* __restrict__ contrib,
                                                   float* __restrict__ acc) {
    extern __shared__ double s_a[];
    const uint32_t fine = 1u << shift;
    uint32_t* s_b = (uint32_t*)(s_a + fine);  // blocks + 1 starts
    const uint32_t f = segs[2 * blockIdx.x], j = segs[2 * blockIdx.x + 1];
    const uint32_t b0 = foff[f], b1 = foff[f + 1];
    const bool multi = b1 - b0 > seg;
    const uint64_t a0 = b0 + (uint64_t)j * seg, a1 = min((uint64_t)b1, a0 + seg);
    for (uint32_t k = threadIdx.x; k < fine; k += 256) s_a[k] = 0.0;
    for (uint32_t k = threadIdx.x; k <= blocks; k += 256) s_b[k] = (uint32_t)start[(uint64_t)f * blocks + k];
    __syncthreads();
    const u32x4* p4 = (const u32x4*)pairs;
    for (uint64_t g = (a0 >> 3) + threadIdx.x; (g << 3) < a1; g += 256) {
        const u32x4 x = __builtin_nontemporal_load(p4 + 2 * g), y = __builtin_nontemporal_load(p4 + 2 * g + 1);
        const uint32_t w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        const uint64_t i0 = g << 3, ia = max(i0, a0);
        uint32_t lo = 0, hi = blocks;  // s_b[lo] <= ia < s_b[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_b[mid] <= ia)
                lo = mid;
            else
                hi = mid;
        }
        float c[8];
#pragma unroll
        for (int r = 0; r < 8; r++) {
            const uint64_t i = i0 + r;
            if (i >= a0 && i < a1) {
                while (i >= s_b[lo + 1]) lo++;  // i < a1 <= s_b[blocks]
                c[r] = contrib[(lo << 16) + (w[r] & 0xFFFFu)];
            } else {
                c[r] = 0.0f;
            }
        }
#pragma unroll
        for (int r = 0; r < 8; r++)
            if (i0 + r >= a0 && i0 + r < a1) unsafeAtomicAdd(&s_a[w[r] >> 16], (double)c[r]);
    }
    __syncthreads();
    const uint64_t base = (uint64_t)f << shift;
    const uint32_t lim = (uint32_t)min((uint64_t)fine, n - base);
    for (uint32_t k = threadIdx.x; k < lim; k += 256) {
        const float y = (float)s_a[pg_place(k)];
        float* at = acc + acc_slot((uint32_t)(base + k));
        if (!multi)
            *at += y;
        else if (y != 0.0f)
            unsafeAtomicAdd(at, y);
    }
}

// contrib = x / D_o, acc cleared: before the first iteration.
__global__ void k_pg_start(uint64_t n, const uint64_t* __restrict__ off, const float* __restrict__ x,
                           float* __restrict__ contrib, float* __restrict__ acc) {
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t d = off[v + 1] - off[v];
        contrib[v] = d ? x[v] / (float)d : 0.0f;
        acc[v] = 0.0f;
    }
}

// An iteration's ranks: x after the last one, else the next iteration's contributions
// (with acc cleared for it), in one pass over the vertices.
template <bool LAST>
__global__ void k_pg_apply(uint64_t n, const uint64_t* __restrict__ off, float* __restrict__ x,
                           float* __restrict__ contrib, float* __restrict__ acc, float base, float damping,
                           const float* __restrict__ inv_n, float restart) {
    for (uint64_t v = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; v < n; v += (uint64_t)gridDim.x * blockDim.x) {
        const float r = (inv_n ? restart * inv_n[v] : base) + damping * acc[v];
        if (LAST) {
            x[v] = r;
        } else {
            const uint64_t d = off[v + 1] - off[v];
            contrib[v] = d ? r / (float)d : 0.0f;
            acc[v] = 0.0f;
        }
    }
}

// ---------------------------------------------------------- filter stream
// One workgroup pass = one chunk of FSTREAM_LINES lines of one task.  All lines of the
// chunk are loaded (the filter engine transfers whole partitions); an edge is pushed
// when it lies in the out-edge range of one of the task's active vertices.
// The chunk's host loads are issued as soon as the chunk is located, so the search for
// its active vertices and their staging overlap the link latency.  Staged ranges are
// chunk-relative 16-bit offsets, and each edge finds its vertex through an owner map
// (the index of the last active vertex starting at or before it, by prefix maximum).
template <class Op>
__global__ __launch_bounds__(LINE_THREADS) void k_push_fstream(const FTask* __restrict__ tasks, uint32_t ntasks,
                                                               uint64_t total_chunks,
                                                               const uint32_t* __restrict__ list,
                                                               const uint64_t* __restrict__ off,
                                                               const uint32_t* __restrict__ col,
                                                               const uint32_t* __restrict__ w, Op op, Pack pk) {
    constexpr uint32_t MAXE = FSTREAM_LINES * 32;  // edges per chunk (1536)
    constexpr int UNROLL = FSTREAM_LINES / LINE_HALVES;
    static_assert(MAXE <= 8 * LINE_THREADS, "owner map prefix covers 8 entries per thread");
    static_assert(FSTREAM_LINES % LINE_HALVES == 0, "whole lines per half wave");
    __shared__ uint16_t s_owner[MAXE];  // chunk position -> staged vertex
    __shared__ uint16_t s_s[MAXE];      // staged vertex range, relative to the chunk start
    __shared__ uint16_t s_e[MAXE];
    __shared__ uint32_t s_val[MAXE];
    __shared__ uint32_t s_tmp, s_wave[LINE_THREADS / 64];
    const uint32_t half = threadIdx.x >> 5, lane = threadIdx.x & 31;
    for (uint64_t c = blockIdx.x; c < total_chunks; c += gridDim.x) {
        // task of chunk c: last t with tasks[t].chunk0 <= c (tasks[0].chunk0 = 0)
        const uint32_t ti = block_search_last(0, ntasks, [&](uint32_t j) { return tasks[j].chunk0 <= c; }, &s_tmp);
        const FTask t = tasks[ti];
        const uint64_t line0 = (t.e0 >> ZC_LINE_SHIFT) + (c - t.chunk0) * FSTREAM_LINES;
        const uint64_t ce0 = max(t.e0, line0 << ZC_LINE_SHIFT);
        const uint64_t ce1 = min(t.e1, (line0 + FSTREAM_LINES) << ZC_LINE_SHIFT);
        const uint32_t cnt = (uint32_t)(ce1 - ce0);  // edges of the chunk, <= MAXE
        // the transfer: every line of the chunk, loads in flight from here on
        uint32_t cv[UNROLL], wv[UNROLL];
#pragma unroll
        for (int r = 0; r < UNROLL; r++) {
            const uint64_t e = ((line0 + half + (uint64_t)LINE_HALVES * r) << ZC_LINE_SHIFT) + lane;
            cv[r] = 0;
            wv[r] = 0;
            if (e >= ce0 && e < ce1) {
                cv[r] = col[e];
                if (Op::weighted && pk.shift == 32) wv[r] = load_w(w, e, pk);
            }
        }
        // active vertices whose out-edge ranges meet [ce0, ce1): list entries [j0, j0 + nv)
        // (the list is in vertex order, so both range ends increase with j)
        uint32_t j0 = t.ja, nv = 0;
        if (t.ja < t.jb && off[list[t.ja] + 1] <= ce0)
            j0 = block_search_last(t.ja, t.jb, [&](uint32_t j) { return off[list[j] + 1] <= ce0; }, &s_tmp) + 1;
        if (j0 < t.jb && off[list[j0]] < ce1)
            nv = block_search_last(j0, t.jb, [&](uint32_t j) { return off[list[j]] < ce1; }, &s_tmp) + 1 - j0;
        if (nv > 0) {  // uniform across the workgroup
            for (uint32_t q = threadIdx.x; q < cnt; q += LINE_THREADS) s_owner[q] = 0;
            __syncthreads();
            for (uint32_t k = threadIdx.x; k < nv; k += LINE_THREADS) {
                const uint32_t v = list[j0 + k];
                const uint64_t vs = off[v], ve = off[v + 1];
                const uint32_t rs = vs > ce0 ? (uint32_t)(vs - ce0) : 0u;
                s_s[k] = (uint16_t)rs;
                s_e[k] = (uint16_t)((ve < ce1 ? ve : ce1) - ce0);
                s_val[k] = op.src(v);
                if (k) s_owner[rs] = (uint16_t)k;  // later vertices start inside the chunk
            }
            __syncthreads();
            block_prefix_max_u16<8>(s_owner, cnt, s_wave);
            auto edge = [&](int r, uint32_t& val) {
                const uint64_t e = ((line0 + half + (uint64_t)LINE_HALVES * r) << ZC_LINE_SHIFT) + lane;
                val = 0;
                if (Op::weighted) wv[r] = pk_w(cv[r], wv[r], pk);
                cv[r] = pk_v(cv[r], pk);
                if (e < ce0 || e >= ce1) return false;
                const uint32_t q = (uint32_t)(e - ce0);
                const uint32_t k = s_owner[q];
                val = s_val[k];
                return q >= s_s[k] && q < s_e[k];
            };
            // The thread's edges are collected and then pushed; batched SSSP takes one edge at a
            // time through its wave form (OpMSssp<1>), since the pushes beside it already fill
            // the memory system: 64 lanes of 2^20 vertices at 25% resident, uniform 16M / R-MAT
            // 16M edges 50.9 / 20.2 ms, four at a time 51.6 / 20.8; found and pushed edge by edge
            // 54.9 / 21.9 and 55.6 / 22.2.  PageRank's adds alone are issued edge by edge:
            // collected they went out in bursts and cost 2% beside the pieces (R-MAT 28 under
            // 8 GB: 3,740 ms, 3,660 edge by edge).
            if constexpr (!std::is_same<Op, OpPr>::value) {
                bool ok[UNROLL];
                uint32_t val[UNROLL];
#pragma unroll
                for (int r = 0; r < UNROLL; r++) ok[r] = edge(r, val[r]);
                push_batch<UNROLL>(op, ok, val, cv, wv);
            } else {
#pragma unroll
                for (int r = 0; r < UNROLL; r++) {
                    uint32_t val;
                    if (edge(r, val)) op.push(val, cv[r], wv[r]);
                }
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ probes
__global__ __launch_bounds__(256) void k_zc_probe_lines(const uint32_t* __restrict__ src, uint64_t nlines,
                                                        uint32_t wpl, uint32_t* __restrict__ sink) {
    const uint32_t lane = threadIdx.x & 31;
    const uint64_t half = (blockIdx.x * (uint64_t)blockDim.x + threadIdx.x) >> 5;
    const uint64_t halves = ((uint64_t)gridDim.x * blockDim.x) >> 5;
    uint32_t acc = 0;
    for (uint64_t line = half; line < nlines; line += halves)
        if (lane < wpl) acc += src[(line << 5) + lane];
    if (acc == 0x9E3779B9u) sink[0] = acc;  // keeps the loads; practically never true
}

__global__ __launch_bounds__(256) void k_zc_probe_stream(const uint4* __restrict__ src, uint64_t n16,
                                                         uint32_t* __restrict__ sink) {
    uint32_t acc = 0;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n16;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint4 v = src[i];
        acc += v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x9E3779B9u) sink[0] = acc;
}

__global__ __launch_bounds__(256) void k_copy_probe(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                    uint64_t n16) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n16;
         i += (uint64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

inline unsigned grid_for(uint64_t items, unsigned per_block, unsigned cap) {
    uint64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    return (unsigned)(g < cap ? g : cap);
}

constexpr unsigned GRID_CAP = 1u << 16;

}  // namespace

hipError_t launch_init(const AlgoState& s, uint64_t n, uint32_t source, float pr_x0, float* pr_x, uint32_t* cur,
                       uint32_t nwords, hipStream_t st) {
    k_init<<<grid_for(n > nwords ? n : nwords, 256, 8192), 256, 0, st>>>(s, n, source, pr_x0, pr_x, cur, nwords);
    return hipGetLastError();
}

hipError_t launch_init_lanes(const AlgoState& s, const LaneSources& src, uint32_t* cur_union, uint32_t nwords,
                             hipStream_t st) {
    k_init_lanes<<<grid_for(s.n << s.lshift, 256, 16384), 256, 0, st>>>(s, src, cur_union, nwords);
    return hipGetLastError();
}

hipError_t launch_settle_lanes(const AlgoState& s, uint32_t nwords, hipStream_t st) {
    if (!s.n) return hipSuccess;
    if (!s.mvisited || !s.lval || s.lshift > 6) return hipErrorInvalidValue;
    k_settle_lanes<<<grid_for(s.n, 256, 4096), 256, 0, st>>>(s, nwords);
    return hipGetLastError();
}

hipError_t launch_extract_lanes(const uint32_t* vals, uint64_t n, uint32_t lshift, const LaneSet& set, bool sub_base,
                                const uint32_t* rank, const LaneRows& out, bool to_host, hipStream_t st) {
    const uint32_t nsel = (uint32_t)__builtin_popcountll(set.mask);
    if (!n || !nsel || lshift > 6 || (set.mask >> 1 >> ((1u << lshift) - 1))) return n && nsel ? hipErrorInvalidValue : hipSuccess;
    const size_t row = sizeof(uint32_t) * ((1u << lshift) + 1);
    if (!to_host || n < EX_WIDE)
        k_extract_lanes<64><<<grid_for(n, 64, 4096), 256, 64 * row, st>>>(vals, n, lshift, set, nsel, sub_base, rank, out);
    else
        k_extract_lanes<256><<<grid_for(n, 256, 4096), 256, 256 * row, st>>>(vals, n, lshift, set, nsel, sub_base, rank,
                                                                             out);
    return hipGetLastError();
}

hipError_t launch_loaded_frontier(uint32_t npart, const uint32_t* pv, const uint8_t* mode, uint32_t mode_mask,
                                  const uint32_t* next, uint32_t* cur2, uint32_t nwords, hipStream_t st) {
    hipError_t e = launch_fill_u32(cur2, nwords, 0u, st);
    if (e != hipSuccess || !npart) return e;
    k_loaded_frontier<<<npart < GRID_CAP ? npart : GRID_CAP, 256, 0, st>>>(npart, pv, mode, mode_mask, next, cur2);
    return hipGetLastError();
}

hipError_t launch_dpr_fold(uint32_t npart, const uint32_t* pv, uint64_t n, float* acc, uint32_t copies, float* delta,
                           double* psum, hipStream_t st) {
    if (!npart) return hipSuccess;
    if (copies < 1 || copies > ACC_COPIES) return hipErrorInvalidValue;
    k_dpr_fold<<<npart < GRID_CAP ? npart : GRID_CAP, 256, 0, st>>>(npart, pv, n, acc, copies, delta, psum);
    return hipGetLastError();
}

hipError_t launch_dpr_activate(uint32_t npart, const uint32_t* pv, const uint64_t* off, const uint8_t* sched,
                               float* delta, float* x, float* contrib, uint32_t* cur, uint32_t nwords, float damping,
                               hipStream_t st) {
    hipError_t e = launch_fill_u32(cur, nwords, 0u, st);
    if (e != hipSuccess || !npart) return e;
    k_dpr_activate<<<npart < GRID_CAP ? npart : GRID_CAP, 256, 0, st>>>(npart, pv, off, sched, delta, x, contrib,
                                                                         cur, damping);
    return hipGetLastError();
}

hipError_t launch_dpr_finish(uint64_t n, float* x, const float* delta, hipStream_t st) {
    if (!n) return hipSuccess;
    k_dpr_finish<<<grid_for(n, 256, 8192), 256, 0, st>>>(n, x, delta);
    return hipGetLastError();
}

hipError_t launch_gather_u32(const uint32_t* src, const uint32_t* rank, uint64_t n, uint32_t* dst, hipStream_t st) {
    if (!n) return hipSuccess;
    k_gather_u32<<<grid_for(n, 256, 8192), 256, 0, st>>>(src, rank, n, dst);
    return hipGetLastError();
}

hipError_t launch_cc_relabel(const uint32_t* lab, const uint32_t* order, const uint32_t* rank, uint64_t n,
                             uint32_t* minold, uint32_t* dst, hipStream_t st) {
    if (!n) return hipSuccess;
    hipError_t e = launch_fill_u32(minold, n, UNREACHED, st);
    if (e != hipSuccess) return e;
    k_cc_min_old<<<grid_for(n, 256, 8192), 256, 0, st>>>(lab, order, n, minold);
    k_cc_canon<<<grid_for(n, 256, 8192), 256, 0, st>>>(lab, minold, rank, n, dst);
    return hipGetLastError();
}

hipError_t launch_cc_link(uint64_t n, const uint64_t* off, const uint32_t* col, uint32_t vmask, uint32_t r, uint32_t* par,
                          hipStream_t st) {
    if (!n) return hipSuccess;
    k_cc_link<<<grid_for(n, 256, 16384), 256, 0, st>>>(n, off, col, vmask, r, par);
    return hipGetLastError();
}

hipError_t launch_cc_compress(uint64_t n, uint32_t* par, hipStream_t st) {
    if (!n) return hipSuccess;
    k_cc_compress<<<grid_for(n, 256, 16384), 256, 0, st>>>(n, par);
    return hipGetLastError();
}

hipError_t launch_cc_rest(uint64_t n, const uint64_t* off, uint32_t done, const uint32_t* par, uint32_t* giant,
                          uint32_t* rest, uint32_t nwords, hipStream_t st) {
    if (!n) return hipSuccess;
    k_cc_giant<<<1, 1024, 0, st>>>(n, par, giant);
    k_cc_rest<<<grid_for(n, 256, 16384), 256, 0, st>>>(n, off, done, par, giant, rest, nwords);
    return hipGetLastError();
}

hipError_t launch_far_min(const uint32_t* far, const uint32_t* dist, uint32_t nwords, uint32_t* out, hipStream_t st) {
    if (!nwords) return hipSuccess;
    k_far_min<<<grid_for(nwords, 256, 8192), 256, 0, st>>>(far, dist, nwords, out);
    return hipGetLastError();
}

hipError_t launch_far_move(uint32_t* far, const uint32_t* dist, uint32_t* cur, uint32_t nwords, uint32_t bound,
                           hipStream_t st) {
    if (!nwords) return hipSuccess;
    k_far_move<<<grid_for(nwords, 256, 8192), 256, 0, st>>>(far, dist, cur, nwords, bound);
    return hipGetLastError();
}

hipError_t launch_sssp_ovf_check(const uint64_t* off, const uint32_t* col, const Pack& pk, const uint32_t* dist,
                                 uint32_t lshift, uint64_t mask, uint64_t n, unsigned long long* out, hipStream_t st) {
    if (!n || !mask || lshift > 6) return lshift > 6 ? hipErrorInvalidValue : hipSuccess;
    k_sssp_ovf_check<<<grid_for(n, 4, 16384), 256, 0, st>>>(off, col, pk, dist, lshift, mask, n, out);
    return hipGetLastError();
}

hipError_t launch_admit_lanes(const AlgoState& s, const LaneSet& set, uint32_t* cur, hipStream_t st) {
    if (!set.mask) return hipSuccess;
    k_admit_lanes<<<1, MAX_LANES, 0, st>>>(s, set, cur);
    return hipGetLastError();
}

hipError_t launch_reset_lanes(const AlgoState& s, uint64_t mask, hipStream_t st) {
    if (!mask || !s.n) return hipSuccess;
    k_reset_lanes<<<grid_for(s.n << s.lshift, 256, 16384), 256, 0, st>>>(s, mask);
    return hipGetLastError();
}

// Vertices per window: 64, fewer on small graphs so that there are PPR_WAVES of them, but whole accesses
// of 64 cells (64 lanes of 70K vertices, whole call: 2.52 ms in windows of 64, 2.25 so; 4,096 or 65,536
// waves 2.27 and 2.32, of 2^18 vertices 5.25 and 5.17 against 5.14).
constexpr uint64_t PPR_WAVES = 16384;
static uint32_t ppr_rows(const AlgoState& s) {
    uint32_t rows = 64;
    while (rows > (64u >> s.lshift) && s.n / rows < PPR_WAVES) rows /= 2;
    return rows;
}

hipError_t launch_ppr_prepare(const AlgoState& s, const uint64_t* off, hipStream_t st) {
    if (!s.n) return hipSuccess;
    const uint32_t rows = ppr_rows(s);
    k_ppr_prepare<<<grid_for(s.n, 4 * rows, 16384), 256, 0, st>>>(s, rows, off);
    return hipGetLastError();
}

hipError_t launch_ppr_apply_next(const AlgoState& s, const uint64_t* off, const LaneSet& set, float damping,
                                 float restart, hipStream_t st) {
    if (!s.n) return hipSuccess;
    const uint32_t rows = ppr_rows(s);
    k_ppr_apply_next<<<grid_for(s.n, 4 * rows, 16384), 256, 0, st>>>(s, rows, off, set, damping, restart);
    return hipGetLastError();
}

hipError_t launch_ppr_apply(const AlgoState& s, float damping, hipStream_t st) {
    if (!s.n) return hipSuccess;
    const uint32_t rows = ppr_rows(s);
    k_ppr_apply<<<grid_for(s.n, 4 * rows, 16384), 256, 0, st>>>(s, rows, damping);
    return hipGetLastError();
}

hipError_t launch_in_lists(const uint64_t* off, const uint32_t* col, const uint32_t* w, const Pack& pk, uint64_t m,
                           uint64_t n, uint32_t* cnt, uint64_t* tot, uint64_t* toff, uint32_t* soff, uint32_t* seg_v,
                           uint32_t* tsrc, uint32_t* tdst, uint32_t* tw, hipStream_t st) {
    if (!n || !m) return hipErrorInvalidValue;
    const uint64_t tiles = in_tiles(n);
    hipError_t e = launch_fill_u32(cnt, n, 0u, st);
    if (e != hipSuccess) return e;
    k_in_count<<<grid_for(m, 256, 16384), 256, 0, st>>>(col, pk.mask, m, n, cnt);
    k_in_tot<<<(unsigned)tiles, 256, 0, st>>>(cnt, n, tot);
    k_in_base<<<1, 64, 0, st>>>(tiles, tot, n, toff, soff);
    k_in_write<<<(unsigned)tiles, 256, 0, st>>>(cnt, n, tot, toff, soff, seg_v);
    k_in_scatter<<<grid_for(m, 256, 16384), 256, 0, st>>>(off, col, w, pk, m, n, toff, cnt, tsrc, tdst, tw);
    return hipGetLastError();
}

template <class P>
static hipError_t pull_op(const AlgoState& s, const InLists& in, hipStream_t st) {
    if (!in.nseg) return hipSuccess;
    uint32_t run = IN_RUN_MAX;
    while (run > std::max(64u, 2u << s.lshift) && ((in.m / run) << s.lshift) / 64 < PULL_WAVES) run /= 2;
    const unsigned gr = grid_for((in.m + run - 1) / run, 256u >> s.lshift, GRID_CAP);
    switch (s.lshift) {
    case 4: k_pull_runs<4, P><<<gr, 256, 0, st>>>(s, in, run); break;
    case 5: k_pull_runs<5, P><<<gr, 256, 0, st>>>(s, in, run); break;
    case 6: k_pull_runs<6, P><<<gr, 256, 0, st>>>(s, in, run); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_pull(const AlgoState& s, const InLists& in, hipStream_t st) {
    if (s.algo == ALGO_MPPR && s.lshift < 4) {
        if (!in.nseg) return hipSuccess;
        const unsigned g = grid_for(in.nseg, 16, GRID_CAP);
        if (s.lshift == 0) k_pull_segs<0><<<g, 256, 0, st>>>(s, in);
        if (s.lshift == 1) k_pull_segs<1><<<g, 256, 0, st>>>(s, in);
        if (s.lshift == 2) k_pull_segs<2><<<g, 256, 0, st>>>(s, in);
        if (s.lshift == 3) k_pull_segs<3><<<g, 256, 0, st>>>(s, in);
        return hipGetLastError();
    }
    if (s.algo == ALGO_MPPR) return pull_op<PullPpr>(s, in, st);
    if (s.algo == ALGO_MSSSP && in.tw) return pull_op<PullSssp>(s, in, st);
    return hipErrorInvalidValue;
}

hipError_t launch_ppr_restart(const AlgoState& s, const LaneSet& set, float restart, hipStream_t st) {
    if (!set.mask) return hipSuccess;
    k_ppr_restart<<<1, MAX_LANES, 0, st>>>(s, set, restart);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t count, uint32_t value, hipStream_t st) {
    if (!count) return hipSuccess;
    k_fill_u32<<<grid_for(count, 256, 8192), 256, 0, st>>>(p, count, value);
    return hipGetLastError();
}

hipError_t launch_stats_select(uint32_t npart, const Units& un, const uint32_t* pv, const uint64_t* off,
                               const uint32_t* cur, uint32_t* clear, uint32_t nwords, const uint64_t* mcur,
                               unsigned long long* lanes, const SelParams& sp, uint8_t* mode, uint32_t* nA,
                               uint32_t* nF, uint64_t* Ea, uint64_t* K, const LevelScan& ls, hipStream_t st) {
    if (!npart) return hipSuccess;
    const unsigned g = grid_for(un.count, 4, GRID_CAP);
    if (ls.cur)
        k_unit_stats<true><<<g, 256, 0, st>>>(un, pv, off, cur, clear, nwords, mcur, lanes, sp, mode, nA, nF, Ea, K, ls);
    else
        k_unit_stats<false><<<g, 256, 0, st>>>(un, pv, off, cur, clear, nwords, mcur, lanes, sp, mode, nA, nF, Ea, K, ls);
    if (un.multis)
        k_part_combine<<<(un.multis + 3) / 4, 256, 0, st>>>(un, pv, off, sp, mode, nA, nF, Ea, K);
    return hipGetLastError();
}

hipError_t launch_scan(uint32_t npart, const uint8_t* mode, const uint32_t* nA, const uint32_t* nF,
                       const uint64_t* Ea, const uint64_t* K, uint32_t* lbase, uint64_t* wbase, Header* hdr,
                       uint64_t* wpre, uint64_t* scratch, const ScanExtra& x, hipStream_t st) {
    const uint32_t ntiles = scan_tiles(npart);
    uint64_t* tile_tot = scratch;
    uint64_t* tile_base = scratch + (uint64_t)ntiles * SCAN_NV;
    if (ntiles) k_scan_tot<<<ntiles, SCAN_THREADS, 0, st>>>(npart, mode, nA, nF, Ea, K, tile_tot);
    k_scan_base<<<1, 64, 0, st>>>(ntiles, tile_tot, tile_base, hdr, wpre, x);
    if (ntiles) k_scan_write<<<ntiles, SCAN_THREADS, 0, st>>>(npart, mode, nA, Ea, K, tile_base, lbase, wbase);
    return hipGetLastError();
}

hipError_t launch_scan_one(uint32_t npart, const uint8_t* mode, const uint32_t* nA, const uint32_t* nF,
                           const uint64_t* Ea, const uint64_t* K, uint32_t* lbase, uint64_t* wbase, uint64_t* wpre,
                           const ScanExtra& x, const ScanHost& host, hipStream_t st) {
    if (npart > SCAN_ONE_MAX) return hipErrorInvalidValue;
    if (npart <= 1024)
        k_scan_one<1><<<1, 1024, 0, st>>>(npart, mode, nA, nF, Ea, K, lbase, wbase, wpre, x, host);
    else if (npart <= 4096)
        k_scan_one<4><<<1, 1024, 0, st>>>(npart, mode, nA, nF, Ea, K, lbase, wbase, wpre, x, host);
    else if (npart <= 8192)
        k_scan_one<8><<<1, 1024, 0, st>>>(npart, mode, nA, nF, Ea, K, lbase, wbase, wpre, x, host);
    else
        k_scan_one<16><<<1, 1024, 0, st>>>(npart, mode, nA, nF, Ea, K, lbase, wbase, wpre, x, host);
    return hipGetLastError();
}

hipError_t launch_select_small(uint32_t npart, const Units& un, const uint32_t* pv, const uint64_t* off,
                               const uint32_t* cur, uint32_t* clear, uint32_t nwords, const uint64_t* mcur,
                               const SelParams& sp, uint8_t* mode, uint32_t* list, uint64_t* wpre, uint32_t* tile_e,
                               uint32_t* tile_l, bool lists, const ScanExtra& x, const ScanHost& host,
                               hipStream_t st) {
    static_assert(SMALL_UNITS <= 64, "one wave lays the partitions out");
    if (!npart || un.count > SMALL_UNITS) return hipErrorInvalidValue;
    k_select_small<<<1, 1024, 0, st>>>(npart, un, pv, off, cur, clear, nwords, mcur, sp, mode, list, wpre, tile_e,
                                       tile_l, lists, x, host);
    return hipGetLastError();
}

hipError_t launch_build_lists(const Units& un, const uint32_t* pv, const uint64_t* off, const uint32_t* cur,
                              const uint8_t* mode, const uint32_t* lbase, const uint64_t* wbase, uint32_t* list,
                              uint64_t* wpre, uint32_t* tile_e, uint32_t* tile_l, hipStream_t st) {
    if (!un.count) return hipSuccess;
    k_build_lists<<<grid_for(un.count, 4, GRID_CAP), 256, 0, st>>>(un, pv, off, cur, mode, lbase, wbase, list, wpre,
                                                                   tile_e, tile_l);
    return hipGetLastError();
}

hipError_t launch_fill2_u32(uint32_t* p, uint64_t np, uint32_t* q, uint64_t nq, uint32_t value, hipStream_t st) {
    if (!(np + nq)) return hipSuccess;
    k_fill2_u32<<<grid_for(np + nq, 1024, 8192), 256, 0, st>>>(p, np, q, nq, value);
    return hipGetLastError();
}

template <class Op>
static hipError_t push_edges_op(const Op& op, const uint32_t* list, const uint64_t* wpre, const uint32_t* tile, uint32_t ja, uint32_t jb,
                                uint64_t lo, uint64_t hi, const uint64_t* off, const uint32_t* col,
                                const uint32_t* w, uint64_t shift, bool compacted, const Pack& pk, hipStream_t st,
                                unsigned cap) {
    const unsigned g = grid_for(((hi - 1) >> EDGE_TILE_SHIFT) - (lo >> EDGE_TILE_SHIFT) + 1, 1, cap ? cap : GRID_CAP);
    if (compacted)
        k_push_edges<Op, true><<<g, EDGE_THREADS, 0, st>>>(list, wpre, tile, ja, jb, lo, hi, off, col, w, shift, op, pk);
    else
        k_push_edges<Op, false><<<g, EDGE_THREADS, 0, st>>>(list, wpre, tile, ja, jb, lo, hi, off, col, w, shift, op, pk);
    return hipGetLastError();
}

hipError_t launch_push_edges(const AlgoState& s, const uint32_t* list, const uint64_t* wpre, const uint32_t* tile, uint32_t ja,
                             uint32_t jb, uint64_t item_lo, uint64_t item_hi, const uint64_t* off,
                             const uint32_t* col, const uint32_t* w, uint64_t shift, bool compacted,
                             hipStream_t st, unsigned cap) {
    if (item_hi <= item_lo || jb <= ja) return hipSuccess;
    switch (s.algo) {
    case ALGO_BFS:
        return push_edges_op(OpBfs{s.visited, s.next, s.val, s.level_next}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, shift, compacted, s.pk, st, cap);
    case ALGO_BFS_WIDE:
        return push_edges_op(OpBfsWide{s.visited, s.val, s.level_next}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, shift, compacted, s.pk, st, cap);
    case ALGO_SSSP:
        return push_edges_op(OpSssp{s.val, s.next, s.overflow, s.far, s.bound}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w,
                             shift, compacted, s.pk, st, cap);
    case ALGO_SSSP_WIDE:
        return push_edges_op(OpSsspWide{{s.val, s.next, s.overflow, s.far, s.bound}, s.marks, (uint8_t)s.tag}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, shift, compacted, s.pk, st, cap);
    case ALGO_CC_WIDE:
        return push_edges_op(OpCcWide{{s.val, s.next}, s.marks, (uint8_t)s.tag}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, shift, compacted, s.pk, st, cap);
    case ALGO_CC:
        return push_edges_op(OpCc{s.val, s.next}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, shift,
                             compacted, s.pk, st, cap);
    case ALGO_CC_LINK:
        return push_edges_op(OpLink{s.val}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, shift, compacted,
                             s.pk, st, cap);
    case ALGO_BFS_RELAX:
        return push_edges_op(OpBfsRelax{s.val, s.next}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, shift,
                             compacted, s.pk, st, cap);
    case ALGO_MBFS_WIDE:
        return push_edges_op(OpMBfsWide(s), list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, shift,
                             compacted, s.pk, st, cap);
    case ALGO_MBFS:
        return push_edges_op(OpMBfs{s.mcur, s.mnext, s.mvisited, s.lval, s.next, s.level_next, s.lshift}, list, wpre, tile, ja, jb,
                             item_lo, item_hi, off, col, w, shift, compacted, s.pk, st, cap);
    case ALGO_MSSSP:
        return push_edges_op(OpMSssp<4>{s.mcur, s.mnext, s.lval, s.next, s.overflow, s.lshift}, list, wpre, tile, ja, jb, item_lo,
                             item_hi, off, col, w, shift, compacted, s.pk, st, cap);
    case ALGO_MPPR:
        return push_edges_op(OpMPpr{s.mcur, s.mnext, s.lx, s.lacc, s.next, s.lshift}, list, wpre, tile, ja, jb, item_lo,
                             item_hi, off, col, w, shift, compacted, s.pk, st, cap);
    default:
        return push_edges_op(OpPr{s.acc, acc_slots(s.n), s.contrib, s.acc_copies - 1}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, shift,
                             compacted, s.pk, st, cap);
    }
}

template <class Op>
static hipError_t push_lines_op(const Op& op, const uint32_t* list, const uint64_t* wpre, const uint32_t* tile, uint32_t ja, uint32_t jb,
                                uint64_t lo, uint64_t hi, const uint64_t* off, const uint32_t* col,
                                const uint32_t* w, unsigned long long* distinct, const Pack& pk, hipStream_t st,
                                unsigned cap = GRID_CAP) {
    const unsigned g = grid_for(((hi - 1) >> LINE_TILE_SHIFT) - (lo >> LINE_TILE_SHIFT) + 1, 1, cap ? cap : GRID_CAP);
    k_push_lines<Op><<<g, LINE_THREADS, 0, st>>>(list, wpre, tile, ja, jb, lo, hi, off, col, w, op, distinct, pk);
    return hipGetLastError();
}

hipError_t launch_push_lines(const AlgoState& s, const uint32_t* list, const uint64_t* wpre, const uint32_t* tile, uint32_t ja,
                             uint32_t jb, uint64_t item_lo, uint64_t item_hi, const uint64_t* off,
                             const uint32_t* col, const uint32_t* w, unsigned long long* distinct, hipStream_t st) {
    if (item_hi <= item_lo || jb <= ja) return hipSuccess;
    switch (s.algo) {
    case ALGO_BFS:
        return push_lines_op(OpBfs{s.visited, s.next, s.val, s.level_next}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, distinct, s.pk, st);
    case ALGO_BFS_WIDE:
        return push_lines_op(OpBfsWide{s.visited, s.val, s.level_next}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, distinct, s.pk, st);
    case ALGO_SSSP:
        return push_lines_op(OpSssp{s.val, s.next, s.overflow, s.far, s.bound}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, distinct, s.pk, st);
    case ALGO_SSSP_WIDE:
        return push_lines_op(OpSsspWide{{s.val, s.next, s.overflow, s.far, s.bound}, s.marks, (uint8_t)s.tag}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, distinct, s.pk, st);
    case ALGO_CC_WIDE:
        return push_lines_op(OpCcWide{{s.val, s.next}, s.marks, (uint8_t)s.tag}, list, wpre, tile, ja, jb, item_lo, item_hi,
                             off, col, w, distinct, s.pk, st);
    case ALGO_CC:
        return push_lines_op(OpCc{s.val, s.next}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, distinct, s.pk, st);
    case ALGO_BFS_RELAX:
        return push_lines_op(OpBfsRelax{s.val, s.next}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, distinct, s.pk, st);
    case ALGO_MBFS_WIDE:
        return push_lines_op(OpMBfsWide(s), list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w, distinct,
                             s.pk, st);
    case ALGO_MBFS:
        return push_lines_op(OpMBfs{s.mcur, s.mnext, s.mvisited, s.lval, s.next, s.level_next, s.lshift}, list, wpre, tile, ja, jb,
                             item_lo, item_hi, off, col, w, distinct, s.pk, st);
    case ALGO_MSSSP:
        return push_lines_op(OpMSssp<4>{s.mcur, s.mnext, s.lval, s.next, s.overflow, s.lshift}, list, wpre, tile, ja, jb, item_lo,
                             item_hi, off, col, w, distinct, s.pk, st);
    case ALGO_MPPR:
        return push_lines_op(OpMPpr{s.mcur, s.mnext, s.lx, s.lacc, s.next, s.lshift}, list, wpre, tile, ja, jb, item_lo,
                             item_hi, off, col, w, distinct, s.pk, st);
    default:
        return push_lines_op(OpPr{s.acc, acc_slots(s.n), s.contrib, s.acc_copies - 1}, list, wpre, tile, ja, jb, item_lo, item_hi, off, col, w,
                             distinct, s.pk, st, s.link_grid);
    }
}

hipError_t launch_pr_prepare(uint64_t n, const uint64_t* off, const float* x, float* contrib, float* acc,
                             uint32_t copies, hipStream_t st) {
    if (!n) return hipSuccess;
    if (copies < 1 || copies > ACC_COPIES + 1) return hipErrorInvalidValue;
    k_pr_prepare<<<grid_for(acc_slots(n), 256, 8192), 256, 0, st>>>(n, off, x, contrib, acc, copies);
    return hipGetLastError();
}

hipError_t launch_pb_hist(const uint32_t* pv, uint32_t vmask, uint64_t cnt, uint32_t fshift, uint32_t nfine,
                          uint32_t* hist, uint32_t* err, hipStream_t st) {
    if (!cnt) return hipSuccess;
    if (nfine == 0 || nfine > PB_MAX_FINE) return hipErrorInvalidValue;
    const unsigned g = (unsigned)std::min<uint64_t>(256, (cnt + 4095) / 4096);
    k_pb_hist<<<g, PB_THREADS, 0, st>>>(pv, vmask, cnt, fshift, nfine, hist, err);
    return hipGetLastError();
}

hipError_t launch_pb_plan(const uint32_t* hist, uint32_t nfine, uint32_t seg, uint32_t* foff, uint32_t* segs,
                          uint32_t* nsegs, hipStream_t st) {
    if (nfine == 0 || nfine > PB_MAX_FINE || seg == 0) return hipErrorInvalidValue;
    k_pb_plan<<<1, PB_PLAN_THREADS, 0, st>>>(hist, nfine, seg, foff, segs, nsegs);
    return hipGetLastError();
}

hipError_t launch_pb_scatter(const uint32_t* in_v, const float* in_c, uint64_t cnt, uint32_t kshift, uint32_t stride,
                             uint32_t nfine, const uint32_t* foff, uint32_t* cursor, uint32_t* out_v, float* out_c,
                             uint32_t* err, hipStream_t st) {
    if (!cnt) return hipSuccess;
    if (nfine == 0 || nfine > PB_MAX_FINE || (stride != 1 && stride != PB_FINE_PER_COARSE)) return hipErrorInvalidValue;
    k_pb_scatter<<<grid_for(cnt, PB_TILE, 2048), PB_THREADS, 0, st>>>(in_v, in_c, cnt, kshift, stride, nfine, foff,
                                                                      cursor, out_v, out_c, err);
    return hipGetLastError();
}

hipError_t launch_pb_tiles(const uint64_t* wpre, uint32_t ja, uint32_t jb, uint64_t wa, uint64_t cnt, uint32_t* tj,
                           hipStream_t st) {
    if (!cnt) return hipSuccess;
    if (jb <= ja) return hipErrorInvalidValue;
    const uint64_t ntiles = (cnt + PB_EXP_TILE - 1) / PB_EXP_TILE;
    k_pb_tiles<<<grid_for(ntiles, 256, 1024), 256, 0, st>>>(wpre, ja, jb, wa, cnt, tj);
    return hipGetLastError();
}

hipError_t launch_pb_expand(const uint32_t* list, const uint64_t* wpre, uint32_t jb, uint64_t wa, uint64_t cnt,
                            const uint32_t* tj, const float* contrib, float* pc, hipStream_t st) {
    if (!cnt) return hipSuccess;
    const uint64_t ntiles = (cnt + PB_EXP_TILE - 1) / PB_EXP_TILE;
    const unsigned g = (unsigned)std::min<uint64_t>(ntiles, 4096);
    if (contrib)
        k_pb_expand<false><<<g, 256, 0, st>>>(list, wpre, jb, wa, cnt, tj, contrib, pc);
    else
        k_pb_expand<true><<<g, 256, 0, st>>>(list, wpre, jb, wa, cnt, tj, nullptr, pc);
    return hipGetLastError();
}

hipError_t launch_pg_pack(const uint32_t* v, uint64_t cnt, uint32_t shift, uint64_t n, uint16_t* slot, uint32_t* err,
                          hipStream_t st) {
    if (!cnt) return hipSuccess;
    if (shift < PG_MIN_SHIFT || shift > PG_MAX_SHIFT) return hipErrorInvalidValue;
    k_pg_pack<<<grid_for(cnt, 256, 8192), 256, 0, st>>>(v, cnt, shift, n, slot, err);
    return hipGetLastError();
}

hipError_t launch_pg_gather(const uint32_t* src, const uint16_t* slot, uint64_t e0, const uint32_t* foff,
                            const uint32_t* segs, uint32_t nsegs, uint32_t seg, uint32_t shift, uint64_t n,
                            const float* contrib, float* acc, hipStream_t st) {
    if (!nsegs) return hipSuccess;
    // sums of 32 KB and more leave room for few workgroups per CU: larger ones
    if (seg == 0 || shift < PG_MIN_SHIFT || shift > PG_MAX_SHIFT) return hipErrorInvalidValue;
    k_pg_gather<<<nsegs, shift >= 12 ? 512 : 256, sizeof(double) << shift, st>>>(src, slot, e0, foff, segs, seg, shift, n, contrib,
                                                                   acc);
    return hipGetLastError();
}

hipError_t launch_rg_build(const uint64_t* off, const uint32_t* col, uint32_t vmask, uint64_t m, uint64_t nv, uint64_t n,
                           uint32_t shift, uint32_t nfine, uint32_t blocks, uint32_t seg, uint32_t* cnt, uint64_t* tot,
                           uint32_t* hist, uint64_t* start, uint32_t* foff, uint32_t* segs, uint32_t* nsegs,
                           uint32_t* pairs, uint32_t* err, hipStream_t st) {
    if (!m || !nv || !blocks || m > UINT32_MAX || shift < PG_MIN_SHIFT || shift > PG_MAX_SHIFT) return hipErrorInvalidValue;
    const uint64_t keys = (uint64_t)nfine * blocks, tiles = in_tiles(keys);
    hipError_t e = launch_fill_u32(cnt, keys, 0u, st);
    if (e != hipSuccess) return e;
    const unsigned g = grid_for(m, RG_CHUNK, 8192);
    const size_t lds = (size_t)nfine * 4;
    if (nfine > RG_MAX_FINE) return hipErrorInvalidValue;
    k_rg_sort<false><<<g, 512, lds, st>>>(off, col, vmask, m, nv, n, shift, nfine, blocks, nullptr, cnt, nullptr, err);
    k_in_tot<<<(unsigned)tiles, 256, 0, st>>>(cnt, keys, tot);
    k_in_base<<<1, 64, 0, st>>>(tiles, tot, keys, start, nullptr);
    k_in_write<<<(unsigned)tiles, 256, 0, st>>>(cnt, keys, tot, start, nullptr, nullptr);
    k_rg_sort<true><<<g, 512, lds, st>>>(off, col, vmask, m, nv, n, shift, nfine, blocks, start, cnt, pairs, err);
    k_rg_hist<<<(nfine + 255) / 256, 256, 0, st>>>(start, nfine, blocks, hist);
    return launch_pb_plan(hist, nfine, seg, foff, segs, nsegs, st);
}

hipError_t launch_rg_gather(const uint32_t* pairs, const uint64_t* start, uint32_t blocks, const uint32_t* foff,
                            const uint32_t* segs, uint32_t nsegs, uint32_t seg, uint32_t shift, uint64_t n,
                            const float* contrib, float* acc, hipStream_t st) {
    if (!nsegs) return hipSuccess;
    const size_t lds = (sizeof(double) << shift) + 4 * ((size_t)blocks + 1);
    if (seg == 0 || shift < PG_MIN_SHIFT || lds > RG_MAX_LDS) return hipErrorInvalidValue;
    k_rg_gather<<<nsegs, 256, lds, st>>>(pairs, start, blocks, foff, segs, seg, shift, n, contrib, acc);
    return hipGetLastError();
}

hipError_t launch_pg_start(uint64_t n, const uint64_t* off, const float* x, float* contrib, float* acc,
                           hipStream_t st) {
    if (!n) return hipSuccess;
    k_pg_start<<<grid_for(n, 256, 8192), 256, 0, st>>>(n, off, x, contrib, acc);
    return hipGetLastError();
}

hipError_t launch_pg_apply(uint64_t n, const uint64_t* off, float* x, float* contrib, float* acc, float base,
                           float damping, const float* inv_n, float restart, bool last, hipStream_t st) {
    if (!n) return hipSuccess;
    if (last)
        k_pg_apply<true><<<grid_for(n, 256, 8192), 256, 0, st>>>(n, off, x, contrib, acc, base, damping, inv_n, restart);
    else
        k_pg_apply<false><<<grid_for(n, 256, 8192), 256, 0, st>>>(n, off, x, contrib, acc, base, damping, inv_n, restart);
    return hipGetLastError();
}

// Slices of the first sort pass: `wg` workgroups of `range` pairs (a multiple of PB_TILE).
void pb_slices(uint64_t cnt, uint32_t* wg, uint64_t* range) {
    const uint64_t tiles = (cnt + PB_TILE - 1) / PB_TILE;
    const uint64_t per = (tiles + PB_A_WG - 1) / PB_A_WG;
    *range = std::max<uint64_t>(per, 1) * PB_TILE;
    *wg = (uint32_t)std::max<uint64_t>(1, (cnt + *range - 1) / *range);
}

hipError_t launch_pb_plan_a(const uint32_t* pv, uint32_t vmask, uint64_t cnt, uint32_t kshift, uint32_t stride,
                            uint32_t nfine, const uint32_t* foff, uint32_t* offA, uint32_t* err, hipStream_t st) {
    if (!cnt) return hipSuccess;
    const uint32_t nkeys = (nfine + stride - 1) / stride;
    if (nfine == 0 || nfine > PB_MAX_FINE || nkeys > PB_LOCAL || (stride != 1 && stride != PB_FINE_PER_COARSE))
        return hipErrorInvalidValue;
    uint32_t wg;
    uint64_t range;
    pb_slices(cnt, &wg, &range);
    k_pb_count_a<<<wg, PB_THREADS, 0, st>>>(pv, vmask, cnt, range, kshift, nkeys, offA, err);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_pb_scan_a<<<nkeys, PB_A_WG, 0, st>>>(offA, wg, nkeys, stride, foff);
    return hipGetLastError();
}

hipError_t launch_pb_scatter_a(const uint32_t* in_v, uint32_t vmask, const float* in_c, uint64_t cnt,
                               uint32_t kshift, uint32_t stride, uint32_t nfine, const uint32_t* foff,
                               const uint32_t* offA, uint32_t* out_v, float* out_c, uint32_t* fcur, uint32_t* err,
                               hipStream_t st) {
    if (!cnt) return hipSuccess;
    const uint32_t nkeys = (nfine + stride - 1) / stride;
    if (nfine == 0 || nfine > PB_MAX_FINE || nkeys > PB_LOCAL || (stride != 1 && stride != PB_FINE_PER_COARSE))
        return hipErrorInvalidValue;
    uint32_t wg;
    uint64_t range;
    pb_slices(cnt, &wg, &range);
    k_pb_scatter_a<<<wg, PB_THREADS, 0, st>>>(in_v, vmask, in_c, cnt, range, kshift, stride, nfine, foff, offA, out_v,
                                              out_c, fcur, err);
    return hipGetLastError();
}

hipError_t launch_pb_accum(const uint32_t* pv, const float* pc, const uint32_t* foff, const uint32_t* segs,
                           const uint32_t* nsegs, uint32_t max_segs, uint32_t seg, uint64_t n, float* acc,
                           uint32_t* err, hipStream_t st) {
    if (!max_segs || !n) return hipSuccess;
    if (seg == 0) return hipErrorInvalidValue;
    k_pb_accum<<<max_segs, PB_ACC_THREADS, 0, st>>>(pv, pc, foff, segs, nsegs, seg, n, acc, err);
    return hipGetLastError();
}

template <class Op>
static hipError_t push_fstream_op(const Op& op, const FTask* tasks, uint32_t ntasks, uint64_t chunks,
                                  const uint32_t* list, const uint64_t* off, const uint32_t* col, const uint32_t* w,
                                  const Pack& pk, hipStream_t st, unsigned cap = GRID_CAP) {
    const unsigned c = cap ? cap : GRID_CAP;
    const unsigned g = (unsigned)(chunks < c ? chunks : c);
    k_push_fstream<Op><<<g, LINE_THREADS, 0, st>>>(tasks, ntasks, chunks, list, off, col, w, op, pk);
    return hipGetLastError();
}

hipError_t launch_push_fstream(const AlgoState& s, const FTask* tasks, uint32_t ntasks, uint64_t total_chunks,
                               const uint32_t* list, const uint64_t* off, const uint32_t* col, const uint32_t* w,
                               hipStream_t st) {
    if (!ntasks || !total_chunks) return hipSuccess;
    switch (s.algo) {
    case ALGO_BFS:
        return push_fstream_op(OpBfs{s.visited, s.next, s.val, s.level_next}, tasks, ntasks, total_chunks, list,
                               off, col, w, s.pk, st);
    case ALGO_BFS_WIDE:
        return push_fstream_op(OpBfsWide{s.visited, s.val, s.level_next}, tasks, ntasks, total_chunks, list, off, col, w,
                               s.pk, st);
    case ALGO_SSSP:
        return push_fstream_op(OpSssp{s.val, s.next, s.overflow, s.far, s.bound}, tasks, ntasks, total_chunks, list, off, col, w, s.pk, st);
    case ALGO_SSSP_WIDE:
        return push_fstream_op(OpSsspWide{{s.val, s.next, s.overflow, s.far, s.bound}, s.marks, (uint8_t)s.tag}, tasks, ntasks, total_chunks, list, off, col,
                               w, s.pk, st);
    case ALGO_CC_WIDE:
        return push_fstream_op(OpCcWide{{s.val, s.next}, s.marks, (uint8_t)s.tag}, tasks, ntasks, total_chunks, list, off, col,
                               w, s.pk, st);
    case ALGO_CC:
        return push_fstream_op(OpCc{s.val, s.next}, tasks, ntasks, total_chunks, list, off, col, w, s.pk, st);
    case ALGO_BFS_RELAX:
        return push_fstream_op(OpBfsRelax{s.val, s.next}, tasks, ntasks, total_chunks, list, off, col, w, s.pk, st);
    case ALGO_MBFS_WIDE:
        return push_fstream_op(OpMBfsWide(s), tasks, ntasks, total_chunks, list, off, col, w, s.pk, st);
    case ALGO_MBFS:
        return push_fstream_op(OpMBfs{s.mcur, s.mnext, s.mvisited, s.lval, s.next, s.level_next, s.lshift}, tasks, ntasks,
                               total_chunks, list, off, col, w, s.pk, st);
    case ALGO_MSSSP:
        return push_fstream_op(OpMSssp<1>{s.mcur, s.mnext, s.lval, s.next, s.overflow, s.lshift}, tasks, ntasks, total_chunks,
                               list, off, col, w, s.pk, st);
    case ALGO_MPPR:
        return push_fstream_op(OpMPpr{s.mcur, s.mnext, s.lx, s.lacc, s.next, s.lshift}, tasks, ntasks, total_chunks,
                               list, off, col, w, s.pk, st);
    default:
        return push_fstream_op(OpPr{s.acc, acc_slots(s.n), s.contrib, s.acc_copies - 1}, tasks, ntasks, total_chunks, list, off, col, w,
                               s.pk, st, s.link_grid);
    }
}

hipError_t launch_pr_apply(uint64_t n, float* x, const float* acc, uint32_t copies, float base, float damping,
                           const float* inv_n, float restart, hipStream_t st) {
    if (!n) return hipSuccess;
    if (copies < 1 || copies > ACC_COPIES + 1) return hipErrorInvalidValue;
    k_pr_apply<<<grid_for(n, 256, 8192), 256, 0, st>>>(n, x, acc, copies, base, damping, inv_n, restart);
    return hipGetLastError();
}

hipError_t launch_dpr_init(uint64_t n, float* delta, const float* inv_n, float restart, hipStream_t st) {
    if (!n) return hipSuccess;
    k_dpr_init<<<grid_for(n, 256, 8192), 256, 0, st>>>(n, delta, inv_n, restart, (float)((double)restart / (double)n));
    return hipGetLastError();
}

hipError_t launch_zc_probe(const uint32_t* src, uint64_t bytes, uint32_t words_per_line, uint32_t* sink,
                           hipStream_t st) {
    if (words_per_line == 0)
        k_zc_probe_stream<<<4096, 256, 0, st>>>((const uint4*)src, bytes / 16, sink);
    else
        k_zc_probe_lines<<<4096, 256, 0, st>>>(src, bytes / 128, words_per_line, sink);
    return hipGetLastError();
}

hipError_t launch_copy_probe(void* dst, const void* src, uint64_t bytes, hipStream_t st) {
    k_copy_probe<<<8192, 256, 0, st>>>((uint4*)dst, (const uint4*)src, bytes / 16);
    return hipGetLastError();
}

hipError_t launch_select_only(uint64_t npart, const uint64_t* E, const uint64_t* nA, const uint64_t* Ea,
                              const uint64_t* Rq, const SelParams& sp, uint8_t* p, hipStream_t st) {
    if (!npart) return hipSuccess;
    k_select_only<<<grid_for(npart, 256, 4096), 256, 0, st>>>(npart, E, nA, Ea, Rq, sp, p);
    return hipGetLastError();
}

// Scratch of the allocation-free selection: the four statistics arrays (uint64 x npart
// each) followed by the engine codes (npart bytes), for at most STATIC_SEL_MAX_PARTS
// partitions.  Each device holds its own copy for the life of the process.  In host code
// the array's name stands for no device address; its address on the current device comes
// from hipGetSymbolAddress, once per device, below.
static __device__ __align__(256) uint64_t scratch[STATIC_SEL_WORDS];

hipError_t static_select_scratch(int device, uint64_t** out) {
    static std::mutex mu;
    static uint64_t* ptr[STATIC_SCRATCH_DEVICES] = {};
    if (device < 0 || device >= STATIC_SCRATCH_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;  // the caller makes the device current
        void* at = nullptr;
        e = hipGetSymbolAddress(&at, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr[device] = (uint64_t*)at;
    }
    *out = ptr[device];
    return hipSuccess;
}

}  // namespace hytm
