// Launch shape of the pairwise kernel: how an evaluation of n_i
// i-particles against n_j j-particles is cut into work-groups and j-ranges
// (Section 3.2's bundles and j-split), and the default shape for a size.
// Shared by the host launch code and, for block steps, by the device.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "nbody.h"

namespace nb {

// Launch geometry of the pairwise kernel for an i-list of ni against nj:
// nb i-blocks of per_blk particles and S j-ranges of jchunk records (a
// multiple of the tile).  Enough work-groups to cover the 256 CUs several
// times, with at least min_tiles tiles per j-range.  Used by the host for direct
// calls and by the device for block steps whose size only it knows.  Small
// self-gravitating sets are latency-bound: a j-range of one tile per
// work-group was the fastest on MI355X from N = 256 to 4096 (N = 1024:
// pairwise 10.7 us against 28 us with four tiles per range).
__host__ __device__ inline void split_plan(int64_t ni, int64_t nj, int per_blk, int tile_j, int split_req,
                                           int* nb_out, int* S_out, int* jchunk_out, int min_tiles = 1) {
    const int64_t nb = (ni + per_blk - 1) / per_blk;
    int64_t S = split_req;
    if (S <= 0) {
        const int64_t target = 2048;
        if (nb <= 0 || nb >= target / 2) {
            S = 1;
        } else {
            S = (target + nb - 1) / nb;
            int64_t smax = nj / ((int64_t)min_tiles * tile_j);
            if (smax < 1) smax = 1;
            if (S > smax) S = smax;
            if (S < 1) S = 1;
        }
    }
    int64_t jchunk = (nj + S - 1) / S;
    jchunk = ((jchunk + tile_j - 1) / tile_j) * tile_j;
    if (jchunk <= 0) jchunk = tile_j;
    int64_t S2 = (nj + jchunk - 1) / jchunk;
    if (S2 < 1) S2 = 1;
    *nb_out = (int)nb;
    *S_out = (int)S2;
    *jchunk_out = (int)jchunk;
}

// Number of j-ranges for an i-list of ni against nj (see split_plan).  Long
// evaluations also split j: with at least kLongWG work-groups in all, the
// last, partly filled round of resident work-groups is a small part of the
// launch.  Each range keeps at least kLongTiles tiles, and the partials stay
// below (kLongWG + i-blocks) x (i per block) x 56 B.  On MI355X at N = 2^20
// this took the large DS evaluation from 749 to 726 ms (4096 i-blocks, 8
// ranges), and 2^17 i against 2^20 j from 96 to 90 ms (64 ranges).
constexpr int64_t kLongWG = 32768;
constexpr int64_t kLongTiles = 64;
// The long-evaluation split keeps its partial sums (8 rows of 8 bytes per
// i and range at most) within this many bytes.
constexpr int64_t kLongPartBytes = (int64_t)1 << 31;
// Ranges of five tiles that hold nj records (the last may be shorter).
inline int64_t fine_ranges(int64_t nj, const nbody_tile& t) { return (nj + 5 * t.tile_j - 1) / (5 * t.tile_j); }
inline int choose_split(int prec, int64_t ni, int64_t nj, const nbody_tile& t, int kind = 0) {
    int nb, S, jc;
    split_plan(ni, nj, t.wg * t.ipt, t.tile_j, 0, &nb, &S, &jc);
    // 64-record tiles, DS: twice the work-groups of split_plan, in ranges of
    // five tiles or more: more than the chip holds at once (2560: ten a CU), so
    // the CUs fill up evenly.  One round depends on how the dispatcher happens
    // to spread it (N = 16384, 2048 work-groups: 201 or 231 us by which kernel
    // ran before; 4096: 204).  Coarse to fine, whole calls: N = 12000 122 to
    // 114 us, 18000 261 to 247, 22000 390 to 354, 30000 698 to 637, 1500 i
    // against 262144 j 355 to 300; N = 20001 loses (288 to 297), and N = 8192
    // would, with two tiles a range (4%).  Five tiles to the record: rounded
    // down to fewer ranges they are six, and 2560 to 3000 work-groups, a
    // second round for a few of them (256 i against 524288 j: 137 us coarse,
    // 141 in six tiles, 138 in five; N = 12000 127 in six).  The other kinds'
    // shorter loops gain from 24 tiles a (coarse) range on only: neighbours at
    // N = 20001, 22 tiles, 342 to 353 us, 22000, 29 tiles, 467 to 421, 40000
    // 1483 to 1268; force-only 181 to 195, 244 to 233, 756 to 677.  Float32
    // keeps its ranges: each is one float32 sum.
    if (prec == 1 && t.tile_j == 64 && nb > 0 && (kind == 0 || jc >= 24 * t.tile_j))
        S = (int)std::max<int64_t>(S, std::min((4096 + nb - 1) / (int64_t)nb, fine_ranges(nj, t)));
    const int64_t per = (int64_t)t.wg * t.ipt;
    const int64_t nbl = (ni + per - 1) / per;
    int64_t Sl = nbl > 0 ? (kLongWG + nbl - 1) / nbl : 1;
    Sl = std::min<int64_t>(Sl, nj / (kLongTiles * t.tile_j));
    Sl = std::min<int64_t>(Sl, kLongPartBytes / (64 * std::max<int64_t>(ni, 1)));
    return (int)std::max<int64_t>(S, Sl);
}

// Default launch shape when neither an override nor a tuned entry exists:
// the fastest shape of the MI355X sweep at 2^20 x 2^20 (256-record LDS
// tiles, software-pipelined LDS reads; two i per lane for DS, one for plain
// FP32) for large problems,
// 64-record tiles for small ones (more j-ranges to spread over the CUs), and
// for the smallest j sets (latency-bound: the time is one work-group's
// sweep) 32- or 16-record tiles in one-wave work-groups.  short_tiles: the
// evaluation kind has those shapes.
inline nbody_tile default_tile(int prec, int64_t ni, int64_t nj, bool short_tiles = true) {
    nbody_tile t;
    const bool large = (double)ni * (double)nj >= 4294967296.0;
    t.tile_j = large ? 256 : 64;
    t.wg = large ? 256 : 128;
    if (!large && short_tiles && nj <= 2048) {
        t.tile_j = nj <= 512 ? 16 : 32;
        t.wg = 64;
    }
    // DS at large sizes: two i per lane (with the long-evaluation split,
    // 683 ms at 2^20 against 709-713 ms for one i per lane, same box);
    // plain FP32 keeps one i per lane (578-580 ms against 594)
    t.ipt = (large && prec == 1) ? 2 : 1;
    t.split = 0;
    t.jsrc = 0;
    t.unroll = large ? (prec == 1 ? 101 : 102) : 0;
    t.waves = 0;
    return t;
}

// Defaults of the force-only (kind 1) and nearest-neighbour (kind 2)
// evaluations: the fastest shapes of the MI355X sweep at 2^20 x 2^20; small
// problems take the small default shape.
inline nbody_tile default_tile_kind(int kind, int prec, int64_t ni, int64_t nj) {
    // the full evaluation's default (two i per lane for DS at large sizes) is
    // also the fastest force-only and neighbour shape of the sweeps
    return default_tile(prec, ni, nj, kind == 0);
}

// No fewer than choose_split gives for this shape against nj j or fewer, of
// any kind: its rules without the rounding to whole tiles, which can leave a
// larger j set with fewer ranges than a smaller one.
inline int64_t split_bound(int prec, int64_t ni, int64_t nj, const nbody_tile& t) {
    const int64_t per = (int64_t)t.wg * t.ipt, nb = std::max<int64_t>(1, (ni + per - 1) / per);
    int64_t S = nb < 1024 ? std::min((2048 + nb - 1) / nb, nj / t.tile_j) : 1;
    if (prec == 1 && t.tile_j == 64) S = std::max(S, std::min((4096 + nb - 1) / nb, fine_ranges(nj, t)));
    const int64_t Sl = std::min((kLongWG + nb - 1) / nb, nj / (kLongTiles * t.tile_j));
    return std::max(S, std::min(Sl, kLongPartBytes / (64 * std::max<int64_t>(ni, 1))));
}

// The most split-partial rows (j-ranges x i) that any evaluation of up to
// max_i i-particles against up to max_j j-particles takes; tile_of(n_i, n_j)
// is its launch shape, split 0 where choose_split fills it in.  The ranges
// fall in steps as the i-blocks grow, towards one of three work-group counts,
// so the most rows stand just before a step; and the j counts at which the
// default shape changes may take more ranges than max_j itself.
template <class TileOf>
int64_t part_rows_upto(int prec, int64_t max_i, int64_t max_j, TileOf tile_of) {
    int64_t rows = 0;
    auto at = [&](int64_t n) {
        if (n < 1 || n > max_i) return;
        for (const int64_t j : {max_j, (((int64_t)1 << 32) - 1) / n, (int64_t)2048, (int64_t)512, n}) {
            const int64_t m = std::min(j, max_j);
            if (m < 1) continue;
            const nbody_tile t = tile_of(n, m);
            const int tj = std::min(t.tile_j, 64);   // eps = 0 and the other kinds may go back to 64 or 128
            const int64_t S = t.split > 0 ? std::min<int64_t>(t.split, (m + tj - 1) / tj) : split_bound(prec, n, m, t);
            if (S > 1) rows = std::max(rows, S * n);
        }
    };
    at(max_i);
    for (const int64_t j : {max_j, (int64_t)2048, (int64_t)512})   // last size below the large shape
        if (j > 0) at((((int64_t)1 << 32) - 1) / j);
    at(65535);                                                    // that of a set against itself
    for (int64_t n = 1; n < max_i; n *= 2) at(n), at(n - 1);      // tuned shapes go by powers of two
    for (const int64_t per : {64, 128, 256, 512, 1024})
        for (const int64_t groups : {(int64_t)2048, (int64_t)4096, kLongWG})
            for (int64_t k = 1; (k - 1) * (k - 1) <= groups; ++k) {
                at(k * per);
                if (k > 1) at(((groups + k - 2) / (k - 1) - 1) * per);   // the most blocks with k ranges
            }
    return rows;
}

// Shape of the pair-symmetric evaluation of n particles (sym.hip): blocks of
// lb particles, bands of nd block distances, each block's stretch of a band
// in np pieces of lp.  tj: the j-tile whose partial sums it forms (64 or 256).
struct SymShape {
    int nb, lb, lbs, nd, np, lp;
    int dists;          // distances 0 .. nb / 2
    size_t bytes;       // float64 rows of one launch
};
// The rows of one launch stay within this many bytes.
constexpr int64_t kSymBytes = (int64_t)1 << 31;
constexpr int kSymGroup = 1024;      // i-particles a work-group holds at a time
constexpr int kSymResident = 1024;   // work-groups on the chip at once: four per CU
// 20001 bodies: 344 us against the general kernel's 291; 25001: 435 against
// 446; force-only 26001: 283 against 311
constexpr int64_t kSymMin = 24576;
constexpr int64_t kSymMax = (int64_t)1 << 24;   // beyond, two rows pass kSymBytes (112 B a particle)
// rows are padded to whole groups, so a shape depends on n by its groups only
constexpr int64_t sym_stride(int64_t n) { return (n + kSymGroup - 1) / kSymGroup * kSymGroup; }
inline SymShape sym_shape(int64_t n, int tj, int quantities) {
    SymShape best{};
    double best_t = 0.0;
    const int64_t row = 8 * (int64_t)quantities * sym_stride(n);
    for (int g = 0; g < 4; ++g) {
        SymShape s;
        s.lbs = 10 + g;
        s.lb = 1 << s.lbs;
        s.nb = (int)((n + s.lb - 1) >> s.lbs);
        s.dists = s.nb / 2 + 1;
        int last_np = 0;
        for (int r = 1; r <= 8; ++r) {
            // about r rounds of work-groups
            const int np = std::max(1, r * kSymResident / s.nb);
            if (np == last_np || (np > 1 && row * (np + 1) > kSymBytes)) continue;
            last_np = np;
            const int64_t most = std::max<int64_t>(1, kSymBytes / row - np);
            const int bands = (int)((s.dists + most - 1) / most);
            s.nd = (s.dists + bands - 1) / bands;
            const int64_t len = (int64_t)s.nd << s.lbs;
            s.lp = (int)(((len + np - 1) / np + tj - 1) / tj * tj);
            s.np = (int)((len + s.lp - 1) / s.lp);
            s.bytes = (size_t)row * (size_t)(s.nd + s.np);
            // time in steps of a work-group (about 1 us): rounds of items and
            // most of another for the CUs' unequal pace (2^17 bodies: 9.3 ms
            // in one round, 8.2 in seven; 40000, force only: 0.69 ms in two,
            // 0.66 in three and a third); the rows' way through memory
            const double rounds = std::max(1.0, (double)s.nb * s.np / kSymResident);
            const double t = bands * ((rounds + 0.8) * (1 << g) * (s.lp + tj / 4 + 40) +
                                      (double)row * (s.nd + s.np) / 2.5e6 + 5);
            if (best_t == 0.0 || t < best_t) {
                best_t = t;
                best = s;
            }
        }
    }
    return best;
}
// Bytes of the rows of every pair-symmetric evaluation of up to `most`
// particles, of either kind.  A shape depends on n by its group of kSymGroup
// and by the j-tile, which changes once over all sizes, so each group's first
// and last size stand for it.  From 2^18 on: all that a launch may take.
inline size_t sym_bytes_upto(int64_t most) {
    if (most < kSymMin) return 0;
    if (most >= (1 << 18)) return (size_t)kSymBytes;
    size_t bytes = 0;
    for (int64_t first = kSymMin; first <= most; first = sym_stride(first) + 1)
        for (const int64_t n : {first, std::min(sym_stride(first), most)})
            for (int kind = 0; kind < 2; ++kind)
                bytes = std::max(bytes, sym_shape(n, default_tile_kind(kind, 1, n, n).tile_j, kind == 1 ? 4 : 7).bytes);
    return bytes;
}

}  // namespace nb
