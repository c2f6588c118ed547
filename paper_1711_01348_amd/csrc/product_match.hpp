// Recognition of sums of products that separate over the function indices (product.hpp).  Host only; included by
// families.cpp.
#pragma once
#include <algorithm>
#include <cmath>

#include "plan.hpp"
#include "product.hpp"

namespace tad {

// Time of a product in cycles of 2.2 GHz.  Tiles go to the 256 compute units in turn, and a unit works on as many at once as registers and LDS leave room
// for; the next one starts when one of them is done.  A tile begins and ends (kEnds, longer where others do at the same time), and between them takes
// stages of kProductStage values of q: the matrix instructions, 512 `rows` cycles, and what is not hidden behind them where it has the unit to itself
// (`alone`), its share of the matrix cores where it has not (`shared`, longer for low tiles: more fragments to read per instruction).
// Fitted to 197 forward passes, 17 .. 6957 x 16 .. 5000 x 20 .. 5400 with every height, both orientations and several numbers of pieces, and to both
// gradients of 225 products in two launches and in one of every height: 4 % from the measured times in the mean.  What is picked takes 0.6 % longer than
// the fastest in the mean and 11 % at most (forward), 0.7 % and 17 % (gradients; 385 x 902 x 1580 56.1 / 48.0 us); with a cost per tile and one per stage,
// the same for all heights, and no account of the units' order 0.8 % and 14 %, 2.1 % and 36 % (1107 x 74 x 1411 26.4 / 20.0).  Heights that earn their
// place: 5 1000 x 1203 x 777 in 64 bits 41 us instead of 53; 7 1433 x 1190 x 306 24.6 / 26.7, 1665 x 1019 x 147 15.8 / 16.7; 6 where a program follows,
// 3000 x 1500 x 64 44 / 48, 4710 x 315 x 76 17.9 / 21.8 (8 was the fastest nowhere).
constexpr int kUnits = 256;
constexpr double kBegin = 3100, kEnds = 3150, kEndsRow = 1000, kEndsMore = 0.36;
// The launch that adds pieces up, and a second launch for the other gradient; launches one after the other take at least 3.9 us each, 5 where the host is slow.
constexpr double kReduceCycles = 4100, kReduceBytes = 2050, kLaunchCycles = 800, kLeastCycles = 10000;
// A program that is applied to the results: where they are stored, in passes over a thread's results of every tile on a unit, which hide little of each other
// (but low tiles: one pass, three on a unit); and for sums in pieces in the launch that adds them up.  Dense layers with tanh, 40 sizes with every height
// and up to 13 pieces: 5 % from the measured times, what is picked takes 1.4 % longer than the fastest in the mean and 8 % at most; 2032 x 481 x 20 with
// tiles of 32 rows, two rounds of them, 12.9 us, of 64 rows 10.4.
constexpr double kOuterLaunch = 9000;
static double outer_cycles(const ProductDesc &d, int rows, int64_t each) {
    const int passes = (2 * rows + d.outer - 1) / d.outer;
    if (d.outer <= 2) return (1500 + 5400.0 * passes) * (1.2 * (double)each - 0.2);
    return rows == 1 && passes == 1 ? 4200 + 2000.0 * (double)each : (2000 + 4400.0 * passes) * (1.25 * (double)each - 0.25);
}
// Results that could be scaled where they are stored, of a sum in pieces: a launch over them (softplus 538 x 473 x 29, the gradient of one operand 25.0 us
// whole, 29.2 in pieces).
constexpr double kScaleLaunch = 10000;
static int64_t stages_of(int64_t q) { return (q + kProductStage - 1) / kProductStage; }
struct TileRate {
    int at_once;
    double alone, shared, ends;
    double stage(int n) const { return std::max(alone, n * shared); }   // of each of n tiles
    double begin_end(int n) const { return ends * (1 + kEndsMore * (n - 1)); }
    double round(int n, int64_t stages) const { return begin_end(n) + (double)stages * stage(n); }
};
static TileRate tile_rate(const ProductDesc &d, int rows) {
    const bool wide = d.a64 && d.b64;
    TileRate r;
    r.at_once = wide ? (rows == 1 ? 2 : 1) : rows == 1 ? 3 : rows <= (d.a64 || d.b64 ? 3 : 4) ? 2 : 1;
    r.alone = 512.0 * rows + (wide ? 457 : 275);
    r.shared = rows == 1 ? (wide ? 865 : 675) : rows == 2 ? 1115 : 497.0 * rows;
    r.ends = kEnds + kEndsRow * rows;
    return r;
}
static int64_t tile_count(const ProductDesc &d, int rows, bool flip) {
    const int64_t R = flip ? d.C : d.R, C = flip ? d.R : d.C;
    return ((R + 16 * rows - 1) / (16 * rows)) * ((C + kProductCols - 1) / kProductCols);
}
// sums of 64-bit operands take three sets of registers: a tile of six does not fit
static int rows_limit(const ProductDesc &d) { return d.a64 && d.b64 ? 5 : 7; }
static double product_cycles(const ProductDesc &d, int rows, bool flip, int pieces, int chunk) {
    const TileRate r = tile_rate(d, rows);
    const int64_t each = (tile_count(d, rows, flip) * pieces + kUnits - 1) / kUnits, rounds = (each + r.at_once - 1) / r.at_once;
    const int64_t stages = stages_of(chunk);
    double t = kBegin + (double)(rounds - 1) * r.round(r.at_once, stages) + r.round((int)(each - (rounds - 1) * r.at_once), stages);
    if (d.scaled && pieces > 1) t += kScaleLaunch;
    if (d.outer) t += pieces > 1 ? kOuterLaunch : outer_cycles(d, rows, each);
    if (pieces == 1) return t;
    t += kReduceCycles + (double)pieces * d.R * d.C * 16.0 / kReduceBytes;   // written and read
    return std::max(t, kLeastCycles * (2 + (d.scaled || d.outer)));
}

void product_shape(ProductDesc &d, size_t most_bytes) {
    d.pair_rows = 0;
    double best = -1;
    for (int flip = 0; flip < 2; ++flip)   // 16 x 100000 results are tiles of 16 x 64, not of 64 x 64 a quarter full
        for (int rows = 1; rows <= rows_limit(d); ++rows) {
            const int64_t tiles = tile_count(d, rows, flip);
            // more pieces than one only where the tiles leave compute units idle, and none shorter than 128
            const int64_t most = tiles < 256 ? std::max<int64_t>(1, std::min<int64_t>(512 / tiles, d.Q / 128)) : 1;
            for (int64_t want = 1; want <= most; want += 1 + want / 8) {
                const int chunk = want == 1 ? d.Q : (int)(((d.Q + want - 1) / want + 127) / 128 * 128);
                const int pieces = (d.Q + chunk - 1) / chunk;
                if (pieces > 1 && (size_t)pieces * d.R * d.C * sizeof(double) > most_bytes) break;
                const double t = product_cycles(d, rows, flip, pieces, chunk);
                if (best >= 0 && t >= best) continue;
                best = t;
                d.rows = rows;
                d.flip = flip;
                d.pieces = pieces;
                d.chunk = chunk;
            }
        }
}

ProductDesc product_turned(const ProductDesc &d) {
    ProductDesc t = d;
    std::swap(t.R, t.C);
    std::swap(t.ar, t.bc);
    std::swap(t.aq, t.bq);
    std::swap(t.a64, t.b64);
    return t;
}

// n0 tiles of s0 stages, then n1 of s1 <= s0, in one launch.  Units that have had the same tiles are followed together, from the end of one of their
// tiles to the next; whole rounds of equal tiles are not followed.  Of units that have a place at about the same time the emptiest one gets the tile.
constexpr double kSoon = 1500;
static double pair_cycles(int64_t n0, int64_t s0, int64_t n1, int64_t s1, const TileRate &r) {
    struct Tile { bool first; double ends, stages; };
    struct Group { double at; int64_t units, ended; int n; Tile tile[3]; };   // the time of the state, tiles of the first kind that end then, what is left of the others
    Group g[4], now[4];   // three at most: units part where either kind of tiles runs out
    int groups = 0;
    const int64_t round = (int64_t)kUnits * r.at_once, stages[2] = {s0, s1};
    const int64_t whole = std::max<int64_t>(0, n0 / round - 1);
    int64_t left[2] = {n0 - whole * round, n1}, longs = left[0];
    double skipped = kBegin + (double)whole * r.round(r.at_once, s0), last = 0;
    // gives the free places of a group's units their next tiles, one place of all of them after the other
    auto start = [&](const Group &from) {
        int count = 1;
        now[0] = from;
        now[0].ended = 0;
        for (bool any = true; any && (left[0] || left[1]);) {
            any = false;
            for (int i = 0; i < count && (left[0] || left[1]); ++i) {
                if (now[i].n == r.at_once) continue;
                const int k = left[0] ? 0 : 1;
                if (left[k] < now[i].units) {
                    now[count] = now[i];
                    now[count++].units -= left[k];
                    now[i].units = left[k];
                }
                left[k] -= now[i].units;
                now[i].tile[now[i].n++] = {k == 0, r.ends, (double)stages[k]};
                any = true;
            }
        }
        for (int i = 0; i < count; ++i) {
            if (now[i].n) g[groups++] = now[i];
            else last = std::max(last, now[i].at);
        }
    };
    // to the end of one of its tiles
    auto advance = [&](Group &p) {
        for (bool done = false; !done;) {
            int running = 0;
            for (int i = 0; i < p.n; ++i) running += p.tile[i].ends <= 0;
            const double step = r.stage(running), slow = r.begin_end(p.n) / r.ends;
            double dt = 1e300;
            for (int i = 0; i < p.n; ++i) dt = std::min(dt, p.tile[i].ends > 0 ? p.tile[i].ends * slow : p.tile[i].stages * step);
            p.at += dt;
            int kept = 0;
            for (int i = 0; i < p.n; ++i) {
                Tile t = p.tile[i];
                if (t.ends > 0) t.ends = t.ends - dt / slow > 1e-3 ? t.ends - dt / slow : 0;
                else t.stages -= dt / step;
                if (t.ends <= 0 && t.stages < 1e-6) {
                    done = true;
                    if (t.first) p.ended += p.units;
                } else p.tile[kept++] = t;
            }
            p.n = kept;
        }
    };
    start({0, kUnits, 0, 0, {}});
    for (int i = 0; i < groups; ++i) advance(g[i]);
    while (groups) {
        int next = 0;
        for (int i = 1; i < groups; ++i)
            if (g[i].at < g[next].at) next = i;
        const double soon = g[next].at + kSoon;
        for (int i = 0; i < groups; ++i)
            if (g[i].at <= soon && g[i].n < g[next].n) next = i;
        const Group p = g[next];
        g[next] = g[--groups];
        longs -= p.ended;
        if (!longs && left[1] > 2 * round) {
            const int64_t more = left[1] / round - 1;
            left[1] -= more * round;
            skipped += (double)more * r.round(r.at_once, s1);
        }
        const int behind = groups;
        start(p);
        for (int i = behind; i < groups; ++i) advance(g[i]);
    }
    return skipped + last;
}

void product_pair(ProductDesc &x, ProductDesc &y) {
    x.pair_rows = y.pair_rows = 0;
    double best = product_cycles(x, x.rows, x.flip, x.pieces, x.chunk) + product_cycles(y, y.rows, y.flip, y.pieces, y.chunk) + kLaunchCycles;
    for (int flips = 0; flips < 4; ++flips) {
        const bool fx = flips & 1, fy = flips >> 1;
        // one kernel: both with operands of the same widths in the same order
        if ((fx ? x.b64 : x.a64) != (fy ? y.b64 : y.a64) || (fx ? x.a64 : x.b64) != (fy ? y.a64 : y.b64)) continue;
        for (int rows = 1; rows <= rows_limit(x); ++rows) {
            const int64_t nx = tile_count(x, rows, fx), ny = tile_count(y, rows, fy);
            const int64_t sx = stages_of(x.Q), sy = stages_of(y.Q);
            const TileRate r = tile_rate(x, rows);
            const double even = ((double)nx * (double)sx + (double)ny * (double)sy) / kUnits;   // stages of a unit, no fewer than this
            if (kBegin + r.ends + std::max(even * r.stage(r.at_once) / r.at_once, (double)std::max(sx, sy) * r.alone) >= best) continue;
            const double t = sx >= sy ? pair_cycles(nx, sx, ny, sy, r) : pair_cycles(ny, sy, nx, sx, r);
            if (t >= best) continue;
            best = t;
            x.pair_rows = y.pair_rows = rows;
            x.pair_flip = fx;
            y.pair_flip = fy;
        }
    }
}

size_t product_partial_bytes(const ProductDesc &d) {
    return d.pieces > 1 ? align256((size_t)d.pieces * (size_t)d.R * (size_t)d.C * sizeof(double)) : 0;
}

bool product_group_stride(const int64_t *off, const int64_t *extent, int count, int64_t &stride) {
    stride = 0;
    int64_t inner = 1;     // values of the indices behind the current one
    bool first = true;
    for (int d = count - 1; d >= 0; --d) {
        if (extent[d] == 1) continue;
        if (first) stride = off[d];
        else if (off[d] != stride * inner) return false;
        first = false;
        inner *= extent[d];
    }
    return stride >= 0;
}

bool product_addressable(const ProductDesc &d) {
    const int64_t limit = (int64_t)1 << 21;
    return d.ar < limit && d.aq < limit && d.bq < limit && d.bc < limit;
}

// Terms from which 32-bit products whose extents are multiples of four run on the contraction family.  Forward and both
// gradients there / here: 256 x 256 x 256 21 / 12 us, 200 x 300 x 400 30 / 15, 76 x 348 x 1656 28 / 18, 400 x 400 x 400 36 / 20, 512 x 512 x 512 29 / 23,
// 1024 x 1024 x 128 26 / 24, 576 x 576 x 576 33 / 34, 640 x 640 x 640 36 / 42, 640 x 1280 x 320 33 / 43; from here on 512 x 512 x 1024 34 / 37, 704 x 704 x 704 39 / 46,
// 100 x 2000 x 2000 52 / 77, 1000 x 1000 x 1000 82 / 112.  Between 2^27 and 2^28 terms the family's tiles of 64 x 64 are the faster ones; the line stays
// where it is because its sums are in 32 bits, and those of these products never were.
constexpr double kContractionTerms = 268435456.0;
// ... and below that, the results of 32-bit products whose sums are so short that storing them is what counts: its tiles store 16 bytes
// per lane.  There / here, rows x columns x terms: 2000 x 1000 x 32 4.9 / 8.0 us, x 128 8.6 / 14.4, 1000 x 4096 x 16 7.3 / 14.4, 128 x 16000 x 16
// 5.2 / 8.1, 4096 x 4096 x 8 18.5 / 46; beyond the line, where the sums stay in 64 bits: 1300 x 1000 x 128 8.0 / 11.5, 1024 x 1024 x 128 5.2 / 8.9,
// 100000 x 64 x 16 10.0 / 22.5, 400 x 400 x 400 12.2 / 8.2.
static bool contraction_stores(const ProductDesc &d) {
    return d.Q <= 128 && std::min(d.R, d.C) >= 128 && (int64_t)d.R * d.C >= 1500000;
}

// General kernels / dense products, M x N x K.  64 bits: 100000 x 16 x 9 18.5 / 28.4 us, x 33 x 9 33 / 52, x 129 x 9 108 / 122, 4096 x 4096 x 8
// 125 / 127; 100000 x 33 x 16 55 / 52, 10001 x 64 x 8 9.6 / 8.6.  32 bits: 100001 x 16 x 8 10.9 / 15.5, x 33 18.8 / 23.0, 100001 x 17 x 9
// 15.8 / 17.3, 10001 x 129 x 9 10.4 / 12.5; 100001 x 33 x 9 21 / 18, 100001 x 17 x 17 25 / 17, 100001 x 16 x 65 34 / 33.
bool product_sum_short(bool f64, int64_t M, int64_t N, int64_t K) {
    if (M * N < ((int64_t)1 << 20)) return false;
    const int64_t least = std::min(M, N);
    if (K < 12) return f64 || least <= 32 || M * N < ((int64_t)1 << 21);
    return !f64 && least <= 16 && K < 40;
}

void match_product(tad_plan &pl) {
    ProductPlan &pp = pl.prod;
    pp = ProductPlan{};
    const tad_expr &e = pl.expr;
    if (pl.flags & TAD_PLAN_GENERIC_ONLY) return;
    if (pl.has_alias || e.n_constraints > 0 || e.n_sum < 1 || e.n_f < 2) return;
    if (e.body != TAD_BODY_MUL) return;
    // the contraction family's tiles in 32 bits are for larger products
    if (pl.fwd_family != TAD_FAMILY_GENERIC && !(pl.fwd_family == TAD_FAMILY_CONTRACTION && pl.terms_total < kContractionTerms)) return;
    for (int s = 0; s < e.n_sum; ++s)
        if (e.sum_lo[s] != 0) return;
    // every function index belongs to one factor: the leading ones to one of them, the trailing ones to the other
    auto moves = [&](int p, int d) { return pl.fwd.off[p][d] != 0; };
    int lead = 0;    // function indices of m
    const int first = moves(0, 0) ? 0 : 1;
    while (lead < e.n_f && moves(first, lead) && !moves(1 - first, lead)) ++lead;
    if (lead == 0 || lead == e.n_f) return;
    for (int d = lead; d < e.n_f; ++d)
        if (moves(first, d) || !moves(1 - first, d)) return;
    int64_t extent[TAD_MAX_EXT];
    int64_t M = 1, N = 1, K = 1;
    for (int d = 0; d < pl.n_ext; ++d) {
        extent[d] = pl.hi[d] - pl.lo[d] + 1;
        (d < lead ? M : d < e.n_f ? N : K) *= extent[d];
    }
    if (M < kProductExtent || N < kProductExtent || K < kProductSum || K >= ((int64_t)1 << 30)) return;
    pp.M = M; pp.N = N; pp.K = K;
    const bool f64 = pl.dtype == TAD_F64;
    for (int q = 0; q < 2; ++q) {
        ProductSide &s = pp.side[q];
        s.operand = q == 0 ? first : 1 - first;
        const int64_t *off = pl.fwd.off[s.operand];
        const int at = q == 0 ? 0 : lead, count = q == 0 ? lead : e.n_f - lead;
        if (!product_group_stride(off + at, extent + at, count, s.sm)) return;
        if (!product_group_stride(off + e.n_f, extent + e.n_f, e.n_sum, s.sk)) return;
    }
    const ProductSide &A = pp.side[0], &B = pp.side[1];
    ProductDesc &f = pp.set.forward;
    f.R = (int)M; f.C = (int)N; f.Q = (int)K;
    f.ar = A.sm; f.aq = A.sk; f.bq = B.sk; f.bc = B.sm;
    f.a64 = f.b64 = f64;
    if (!product_addressable(f)) return;
    const bool contraction = pl.fwd_family == TAD_FAMILY_CONTRACTION;
    pp.forward_on = contraction ? !contraction_stores(f) : !product_sum_short(f64, M, N, K);
    for (int q = 0; q < 2; ++q) {
        ProductSide &s = pp.side[q];
        const ProductSide &o = pp.side[1 - q];
        const int64_t X = q == 0 ? M : N, Y = q == 0 ? N : M;   // extents of the factor's own and of the other function index
        const int64_t gx = q == 0 ? N : 1, gy = q == 0 ? 1 : N;  // strides of the gradient of the sum along them
        // the products fill the tensor only if its elements and the pairs (m, k) or (n, k) are the same thing
        const bool rows = s.sm == K && s.sk == 1, cols = s.sm == 1 && s.sk == X;
        if (!pl.ap[s.operand].derived || pl.arg_count[s.operand] != X * K || !(rows || cols)) continue;
        s.k_major = !rows;
        ProductDesc &d = pp.set.grad[q];
        d.Q = (int)Y;
        if (rows) { d.R = (int)X; d.C = (int)K; d.ar = gx; d.aq = gy; d.bq = o.sm; d.bc = o.sk; }   // sum_y g(x, y) O(k, y)
        else { d.R = (int)K; d.C = (int)X; d.ar = o.sk; d.aq = o.sm; d.bq = gy; d.bc = gx; }        // sum_y O(k, y) g(x, y)
        d.a64 = d.b64 = f64;
        if (!product_addressable(d) || (contraction && contraction_stores(d))) continue;
        s.grad = true;
    }
    auto shape = [&](ProductSet &set, size_t most) {
        size_t bytes = 0;
        for (ProductDesc *d : {&set.forward, &set.grad[0], &set.grad[1]}) {
            if (!(d == &set.forward ? pp.forward_on : pp.side[d - set.grad].grad)) continue;
            product_shape(*d, most);
            bytes = std::max(bytes, product_partial_bytes(*d));
        }
        if (pp.side[0].grad && pp.side[1].grad) product_pair(set.grad[0], set.grad[1]);
        set.ws_bytes = bytes;
    };
    shape(pp.set, SIZE_MAX);
    const size_t family = align256(pl.ws_bytes), array = TAD_STATIC_SCRATCH_BYTES;
    if (family <= array && family + pp.set.ws_bytes > array) {
        pp.lean = pp.set;
        shape(pp.lean, array - family);
        pp.lean_on = true;
    }
    pp.on = pp.forward_on || pp.side[0].grad || pp.side[1].grad;
}

}  // namespace tad
