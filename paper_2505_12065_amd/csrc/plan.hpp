// What a call does, decided on the host: tiles, slabs, groups and parts of the exact search, LDS layouts and the choice of
// kernel of the graph search.  Plain C++ without the GPU's headers, so that the rules can be compiled and looked at alone.
#pragma once

#include <limits.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

#include "../../include/ann.h"

namespace ann {

constexpr int WAVE = 64;
constexpr size_t LDS_MAX = 160 * 1024;   // LDS of one gfx950 compute unit
constexpr size_t CAND_BYTES = 8;         // a (score, id) pair in the workspace
inline int elem_bytes(int dtype) { return dtype == ANN_F32 ? 4 : 2; }

// ---- exact search, streaming kernel -----------------------------------------------------------------
constexpr int LANE_KP = 4;                            // entries of a lane's list
constexpr int STREAM_NQG_MAX(int elem_bytes) { return elem_bytes == 2 ? 4 : 2; }   // fp32: eight accumulators a group
constexpr int STREAM_WG_PER_CU(int elem_bytes, int nqg, int waves) { return waves == 16 || (elem_bytes == 4 && nqg > 1) ? 1 : 2; }

constexpr int STREAM_LDS_STEPS = (int)((LDS_MAX - 16 * 1024) / (WAVE * 16));   // steps of 64 bytes of a group of 16 queries that LDS holds

// Geometry and options of a flat_stream_kernel launch.
struct StreamPlan {
    int nqg = 1;                 // groups of 16 queries a workgroup serves, 1 .. STREAM_NQG_MAX
    int G = 1;                   // workgroups side by side over the queries, ceil(B / (16 nqg))
    int P = 1;                   // slabs of the corpus
    int waves = 8;               // wavefronts per workgroup
    int lds_steps = 1;           // 64-byte steps of a query held in LDS
    int batch = 4;               // loads of a row that are requested together
    int K = 4;                   // entries of a slab's list: k rounded up to a multiple of 4
    int slots() const { return P * waves; }
};
inline size_t stream_lds_bytes(int nqg, int lds_steps, int waves) {
    const size_t q = (size_t)nqg * lds_steps * WAVE * 16;
    const size_t m = (size_t)nqg * 16 * (4 * waves * LANE_KP + 4) * CAND_BYTES;
    return q > m ? q : m;
}

// Wavefronts of a flat_stream_kernel workgroup: 8, or 16 when the queries' LDS leaves room for one
// workgroup per compute unit only (the corpus loads in flight are what keeps HBM busy).
inline int stream_waves(int elem_bytes, int nqg, int lds_steps) {
    return elem_bytes == 2 && nqg >= 2 && stream_lds_bytes(nqg, lds_steps, 8) > LDS_MAX / 2 ? 16 : 8;
}

// ---- exact search, matrix-core kernel ----------------------------------------------------------------
template <int WMF_, int WNF_, int NWM_, int NWN_, int STAGES_, int PER_CU_, int SB_ = 64>
struct WideCfg {
    static constexpr int WMF = WMF_, WNF = WNF_, NWM = NWM_, NWN = NWN_, STAGES = STAGES_, PER_CU = PER_CU_;
    static constexpr int WAVES = NWM * NWN, THREADS = WAVES * WAVE;
    static constexpr int BM = 32 * WMF * NWM, BN = 32 * WNF * NWN;
    static constexpr int SB = SB_, CPR = SB / 16, RPB = 1024 / SB;      // bytes and 16-byte chunks of a row in a stage; rows to a block
    static constexpr int A_BLK = BM / RPB, BLKS = A_BLK + BN / RPB;     // 1 KB blocks of a stage
    static constexpr int LPW = BLKS / WAVES;                            // blocks loaded per wave and stage
    static_assert(BLKS % WAVES == 0, "blocks must divide evenly over the waves");
    static constexpr int STAGE_BYTES = BLKS * 1024, LDS_BYTES = STAGES * STAGE_BYTES;
};
using WideLarge = WideCfg<4, 2, 2, 4, 4, 1>;              // 256 x 256, 8 waves
using WideTall = WideCfg<4, 2, 4, 2, 4, 1>;               // 512 x 128, 8 waves
using WideMid = WideCfg<2, 2, 4, 2, 3, 1, 128>;           // 256 x 128, 8 waves
using WideSquare = WideCfg<2, 2, 2, 2, 2, 2, 128>;        // 128 x 128, 4 waves, two workgroups per compute unit
using WideThin = WideCfg<2, 1, 2, 2, 3, 2, 128>;          // 128 x 64, 4 waves, two workgroups per compute unit
using WideTiny = WideCfg<1, 1, 2, 2, 4, 2, 128>;          // 64 x 64, 4 waves, two
using WideShort = WideCfg<2, 1, 2, 2, 4, 3>;              // 128 x 64, 4 waves, three: half lines, for short rows

constexpr int WIDE_LARGE = 0, WIDE_TALL = 1, WIDE_MID = 2, WIDE_THIN = 3, WIDE_TINY = 4, WIDE_SHORT = 5, WIDE_SQUARE = 6;
struct WidePlan {
    int cus, shape, wmf;         // compute units; workgroup tile (a WideCfg); its row fragments per wave
    int NT, P;                   // query tiles x slabs of the corpus
    int gs_log;                  // a maximum stands for 2^gs_log rows
    int64_t slots, n;            // rows of whole tiles; groups they make
};

template <class C>
inline void geometry(WidePlan &pl, int cus, int64_t N, int B) {
    const int64_t tiles = (N + C::BM - 1) / C::BM;
    pl.cus = cus;
    pl.wmf = C::WMF;
    pl.NT = (B + C::BN - 1) / C::BN;
    const int64_t cap = (int64_t)cus * C::PER_CU / pl.NT;
    pl.P = (int)(cap < 1 ? 1 : cap < tiles ? cap : tiles);
    pl.slots = tiles * C::BM;
}
inline void wide_geometry(WidePlan &pl, int shape, int cus, int64_t N, int B) {
    pl.shape = shape;
    switch (shape) {
    case WIDE_LARGE: return geometry<WideLarge>(pl, cus, N, B);
    case WIDE_TALL: return geometry<WideTall>(pl, cus, N, B);
    case WIDE_MID: return geometry<WideMid>(pl, cus, N, B);
    case WIDE_TINY: return geometry<WideTiny>(pl, cus, N, B);
    case WIDE_SHORT: return geometry<WideShort>(pl, cus, N, B);
    case WIDE_SQUARE: return geometry<WideSquare>(pl, cus, N, B);
    default: return geometry<WideThin>(pl, cus, N, B);
    }
}

inline int wide_rows(int shape) {                         // corpus rows of a tile
    return shape == WIDE_LARGE ? WideLarge::BM : shape == WIDE_TALL ? WideTall::BM : shape == WIDE_MID ? WideMid::BM
           : shape == WIDE_TINY ? WideTiny::BM : shape == WIDE_SHORT ? WideShort::BM : shape == WIDE_SQUARE ? WideSquare::BM : WideThin::BM;
}

// ---- exact search, the whole call ----------------------------------------------------------------------
constexpr int P_MAX = 2048;      // most slabs of the streaming kernel

// Few queries against few rows.  flat_scores_kernel: tiles of 16 rows x 16 queries, a wave each, and flat_pick_kernel.  It has no tile
// that spares the L1s, so the line is that of the bytes they bring in; short rows make the pick, which looks at every score, the larger part.
// Where the streaming kernel's lists would take the call instead, they pay longest (a little less where one group of 16 queries is well filled); the
// matrix-core kernel's tiles are the better the more queries fill them.  us, lists / this: 10 000 x 128 fp32, B = 16, k = 10 11.6 / 10.3; 21 025 x 480,
// B = 14 13.8 / 12.4; 18 204 x 416, B = 20 18.1 / 14.8; but 27 070 x 896, B = 16 17.4 / 21.4; 33 953 x 64, B = 8 10.0 / 12.6.  Matrix cores / this: 200 x 768, B = 1
// 8.5 / 6.3, B = 256 9.6 / 7.2; 2860 x 352, B = 1 10.7 / 6.2; but 12 383 x 768, B = 22 12.7 / 17.5; 5087 x 1984, B = 17 14.5 / 18.7; 2781 x 2496, B = 38 14.7 / 19.2; 8691 x
// 192, B = 57 10.5 / 12.8; 1024 x 768, B = 512 10.4 / 17.3.  Of 1068 16-bit calls of 129 to 60 000 rows and B = 1 to 1024 0.874 times as long on average, 17 longer by
// more than 3 %, 14 % at most (by one line of 95 000 up to 64 queries, 35 000 beyond: 0.878, 62, 70 %).  fp32 0.72 times, 2 and 8 %.
// flat_direct_kernel: one launch, up to 128 rows in one workgroup, which then has them all to bring in: 31 x 928, B = 8 5.8 (scores 6.7), 26 x
// 1760, B = 4 6.8; from some 60 KB (fp32, whose products are longer, 100) scores where the call may use the workspace (more than 64 rows and k > 4).
constexpr int DIRECT_WAVES = 8, DIRECT_ROWS = 16 * DIRECT_WAVES;
inline int direct_held(int d, int elem_bytes) {           // steps of a query in LDS
    const int steps = ((d * elem_bytes + 63) / 64 + 3) & ~3;
    return steps < STREAM_LDS_STEPS ? steps : STREAM_LDS_STEPS;
}
inline size_t direct_lds_bytes(int d, int elem_bytes) {
    const size_t q = (size_t)direct_held(d, elem_bytes) * WAVE * 16, m = 16 * (4 * DIRECT_WAVES * LANE_KP + 4) * CAND_BYTES;
    return q > m ? q : m;
}
inline int64_t score_tiles(int64_t N, int B) { return (N + 15) / 16 * (((int64_t)B + 15) / 16); }
inline bool scores_pay(int64_t N, int row_bytes, int dtype, int B, bool lists) {
    const double most = dtype == ANN_F32 ? 48e3 : lists ? (B > 8 && B <= 16 ? 75e3 : 95e3)
                        : B <= 8 ? 95e3 : B <= 16 ? 60e3 : 35e3;
    return (double)score_tiles(N, B) * sqrt(row_bytes + 256.0) * (1 + (double)N / (100.0 * row_bytes)) <= most;
}
inline bool direct_pays(int64_t N, int row_bytes, int dtype) { return N <= DIRECT_ROWS && N * row_bytes < (dtype == ANN_F32 ? 100 : 60) * 1000; }
// ... or the streaming kernel's one slab, whose scores have the same bits.  It starts quicker where there is hardly a row (7 x 32, B = 2 4.0 / 4.8),
// holds two workgroups a compute unit for many queries (3 x 832 fp32, B = 11 876 25.4 / 37.2), and goes by whole runs of four steps: rows that end inside
// one cost it much.  1048 calls of up to 128 rows, its us / flat_direct_kernel's.  Whole runs: 128 x 128, B = 16 4.95 / 4.38; 16 x 384, B = 64 4.54 / 4.04; but
// 16 x 1536, B = 16 6.67 / 8.41; 128 x 768, B = 1 9.30 / 9.25; fp32 128 x 64, B = 16 6.39 / 5.38, 64 x 384, B = 64 8.13 / 9.83, 128 x 384, B = 64 10.6 / 14.1.
// Others: 17 x 496, B = 1 6.34 / 4.36; 35 x 3944, B = 578 22.5 / 17.0; fp32 18 x 4048, B = 554 70.9 / 62.3, 121 x 272, B = 65 10.0 / 11.4.  By this line 0.924 times as long as the
// streaming kernel on average (the better of both 0.911), eight calls longer by 5 to 9 %; by bytes alone, as for scores, 0.945, 58 longer by up to 26 %.
inline bool direct_quick(int cus, int64_t N, int row_bytes, int dtype, int B) {
    if (N > DIRECT_ROWS || N * row_bytes < 2000 || (B + 15) / 16 > cus) return false;
    if (row_bytes % 256 == 0) return dtype == ANN_F32 ? row_bytes <= 512 && N * row_bytes <= 48000 : row_bytes <= 1024;
    return dtype != ANN_F32 || N <= 64 || row_bytes <= 384 || row_bytes >= 4096;
}

struct FlatPlan {
    bool scores;             // flat_scores_kernel and flat_pick_kernel (w.n scores a query), or
    StreamPlan st;           // streaming kernel with lists, unless
    bool direct;             // ... of one slab: no merge
    bool quick;              // ... by flat_direct_kernel
    bool wide;               // the matrix-core kernel, or
    bool by_fill;            // ... its tile by the first rule
    bool maxima;             // the streaming kernel with group maxima takes the call, `part` queries and `rows` rows at a time
    WidePlan w;
    int part;
    int64_t rows;
    size_t best_ofs;         // rows < N: where the k best so far of every query of a part stand in the workspace
    size_t ws_bytes;
};

constexpr int WIDE_MIN_B = 65;   // smallest batch sent to the matrix-core path
// Workspace that the group maxima of one launch may take; a call that needs more runs one part after the other.
constexpr size_t WIDE_WS_MAX = (size_t)1 << 30;
// A call whose maxima do not fit takes the queries in parts, as long as those are as many as a tile has columns (fp32: as
// keep the products ahead of the reading): every part reads the whole corpus again.  Where fewer would fit, it takes the
// corpus in parts instead, all queries (up to PART_MAX_B) against each, and the k best so far pass from part to part: a
// part costs two launches and a look at its maxima, some 20 us.  8 MiB of maxima, before (queries in parts of 6 to 128) /
// now / at once, ms: 1 M x 768, B = 512 1.76 / 0.96 / 0.88; 21 M x 384, B = 128 62.5 / 3.66 / 3.59, B = 512 344 / 10.3 / 9.45.
constexpr int PART_MIN_B = 256, PART_MIN_B_F32 = 128, PART_MAX_B = 1024;
constexpr int64_t PART_MIN_ROWS = 8192;          // fewer are not worth a launch: the call does not fit

// The loads of 64 bytes of a row that go together; a lane has two such batches in flight.  What decides is how the batches divide the lines of a
// row and what the last one loads for nothing, and with several groups of queries, whose products take longer, that requests come in small portions.
// 16 bits, us, batches of 4 / this:
//   up to 16 queries, rows that end in a sector of 64 bytes or half a line: 3, and 5 where that is the row: 1 M, B = 1 x 264 109 / 101, x 136 62.5 / 56.7, x 160
//     70.9 / 61.5, x 776 310 / 292, x 800 287 / 272, x 1000 387 / 369; 100 k x 616, B = 4 38.2 / 36.5; but 1 M x 104 48.3 / 55.7, x 224 84.4 / 86.2 by 3.
//   more queries, such rows: 5 or 3 where that divides the row: 1 M x 776, B = 48 316 / 300; x 456, B = 32 188 / 180; 3 M x 160, B = 32 212 / 186; 1 M x 264,
//     B = 48 128 / 121; else 4 (1 M x 616, B = 48 251 / 258 by 3).
//   whole lines: two batches of 2 are half the bytes in flight, and a batch ends with its row.  With 17 to 32 queries, whose products cover less, what that
//     costs grows with the row: 1 M x 192, 256, 320, 384, 512, 768, 1024 0.92, 0.93, 0.95, 0.98, 1.01, 1.026, 1.036 times as long by 2, 1.6 M x 128 86 / 91: 2 for 384 to
//     640 bytes (1 M x 256 103 / 95.7).  More queries: 1 M x 448, 512, 768, 1024, B = 48 0.92, 0.95, 0.98, 0.99, B = 64 0.95, 0.96, 0.954, 0.98; 21 M x 384, B = 64, k = 5 2706 / 2657;
//     shorter 3 M x 192 and 320, B = 48 0.93 and 0.945, but x 192, B = 55 1.03, x 256, B = 64 303 / 311: 2 from 768 bytes on.
// fp32, up to 16 queries, whole sectors of 64 bytes, of which batches of 4 load idle ones or split a line between two tiles: 2 where the row is
//   2 or 6 or 10 ... of them (1 M x 96, B = 4 80.6 / 73.5; 100 k x 208, B = 12 27.9 / 25.8; 270 sizes up to x 1024 0.96), an odd number up to 13 (x 80
//     0.94, x 208 0.94; but 3 M x 240 1 / 1.02, 561 k x 752, B = 10 304 / 316), and whole batches of 4 of 8 to 32 sectors, for their smaller portions (x 128 0.945; but
//     131 k x 1024, B = 4 110 / 121, 3.2 M x 64, B = 13 1 / 1.02).  Not 1 M x 300 236 / 256, nor more queries (300 k x 256, B = 40 128 / 136).
inline int stream_batch(int row_bytes, int dtype, int nqg) {
    const int steps = (row_bytes + 63) / 64;
    if (dtype == ANN_F32) {
        if (nqg > 1 || row_bytes % 64 != 0) return 4;
        const bool pays = steps % 4 == 2 || (steps % 2 == 1 ? steps <= 13 : steps >= 8 && steps <= 32);
        return pays ? 2 : 4;
    }
    if (row_bytes % 128 == 0)
        return (nqg >= 3 && row_bytes >= 768) || (nqg == 2 && row_bytes >= 384 && row_bytes <= 640) ? 2 : 4;
    if (steps % 5 == 0 && (nqg > 1 || steps == 5)) return 5;
    if (nqg > 1) return steps % 3 == 0 && steps % 4 != 0 ? 3 : 4;
    return (row_bytes % 64 != 0 && steps >= 9) || (steps + 2) / 3 * 3 <= (steps + 3) / 4 * 4 ? 3 : 4;
}

// The streaming kernel's geometry.
// K: see the kernel; unit: rows that go to a wave together.
inline StreamPlan stream_plan(int cus, int64_t N, int d, int dtype, int B, int K, int unit) {
    StreamPlan pl;
    pl.K = K;
    const int steps = (d * elem_bytes(dtype) + 63) / 64;
    const int fit = STREAM_LDS_STEPS;
    const int n16 = (B + 15) / 16;
    int nqg = fit / steps;
    nqg = nqg < 1 ? 1 : nqg > STREAM_NQG_MAX(elem_bytes(dtype)) ? STREAM_NQG_MAX(elem_bytes(dtype)) : nqg;
    nqg = nqg > n16 ? n16 : nqg;
    pl.lds_steps = steps < fit ? steps : fit;
    // as many queries per workgroup as possible read the corpus least often; fewer when the tiles of 16 rows would not
    // give every compute unit a workgroup of 8 waves
    const int64_t tiles = (N + unit - 1) / unit;
    while (nqg > 1 && tiles * ((n16 + nqg - 1) / nqg) < (int64_t)cus * 8) --nqg;
    pl.G = (n16 + nqg - 1) / nqg;
    pl.nqg = (n16 + pl.G - 1) / pl.G;
    pl.waves = stream_waves(elem_bytes(dtype), pl.nqg, pl.lds_steps);
    pl.batch = stream_batch(d * elem_bytes(dtype), dtype, pl.nqg);
    int occ = (int)(LDS_MAX / stream_lds_bytes(pl.nqg, pl.lds_steps, pl.waves));
    const int most = STREAM_WG_PER_CU(elem_bytes(dtype), pl.nqg, pl.waves);   // measured: more than 2 do not help
    occ = occ < 1 ? 1 : (occ > most ? most : occ);
    // every wave takes whole 16-row tiles in rounds; size the grid so that the last round
    // is as full as the others instead of leaving most of the chip idle
    int64_t cap = (int64_t)cus * occ / pl.G;
    cap = cap < 1 ? 1 : (cap > P_MAX ? P_MAX : cap);
    const int64_t rounds = (tiles + cap * pl.waves - 1) / (cap * pl.waves);
    const int64_t P = (tiles + rounds * pl.waves - 1) / (rounds * pl.waves);
    pl.P = (int)(P < cap ? P : cap);
    return pl;
}

// Maxima of a query, one of 2^g rows: N is a whole number of tiles (wmf > 0), or any number, and there are a multiple of 4.
inline int64_t maxima_of(int wmf, int64_t N, int g) { return wmf > 0 ? N >> g : (((N - 1) >> g) + 1 + 3) & ~(int64_t)3; }

// Whether flat_pick_kernel takes rows of so many bytes in runs of 24 steps (both sides measured there).
inline bool pick_runs(int cus, size_t row_bytes, size_t step_bytes, int B) {
    const size_t steps = row_bytes / step_bytes;
    return steps >= 24 && (B <= 4 * cus || steps >= 72);
}

// Threads of a flat_pick_kernel workgroup: a wave for single rows of a small corpus; else a wave per 32 rows to score and per 4096 maxima, two
// at least; eight only where every query has a compute unit to itself.
inline int pick_threads(int cus, int gs_log, int64_t n, int B, int k) {
    const int rows = k << gs_log;
    if (gs_log == 0 && n <= 2048) return WAVE;
    if (gs_log > 0 && rows <= 64 && n <= 8192) return 2 * WAVE;
    return (rows > 128 || n > 8192) && B <= cus ? 8 * WAVE : 4 * WAVE;
}

// Rows per group of the matrix-core kernel, by the time of what follows the products, in us: 4 bytes of maxima are written in small
// pieces and read again, at 1.6 TB/s over all queries, the rows of k groups are read at 4.5 TB/s; one query alone waits for its maxima (twice,
// 1024 a wave at a time) and, unless groups are single rows, for its rows (32 a wave, 24 steps of 32 bytes at once); and over all queries
// every wave takes its turn on a SIMD, 1.3 us beside its rows.  The constants are fitted to 648 calls of 200 to 3 M rows, 1 to 5000 queries, d = 8 to 2048,
// k = 1 to 16: on average 0.4 % behind the best size of each, 2 % of them by more than 5 %, the worst 20 (without the turns, fitted up to 1000
// queries, 1.2 %, 7 % and 68: 1216 x 848, B = 4933, k = 1 single rows / groups of 4 30.5 / 51.3, 766 x 8, B = 2357, k = 10 11.8 / 16.5).
// fp32 (wmf = 0) writes whole lines and keeps its own constants: 300 k x 128, B = 64 groups of 16 / 32 / 64 rows 78 / 76 / 75, k = 10
// 83 / 83 / 88, B = 300, k = 16 333 / 325 / 346.
// most: maxima of a query that there is room for; the largest groups where no size fits.
inline int wide_group_log(int cus, int wmf, int64_t N, int row_bytes, int B, int k, size_t most) {
    int best = 0;
    double least = INFINITY;
    for (int g : {0, 2, 4, 5, 6}) {
        if (wmf == 0 ? g < 4 : (1 << g) > 16 * wmf) continue;
        if ((size_t)maxima_of(wmf, N, g) > most) { best = g; continue; }
        const double n = (double)N / (1 << g), rows = (double)k * (1 << g), units = ceil(rows / 32);
        double us;
        if (wmf == 0) {
            const int waves = B <= cus ? 8 : 4;           // of a query
            us = 2.0 * n * B / 1e6 + 1.6 * n / (1024 * waves) + rows * row_bytes * B / 4e6 + 1.2 * ceil(rows / (32 * waves)) * ceil(row_bytes / 384.0);
        } else {
            const int waves = pick_threads(cus, g, (int64_t)n, B, k) / WAVE;
            us = 2.5 * n * B / 1e6 + 1.8 * n / (1024 * waves) + 1.3 * waves * B / (4.0 * cus);
            if (g > 0) us += rows * row_bytes * B / 4.5e6 + 2.6 + ceil(units / waves) * (1 + row_bytes / 1280.0) + 0.1 * units * B / (4.0 * cus);
        }
        if (us < least) { least = us; best = g; }
    }
    return best;
}

// The tile of the matrix-core kernel, first rule: the largest of which there are enough for the chip.  Larger tiles move fewer bytes per
// product, so what decides is how full the chip gets; us, d = 768, inputs not in the caches:
//                          256 x 256   512 x 128   256 x 128   128 x 64   64 x 64   (the 128 x 128 tile of half-line stages that
//   4000, B = 400              34          39          25         17         16       stood between them: 20)
//   4000, B = 1000             39          44          30         25         27       28
//   16 k, B = 100 / 256        35 / 39     43 / 44     27 / 28    18 / 26    19 / 29  25 / 27
//   16 k, B = 512              43          47          34         38         44       37
//   50 k, B = 64 / 128         40 / 41     46 / 48     32 / 33    32 / 41    35 / 44  37 / 41
//   50 k, B = 256              43          48          47         55         63       57
//   300 k, B = 128 / 512       149 / 291   132 / 322   112 / 316  143 / 401  -        148 / 365
//   1 M, B = 128 / 512         450 / 887   340 / 976   332 / 984  -          -        441 / 1160
// (The K loop of the last three has lost another 2 to 4 % since.)  Short rows in long slabs keep 512 x 128 (1 M x 384, B = 128: 180 against 187; 1 M x 128 75 / 80; 300 k x 128, B = 400 66 / 72; fewer
// tiles than four for each compute unit: equal at 130 k x 384, B = 400, and 73 against 63 at 300 k x 384, B = 100).  Queries are padded
// to whole tiles; the tiles of 128 queries run at 12/13 of the rate of the other, so they take over where they save more
// than that (1 M x 768, B = 300: 822 -> 745).
// 128 x 64 comes in two forms.  Whole lines of a row of up to 32 elements are half empty, and half lines leave room for three
// workgroups a compute unit, which is one round instead of two where there are tiles for more than two.  Whole / half lines: 3.7 M x 8, B = 6
// 80 / 56; 1.2 M x 24, B = 18 33.9 / 26.0; 1.3 M x 32, B = 54 35.4 / 28.5; 45 k x 8, B = 11 9.5 / 9.1; 35 k x 224, B = 85 16.0 / 14.5, 90 k x 88,
// B = 28 13.3 / 11.8; but 2.7 M x 64, B = 3 79 / 90; 107 k x 384, B = 28 21.9 / 23.7; 23 k x 376, B = 133 18.9 / 19.5.
inline int wide_thin(int cus, int64_t N, int d, int B) {
    const int64_t tiles = (N + WideThin::BM - 1) / WideThin::BM * ((B + WideThin::BN - 1) / WideThin::BN);
    return d <= 32 || (d <= 256 && tiles > 2 * (int64_t)cus && tiles <= 3 * (int64_t)cus) ? WIDE_SHORT : WIDE_THIN;
}
// Stages of a tile by lines, in chunks of 16 bytes: rows begin at multiples of `least` in a line, so 8 - least is the most that comes before them.
inline int wide_lines(int d) {
    const int nch = d / 8, least = (nch | 8) & -(nch | 8);
    return (nch + 8 - least + 7) / 8;
}
// Whether 256 x 128 and 128 x 64 tiles go by the lines of memory that rows lie in (flat_wide_kernel's BY_LINE: same bits): rows that are no whole
// number of lines, of corpora that come from memory.  The selects cost what the requests save where the corpus stays in the caches: us, stages
// of rows / of lines, read again / after others: 80 k x 520, B = 77 30.9 / 31.3, 31.3 / 31.9; 80 k x 776 39.9 / 40.1, 50.7 / 44.8; 123 457 x 776 43.4 / 43.5,
// 56.4 / 51.3; 640 k x 776 242 / 219, 242 / 220; 300 k x 200, B = 40 32.7 / 31.6, 41.8 / 37.3.  Half lines, which fewer requests divide: 123 457 x 800, B = 77
// 41.8 / 43.1, 52.4 / 51.5; 160 k x 800 56.9 / 57.3, 70.7 / 68.3; 1 M x 800, B = 128 387 / 365, 399 / 368; 800 k x 160, B = 77 78.2 / 76.1.  Up to a line
// the stages are mostly first and last ones: 1.5 M x 72, B = 24 63 / 68, 600 k x 120, B = 40 44.5 / 46.6.
// Corpora of less than 256 MiB, the cache in front of the memory, only where that costs nothing when they are read again, as by one call after
// another: no stage more than by rows and one tile of queries, read again 0.985 times as long, after others 0.90 (98 sizes).  With a stage more, read
// again 1.024 times (141 881 x 488, B = 170 54.2 / 59.4, 287 599 x 240, B = 78 39.0 / 42.1), with more tiles, whose rows come from the caches but once, 1.03 to
// 1.05 (136 205 x 688, B = 210 76.6 / 81.6).  From 256 MiB on all gain, read again or not: 0.92.
constexpr int64_t WIDE_BEYOND_CACHES = 1 << 28;
inline bool wide_by_line(int64_t N, int d, int col_tiles) {
    if (d <= 128 || d % 64 == 0) return false;
    if (N * d * 2 >= WIDE_BEYOND_CACHES) return true;
    return N * d * 2 >= 128000000 && d % 32 != 0 && col_tiles == 1 && wide_lines(d) == (d + 63) / 64;
}
inline int wide_shape(int cus, int64_t N, int d, int B) {
    auto tiles = [&](int bm, int bn) { return (N + bm - 1) / bm * ((B + bn - 1) / bn); };
    const int64_t cols256 = (B + 255) / 256 * 256, cols128 = (B + 127) / 128 * 128;
    if (8 * tiles(256, 256) >= 5 * (int64_t)cus && 12 * cols256 <= 13 * cols128) return WIDE_LARGE;
    if (B > 64 && d <= 512 && tiles(512, 128) >= 4 * (int64_t)cus) return WIDE_TALL;
    if (B > 64 && 4 * tiles(256, 128) >= 3 * (int64_t)cus) return WIDE_MID;
    return tiles(128, 64) > cus ? wide_thin(cus, N, d, B) : WIDE_TINY;
}

// Second rule, for batches beyond 64 queries with tiles for more than one round of small ones: by the rounds of tiles that the slowest
// compute unit goes through, since a last round that is nearly empty costs a whole one.  A tile takes a + b (lines of 128 bytes) us
// with the chip full of its kind; where two workgroups share a compute unit and do not fill it, less by `share` of what is missing.  The
// 128 x 128 tile stands between: two fragments each way (a byte read from LDS feeds half as many products again as with 128 x 64) and
// two workgroups to a compute unit, which fill each other's waits, so that two stages do.  Constants fitted to 287 calls of 200 to 2.5 M rows,
// 66 to 8192 queries, d = 72 to 1024: 0.8 % behind the best tile on average (the first rule 3.2 %).  1256 other calls whose tile it changes take 0.938 times as long
// on average, 31 of them longer by more than 2 %, 12.5 % at most (before the lines of wide_tile 0.940, 108, 13.6 %).  First rule / this, us: 977 x 768, B = 5000, k = 16 26.6 / 25.2; 2000 x 768, B = 3000 26.9 / 24.0; 24 k x 768, B = 200 26.2 / 21.9;
// 10.5 k x 768, B = 6152 211 / 195; 46 k x 384, B = 883 72.4 / 66.3; 38.8 k x 776, B = 68 32.9 / 27.4; 110 k x 384, B = 535 82 / 76.
// Corpora beyond 64 MB come from memory, where tiles of few queries read them too often (110 k x 768, B = 301 92 by 256 x 128, 101 by 128 x 128, 105 by
// 128 x 64); rows of up to 64 elements are mostly start and end of a tile (10 k x 64, B = 808 18.7 / 20.7).
inline double wide_rounds_us(int shape, int cus, int64_t N, int d, int B) {
    double a, b, share = 0;
    int lines = 2 * ((d + 63) / 64), bm, bn, per_cu = 1;  // half lines
    auto tile = [&](auto c) {
        bm = decltype(c)::BM;
        bn = decltype(c)::BN;
        per_cu = decltype(c)::PER_CU;
        if (decltype(c)::SB == 64) lines = (d + 31) / 32;
    };
    switch (shape) {
    case WIDE_LARGE: tile(WideLarge{}); a = 1.26; b = 1.35; break;
    case WIDE_TALL: tile(WideTall{}); a = 1.32; b = 1.51; break;
    case WIDE_MID: tile(WideMid{}); a = 0.93; b = 0.69; break;
    case WIDE_SQUARE: tile(WideSquare{}); a = 0.94; b = 0.52; share = 0.40; break;
    default: tile(WideThin{}); a = 0.61; b = 0.43; share = 0.10; break;
    }
    const int64_t slots = (int64_t)cus * per_cu, rows = (N + bm - 1) / bm, cols = (B + bn - 1) / bn;
    const int64_t slabs = slots / cols < 1 ? 1 : slots / cols < rows ? slots / cols : rows, groups = slabs * cols;
    const double rounds = (double)((rows + slabs - 1) / slabs * ((groups + slots - 1) / slots));
    const double full = (double)(groups < slots ? groups : slots) / cus;              // workgroups on a compute unit
    return rounds * (a + b * lines / 2 * (1 + share * (full > 1 ? full - 1 : 0)));
}
inline int wide_tile(int cus, int64_t N, int d, int B, int k) {
    int first = wide_shape(cus, N, d, B);
    // Lines of memory instead of 512 x 128, us: 600 k x 232, B = 77 93.8 / 85.1; 640 k x 456, B = 77 165 / 146; 1 M x 456, B = 128 271 / 248; 1.5 M x 200,
    // B = 128 189 / 182; but 4 M x 184, B = 100 412 / 414, by half lines 2 M x 352, B = 100 344 / 349, and 216, of whose lines a third is not the row,
    // 2.5 M, B = 127 1 / 1.014, 2.2 M, B = 99 1 / 1.024 (800 k, B = 77 1 / 0.96; 232, 240 and 248 2.5 M, B = 127 0.95, 1.002, 0.98).  Corpora of less than 256 MiB,
    // read again: 247 898 x 280, B = 108 38.8 / 42.3, 360 486 x 208, B = 81 45.4 / 48.0.
    const bool apart = d % 32 != 0 && d >= 200 && 10 * (8 * wide_lines(d) - d / 8) <= 24 * wide_lines(d);
    const bool tall = !(apart && N * d * 2 >= WIDE_BEYOND_CACHES);
    if (first == WIDE_TALL && !tall) first = WIDE_MID;
    if (B <= 64 || d <= 64 || first == WIDE_TINY) return first;
    const bool cached = N * d * 2 <= 64000000;
    if (!cached && (first == WIDE_THIN || first == WIDE_SHORT)) return first;
    // (the model takes the half-line tile for the one of whole lines: 38 784 x 96, B = 68 12.9 / 13.8 by 128 x 128, 1025 x 72, B = 4097 21.0 / 21.5, 22 463 x
    // 160, B = 133 3 % longer; from 161 elements on 0.97 times as long)
    if (first == WIDE_SHORT && d <= 160) return first;
    int best = first;
    const double stays = wide_rounds_us(first, cus, N, d, B);
    double least = (cached ? 0.95 : 0.93) * stays;        // (closer than that the model does not tell them apart)
    for (int shape : {WIDE_LARGE, WIDE_TALL, WIDE_MID, WIDE_SQUARE, WIDE_THIN}) {
        if ((!cached && (shape == WIDE_SQUARE || shape == WIDE_THIN)) || (shape == WIDE_TALL && !tall)) continue;
        const double us = wide_rounds_us(shape, cus, N, d, B);
        // (256 x 128 with a half empty last round runs faster in it than the model has it: 15.7 k x 384, B = 839 29.7 / 32.1 by 256 x 256; and the pick of long
        // answers, which the model leaves out, has more to do behind the large tiles: 17.0 k x 128, B = 867, k = 16 24.8 / 28.2 by 512 x 128)
        if (first == WIDE_MID && (shape == WIDE_LARGE || shape == WIDE_TALL) && us > (k > 10 && cached ? 0.84 : shape == WIDE_LARGE ? 0.9 : 1) * stays) continue;
        if (us < least) { least = us; best = shape; }
    }
    return best == WIDE_THIN ? wide_thin(cus, N, d, B) : best;
}

// Whether the matrix-core kernel takes a call, or the streaming kernel, which reads large corpora at the rate of HBM for up to
// 64 queries but sorts lists: some 400 clocks a tile of 16 rows and group of 16 queries, whatever d is.  That shows where
// rows are short or the corpus is in the caches; and a wave takes all columns of its rows, a serial chain where there are
// few rows and many columns.  Streaming / matrix-core, us of a call (k = 3 where nothing else is said; 10 to 11 us are the host's):
//   up to 16 Ki rows (no more 64 x 64 tiles than compute units): long rows 1000 x 768, B = 2 14.8 / 12.3; 4000 x 768 15.2 / 12.3; x 384
//   12.4 / 11.2; 16 k x 768, B = 16 16.7 / 15.0, x 384 14.0 / 12.7; long lists 8000 x 128, k = 16 12.6 / 11.3.  Short rows and lists are
//   level, single-row maxima cost a little more than lists of 4: 6000 x 64, B = 64 11.0 / 12.4; 14 k x 256, B = 16 11.6 / 12.2; but 16 k x 128,
//   B = 40 12.9 / 12.4.
//   queries that do not fit the LDS together, so that the corpus is read twice: 128 k x 1280, B = 48 / 56 77 / 83, 102 / 84; 300 k x 2048,
//   B = 32 / 40 241 / 274, 323 / 275.
//   rows of up to 128 bytes: 64 k x 64, B = 1 13.7 / 11.7; 1 M x 64, B = 1 45 / 38, B = 64 107 / 45; 4 M x 32, B = 8 133 / 96.  (1 M x 96, B = 8
//   48 / 57.)
//   up to 16 queries, at most 480 bytes a row up to 128 Ki rows, 192 up to 512 Ki: 66 k x 112, B = 2 15.6 / 11.7; 55 k x 192, B = 1 17.4 / 13.7;
//   81 k x 160, B = 10 19.1 / 13.2; 97 k x 160, B = 14 20.3 / 14.4; 72 k x 240, B = 6 19.3 / 16.6; 211 k x 96, B = 6 23.8 / 20.2; but 100 k x 248,
//   B = 2 18.1 / 18.9; 112 k x 256, B = 14 18.2 / 19.2; 180 k x 224, B = 12 25.5 / 26.5; 454 k x 128, B = 14 29.7 / 31.1.
//   up to 32 Ki rows: 20 k x 768, B = 16 / 24 16.2 / 18.9, 22.0 / 19.3; x 384, B = 24 16.4 / 16.5; 32 k x 768, B = 48 26 / 24.
//   up to 128 Ki rows, by queries against d: 64 k x 128, B = 16 / 24 13.3 / 13.2, 16.8 / 13.2; 64 k x 768, B = 32 / 48 31 / 33, 36 / 33; 128 k x 256,
//   B = 16 / 24 20.6 / 23.5, 24.8 / 23.7.
//   beyond, by groups of 16 queries: lists cost a row the same whatever its length, and as long again until they are settled; the matrix cores cost more
//   for every element.  So lists are quicker where N (d - r) > q, r elements for what a row costs and q, in millions, for settling; with 17 to 32 queries
//   r = 67.5, q = 65; to 48 82.5, 150; to 64 110, 180.  A row that batches of loads do not divide costs lists about half of what is loaded for nothing
//   (x 192 in batches of 128 elements), and long answers of 0.5 to 1.25 Mi rows cost the matrix cores 2 %, groups of rows scored again (3 to 5 % less beyond
//   4 Mi, which the line leaves out).  Fitted to both kernels at 725 sizes within 0.6 to 1.7 times the line, 131 k to 22 M rows.  Of 7 941
//   pairs of times within 0.6 to 1.45 times of it, corpora below 256 MiB read again too, which moves them to the matrix cores: 1.8 % behind the better
//   of the pair on average (the line by queries 4.2 %), 1.2 % of the pairs more than 5 % longer than by the line by queries, by most for full
//   groups of 17 to 32 queries, which lists take in less time (8.5 M x 72, B = 32 353 / 301; 9.0 M x 72, B = 24 1 / 1.06).  Rows of 768 elements and more keep their lists (341 k x 840, B = 51 141 / 126, 133 k x 960, B = 39
//   69 / 62; from 500 k rows on they are the quicker ones).  us, two, three and four groups: 300 k x 96, B = 20 28.2 / 21.0, x 288, B = 32
//   45.1 / 48.5; 1 M x 128, B = 24 64.7 / 59.9, x 192, B = 32 77.6 / 83.8; 3 M x 128, B = 32 148 / 183; 138 k x 464, B = 44, k = 5 50.5 / 38.7; 1 M x 256, B = 48
//   110 / 117; 1.03 M x 232, B = 45 116 / 124; 4.4 M x 88, B = 41, k = 5 288 / 221; 207 k x 520, B = 45 67.7 / 55.5; 1 M x 320, B = 64 153 / 148, x 384 158 / 171;
//   949 k x 320, B = 53, k = 5 145 / 148; 1.5 M x 256, B = 64 167 / 179; 3.1 M x 192, B = 51, k = 16 323 / 293; 16.8 M x 96, B = 54, k = 5 1036 / 919.
inline bool many_queries(int64_t N, int d, int B) { return B * (N <= 128 * 1024 ? 16 : N <= 512 * 1024 ? 8 : 4) >= d; }
inline bool queries_apart(int d, int B) {                 // 16 bits: they do not fit the LDS together
    const int groups = (B + 15) / 16, steps = (d * 2 + 63) / 64;
    return groups > 1 && groups * steps > STREAM_LDS_STEPS;
}
// 16-bit calls that the line by queries leaves to lists, whichever kernel the line by groups of queries gives them: callers go by the error that a
// buffer too small for lists gives (ann_set_workspace), so it stays where it was.
inline bool lists_must_fit(int64_t N, int d, int B) {
    return B > 16 && B < WIDE_MIN_B && N > 128 * 1024 && d > 64 && !queries_apart(d, B) && !many_queries(N, d, B);
}
inline bool wide_beats_lists(int64_t N, int d, int B, int k) {
    const int groups = (B + 15) / 16, steps = (d * 2 + 63) / 64, batch = stream_batch(d * 2, ANN_F16, groups);
    const double r = groups <= 2 ? 67.5 : groups == 3 ? 82.5 : 110, q = groups <= 2 ? 65e6 : groups == 3 ? 150e6 : 180e6;
    const double answers = k > 4 && N > 512 * 1024 && N <= 1280 * 1024 ? 0.96 : 1;
    const int idle = ((steps + batch - 1) / batch * batch - steps) * 32;           // elements loaded for nothing
    return d < 768 && d - 0.5 * idle <= answers * (r + q / (double)N);
}
inline bool use_wide(int64_t N, int d, int dtype, int B, int k) {
    if (dtype == ANN_F32) return false;
    if (B >= WIDE_MIN_B) return true;
    if (N <= 16 * 1024) return k > 4 || d >= 384 || (N > 6000 && B > 32);
    if (d <= 64 || queries_apart(d, B)) return true;
    if (N <= 32 * 1024) return B > 32 || (B > 16 && d >= 768);
    if (B <= 16) return N <= 128 * 1024 ? d <= 240 : N <= 512 * 1024 && d <= 96;
    return N <= 128 * 1024 ? many_queries(N, d, B) : wide_beats_lists(N, d, B, k);
}

// fp32 keeps lists for up to 16 queries (HBM-bound on large corpora) and wherever picking costs more than the lists: the rows
// of k groups (10 k d rows of scoring they are worth) and the launch-bound sizes.  Lists / maxima, us: 250 k x 64, B = 1000
// 787 / 453; 1 M x 196, B = 100 818 / 666; 64 k x 384, B = 300 194 / 185; 16 k x 384, B = 1000, k = 16 164 / 208.
inline bool use_f32_maxima(int64_t N, int d, int B, int k) {
    return B > 16 && N >= (int64_t)10 * k * d && N * B >= (int64_t)32768 * d;
}

// One pass of pl.part queries over pl.rows rows by a kernel that leaves group maxima; `room` bytes for them if that can be.
inline size_t maxima_pass(FlatPlan &pl, int cus, int d, int dtype, int k, size_t room) {
    const int64_t N = pl.rows;
    const int B = pl.part;
    const size_t most = room / ((size_t)B * sizeof(float));
    if (pl.wide) {
        wide_geometry(pl.w, pl.by_fill ? wide_shape(cus, N, d, B) : wide_tile(cus, N, d, B, k), cus, N, B);
        // A tile's groups have 16 wmf rows at most: where those are too many, the tile of 64 if there are enough for the chip,
        // else the one of 32 that pads least (300 k x 64, B = 300 in 1 MiB: 7 parts of the corpus, 14 by groups of 32).
        if (pl.w.wmf < 4 && (size_t)maxima_of(pl.w.wmf, pl.w.slots, 3 + pl.w.wmf) > most) {
            if (8 * ((N + WideTall::BM - 1) / WideTall::BM) * ((B + WideTall::BN - 1) / WideTall::BN) >= 5 * (int64_t)cus)
                wide_geometry(pl.w, WIDE_TALL, cus, N, B);
            else wide_geometry(pl.w, wide_thin(cus, N, d, B), cus, N, B);
        }
        pl.w.gs_log = wide_group_log(cus, pl.w.wmf, pl.w.slots, d * 2, B, k, most);
        pl.w.n = maxima_of(pl.w.wmf, pl.w.slots, pl.w.gs_log);
    } else {
        pl.w.cus = cus;
        pl.w.gs_log = wide_group_log(cus, 0, N, d * 4, B, k, most);
        pl.w.n = maxima_of(0, N, pl.w.gs_log);
        pl.st = stream_plan(cus, N, d, dtype, B, 1 << (pl.w.gs_log - 4), 1 << pl.w.gs_log);
    }
    return (size_t)B * (size_t)pl.w.n * sizeof(float);
}
// The same for the last part of a call, which may be smaller: same kernel, same groups.
inline FlatPlan maxima_part(FlatPlan pl, int64_t rows, int part, int d, int dtype) {
    if (rows == pl.rows && part == pl.part) return pl;
    pl.rows = rows;
    pl.part = part;
    if (pl.wide) {
        wide_geometry(pl.w, pl.w.shape, pl.w.cus, rows, part);
        pl.w.n = maxima_of(pl.w.wmf, pl.w.slots, pl.w.gs_log);
    } else {
        pl.w.n = maxima_of(0, rows, pl.w.gs_log);
        pl.st = stream_plan(pl.w.cus, rows, d, dtype, part, 1 << (pl.w.gs_log - 4), 1 << pl.w.gs_log);
    }
    return pl;
}
// A call on group maxima in `limit` bytes of workspace; false if it does not fit (pl.ws_bytes: what one pass would take).
inline bool maxima_plan(FlatPlan &pl, int cus, int64_t N, int d, int dtype, int B, int k, size_t limit) {
    pl.rows = N;
    pl.part = B;
    const bool by_fill = pl.by_fill || !pl.wide;
    pl.by_fill = true;
    const size_t all = pl.ws_bytes = maxima_pass(pl, cus, d, dtype, k, limit);
    // The tile that takes the fewest rounds, if its maxima fit at once: what must go in parts keeps the first rule, which the lines of small
    // buffers were drawn with.  (No less is asked for than the first rule's tile needs: what ann_flat_workspace_bytes of 8 MiB at
    // most says of the static entry point stays true.)
    if (!by_fill) {
        FlatPlan own = pl;
        own.by_fill = false;
        const size_t bytes = maxima_pass(own, cus, d, dtype, k, limit);
        if (bytes <= limit) {
            own.ws_bytes = all <= limit && all > bytes ? all : bytes;
            pl = own;
            return true;
        }
    }
    if (all <= limit) return true;
    // queries in parts
    const size_t fit = limit / ((size_t)pl.w.n * sizeof(float));
    if (fit >= (size_t)(pl.wide ? PART_MIN_B : PART_MIN_B_F32)) {
        const int parts = (int)((B + fit - 1) / fit);
        pl.part = (B + parts - 1) / parts;
        if (pl.part > 256 && (size_t)((pl.part + 255) & ~255) <= fit) pl.part = (pl.part + 255) & ~255;
        while ((pl.ws_bytes = maxima_pass(pl, cus, d, dtype, k, limit)) > limit) --pl.part;   // (another tile, a few groups more)
        return true;
    }
    // the corpus in parts: whole rounds of the tiles, or as many rows as fit
    for (pl.part = B < PART_MAX_B ? B : PART_MAX_B; pl.part >= 1; pl.part /= 2) {
        const size_t best = (size_t)pl.part * k * sizeof(uint64_t);
        if (best >= limit) continue;
        const size_t room = limit - best;
        pl.rows = (int64_t)(room / ((size_t)pl.part * sizeof(float))) << 6;
        while (pl.rows >= PART_MIN_ROWS) {
            pl.rows = pl.rows < N ? pl.rows : N;
            const int64_t have = pl.rows;
            maxima_pass(pl, cus, d, dtype, k, room);
            const int64_t round = pl.wide ? (int64_t)pl.w.P * wide_rows(pl.w.shape) : (int64_t)pl.st.P * pl.st.waves << pl.w.gs_log;
            if (pl.rows < N) pl.rows -= pl.rows >= round ? pl.rows % round : pl.rows % 512;
            const size_t bytes = maxima_pass(pl, cus, d, dtype, k, room);
            if (bytes <= room) {
                pl.best_ofs = (bytes + 7) & ~(size_t)7;
                pl.ws_bytes = pl.best_ofs + best;
                if (pl.ws_bytes <= limit) return true;
            }
            pl.rows = have / 2;                           // (groups of the tile that so few rows get are smaller)
        }
    }
    pl.rows = N;
    pl.part = B;
    pl.ws_bytes = all;
    return false;
}

// A call on lists.
inline void lists_plan(FlatPlan &pl, int cus, int64_t N, int d, int dtype, int B, int k, size_t limit) {
    pl.st = stream_plan(cus, N, d, dtype, B, (k + 3) & ~3, 16);
    if (pl.direct) {
        pl.st.P = 1;
        pl.st.batch = 4;
        return;
    }
    // lists that do not fit: fewer slabs, down to a quarter of those that fill the chip
    const size_t slab = (size_t)B * pl.st.K * CAND_BYTES, fit = limit / slab;
    if (fit < (size_t)pl.st.P && fit >= 1 && 4 * fit >= (size_t)pl.st.P) pl.st.P = (int)fit;
    pl.ws_bytes = slab * pl.st.P;
}

// A call of up to 64 queries whose maxima do not fit at once: the matrix-core kernel in parts, or lists in one pass, whichever takes
// less, in us.  A part costs 8 us beside the rows of its k groups, and its tiles go in rounds of one for every compute unit;
// lists read the corpus more than once where the queries do not fit the LDS together, cost more with every group of 16
// queries, and have too few workgroups where their slabs are cut.  Fitted to 220 calls of 20 k to 20 M rows, d = 8 to 4096, in 16 KB to
// 8 MiB: 1 % behind the better side on average (always in parts 12 %, always lists 74 %), half again as long at worst.  Lists / parts:
// 1 M x 128, B = 64 in 1 MiB 107 / 146; 16 M x 64, B = 32 in 1 MiB 486 / 905; 1.9 M x 24, B = 4 in 85 KB 61 / 96; but 4 M x 64, B = 64 in
// 8 MiB 301 / 144; 16 M x 8, B = 1 in 63 KB 436 / 286; 1.6 M x 1600, B = 57 in 123 KB 4354 / 2649.
inline double parts_us(const FlatPlan &pl, int64_t N, int d, int B, int k) {
    const int64_t parts = (N + pl.rows - 1) / pl.rows;
    const double round = (double)pl.w.cus * wide_rows(pl.w.shape), row = ceil(d / 32.0) * 64 / 6.1e6;
    const double rounds = (parts - 1) * ceil(pl.rows / round) + ceil((N - (parts - 1) * pl.rows) / round) + 0.3 * parts;
    const double pick = (double)(k << pl.w.gs_log) * d * 2 * pl.part / 4e6;
    return (B + pl.part - 1) / pl.part * (parts * (8 + pick) + 1.1 * rounds * round * row);
}
inline double lists_us(const FlatPlan &pl, int cus, int64_t N, int d, int dtype, int B, int k) {
    FlatPlan whole{};
    lists_plan(whole, cus, N, d, dtype, B, k, SIZE_MAX);
    const double all = (double)whole.st.P * whole.st.G, wgs = (double)pl.st.P * pl.st.G, groups = (B + 15) / 16, rows = N * 1e-6;
    const double cut = wgs >= cus ? 1 + 0.3 * (all / wgs - 1) : (1 + 0.3 * (fmax(all / cus, 1.0) - 1)) * fmin(all, cus) / wgs;
    const double read = (0.45 + 0.6 * pl.st.G) * rows * d * 2 / 6.1 * cut;
    return fmax(read, rows * (24 + 3 * groups) * cut + groups * fmin(35, 2 + 8 * rows)) + 10;
}

// by_fill: the tile by the first rule (the static entry point, whose lines were drawn with it).
// in_parts: a call keeps its kernel, and its bits, where that takes parts (the static entry point, whose workspace is of one size).
inline FlatPlan flat_plan(int cus, int64_t N, int d, int dtype, int B, int k, size_t limit, bool in_parts = false, bool by_fill = false) {
    FlatPlan pl{};
    pl.by_fill = by_fill;
    pl.part = B;
    pl.rows = N;
    const int row_bytes = d * elem_bytes(dtype);
    const size_t scores = (size_t)B * (size_t)((N + 3) & ~(int64_t)3) * sizeof(float);
    const bool few = scores_pay(N, row_bytes, dtype, B, !use_wide(N, d, dtype, B, k)), one = direct_pays(N, row_bytes, dtype);
    // So few rows never need a workspace, whatever their length and the batch: such searches may overlap anything, and each other.
    const bool none = N <= (k <= 4 || dtype == ANN_F32 ? DIRECT_ROWS : DIRECT_ROWS / 2);
    pl.scores = few && !none && !one && scores <= limit;
    if (pl.scores) {
        pl.w.cus = cus;
        pl.w.n = (N + 3) & ~(int64_t)3;
        pl.ws_bytes = scores;
        return pl;
    }
    // A corpus of one tile per wave of a workgroup: its lists are the answer, one launch instead of two (64 x 1024, B = 8192, k = 16 23.1 -> 17.3 us).
    // Lists of 4 per lane are complete there whatever k is, since a lane sees four rows; selecting k > 4 from all eight
    // waves costs more than the launch saves where the other way is group maxima (128 x 1024 bf16, B = 5000, k = 16: 19.3 / 23.3).
    pl.direct = none || (few && N <= DIRECT_ROWS);
    pl.quick = pl.direct && direct_quick(cus, N, row_bytes, dtype, B);
    pl.maxima = !pl.direct && dtype == ANN_F32 && use_f32_maxima(N, d, B, k);
    pl.wide = !pl.direct && use_wide(N, d, dtype, B, k);
    if (pl.wide && !in_parts && lists_must_fit(N, d, B)) {
        FlatPlan lists{};
        lists.part = B;
        lists.rows = N;
        lists_plan(lists, cus, N, d, dtype, B, k, limit);
        if (lists.ws_bytes > limit) return lists;
    }
    auto plan = [&] {
        if (pl.wide || pl.maxima) maxima_plan(pl, cus, N, d, dtype, B, k, limit);
        else lists_plan(pl, cus, N, d, dtype, B, k, limit);
    };
    plan();
    const bool fits = pl.ws_bytes <= limit;
    if (dtype == ANN_F32 || B >= WIDE_MIN_B || (fits && (!pl.wide || in_parts || (pl.rows == N && pl.part == B)))) return pl;
    // The other kernel, if its workspace fits: where the first has none (lists of less than a quarter of their slabs: only for many
    // queries), or would need parts that take longer than lists.  Where neither fits ws_bytes says so.
    if (!pl.wide && (pl.direct || N <= 32 * 1024 || !many_queries(N, d, B))) return pl;
    const FlatPlan first = pl;
    pl = FlatPlan{};
    pl.by_fill = by_fill;
    pl.part = B;
    pl.rows = N;
    pl.wide = !first.wide;
    plan();
    if (pl.ws_bytes > limit || (fits && lists_us(pl, cus, N, d, dtype, B, k) >= parts_us(first, N, d, B, k))) return first;
    return pl;
}

// Long answers of large batches that the static workspace takes though one pass does not fit it.  They once needed a list of 16
// pairs per slab or a candidate array per query; callers go by the error that the latter gave, so the line stays where it was
// (for a 16-bit corpus of over 32 Ki rows, where slabs depended on d, at the fewest there were).
inline bool static_takes_long(int64_t N, int d, int dtype, int B) {
    if (dtype != ANN_F32 && (d % 32 == 0 || N >= 128 * 1024)) return false;
    const int64_t rows = dtype == ANN_F32 ? 32 : 128, most = dtype == ANN_F32 ? 1024 : 128, slabs = (N + rows - 1) / rows;
    return (slabs < most ? slabs : most) * B * 16 * (int64_t)CAND_BYTES <= ANN_STATIC_WORKSPACE_BYTES;
}
// ... and the line of one pass: that of the call's tile, of the one that pads least, and where tiles of 512 x 128 would do, of their larger
// groups.  (The group sizes are those of earlier constants, which the line was drawn by, and not those that the call gets.)
inline int static_group_log(int cus, int wmf, int64_t N, int row_bytes, int B, int k) {
    const int waves = B <= cus ? 8 : 4;
    int best = 0;
    double least = INFINITY;
    for (int g : {0, 2, 4, 5, 6}) {
        if ((1 << g) > 16 * wmf) continue;
        if ((size_t)maxima_of(wmf, N, g) > WIDE_WS_MAX / ((size_t)B * sizeof(float))) { best = g; continue; }
        const double n = (double)N / (1 << g), rows = (double)k * (1 << g);
        double us = 3.0 * n * B / 1e6 + 1.2 * n / (1024 * waves);
        if (g > 0) us += rows * row_bytes * B / 5e6 + 3.5 + 0.4 * ceil(rows / (32 * waves)) * ceil(row_bytes / 768.0);
        if (us < least) { least = us; best = g; }
    }
    return best;
}
inline bool static_one_pass(const WidePlan &w, int64_t N, int d, int B, int k) {
    const int log = static_group_log(w.cus, w.wmf, w.slots, d * 2, B, k);
    int64_t n = maxima_of(1, (N + 63) / 64 * 64, log);
    const int64_t own = maxima_of(w.wmf, w.slots, log), tall = (N + 511) / 512;
    n = own < n ? own : n;
    if (w.shape == WIDE_MID && 8 * tall * ((B + 127) / 128) >= 5 * (int64_t)w.cus) {
        const int64_t g = maxima_of(4, tall * 512, static_group_log(w.cus, 4, tall * 512, d * 2, B, k));
        n = g < n ? g : n;
    }
    return (size_t)B * (size_t)n * sizeof(float) <= (size_t)ANN_STATIC_WORKSPACE_BYTES;
}
// The plan of a call on the static workspace of `bytes` bytes, ANN_STATIC_WORKSPACE_BYTES and room for the best so far behind
// them; ws_bytes > bytes: refused.
inline FlatPlan static_plan(int cus, int64_t N, int d, int dtype, int B, int k, size_t bytes) {
    if (k > 4 && B >= 256 && !static_takes_long(N, d, dtype, B)) {
        FlatPlan pl = flat_plan(cus, N, d, dtype, B, k, WIDE_WS_MAX, false, true);
        if (pl.wide && pl.ws_bytes > (size_t)ANN_STATIC_WORKSPACE_BYTES && static_one_pass(pl.w, N, d, B, k))
            pl = flat_plan(cus, N, d, dtype, B, k, ANN_STATIC_WORKSPACE_BYTES, false, true);
        if (pl.ws_bytes > (size_t)ANN_STATIC_WORKSPACE_BYTES && pl.ws_bytes <= bytes) pl.ws_bytes = bytes + 1;
        return pl;
    }
    return flat_plan(cus, N, d, dtype, B, k, bytes, true, true);
}

// ---- graph search ---------------------------------------------------------------------------------------
constexpr int GRAPH_THREADS = 256;
constexpr int GRAPH_WAVES = GRAPH_THREADS / WAVE;
constexpr int LANES_PER_ROW = 8;
constexpr int ROWS_PER_PASS = GRAPH_THREADS / LANES_PER_ROW;   // 32 neighbours scored at once
constexpr int RMAX_LDS = 256;                                  // row stride of the read-ahead buffers (>= R)

constexpr int GRAPH_DENSE_MIN_B = 1280;   // batches beyond this run three graph-search workgroups per compute unit
constexpr int GRAPH_EF_DOUBLE = 2048;    // candidate lists up to this length are double-buffered in LDS
constexpr int GRAPH_EF_TWO_LEVEL = 512;  // beyond this, graphs of at most 32 slots per node use the two-level list
struct GraphLds {
    // byte offsets into dynamic LDS; all 16-byte aligned
    uint32_t q, ls0, ls1, li0, li1, cs, ci, cpos, cache, ctl, adj, um, rq, co, total;
    uint32_t cache_bits, rp;
    // two-level list (search ranges beyond GRAPH_EF_TWO_LEVEL on graphs of at most 32 slots per node):
    // ms / mi hold the large part of the list, ls0 .. li1 the small part (GRAPH_DELTA entries each)
    uint32_t two_level, ms, mi;
};
constexpr int GRAPH_DELTA = 256;
// The two-level layout keeps its small regions at fixed byte offsets at the start of LDS (the kernel
// then addresses them with immediates and needs no register per region); the large part of the
// list and the query, whose sizes depend on ef and d, follow.
constexpr uint32_t TL_LS0 = 0, TL_LI0 = 4 * GRAPH_DELTA, TL_LS1 = 8 * GRAPH_DELTA, TL_LI1 = 12 * GRAPH_DELTA;
constexpr uint32_t TL_CS = 16 * GRAPH_DELTA, TL_CI = TL_CS + 128, TL_CPOS = TL_CI + 128, TL_CTL = TL_CPOS + 128;
constexpr uint32_t TL_ADJ = TL_CTL + 32, TL_UM = TL_ADJ + 256;
constexpr uint32_t TL_MS = TL_UM + 8 * (16384 / 64) + 32;   // um: a bit per entry of the longest list, and 4 words
// words of one query's visited bitset: one bit per node, rounded to 64-byte units
inline int64_t visited_words(int64_t N) { return (N + 511) / 512 * 16; }

// graph_step_kernel (graphs of at most 32 slots per node, lists of up to GRAPH_EF_TWO_LEVEL entries): how it runs a call, and its LDS
constexpr int GRAPH_STEP_MAX_R = 32;
struct StepLds {
    // fixed byte offsets: scores, ids, positions, numbers of a step's neighbours (64 each), marks, then the scratch of every wave
    static constexpr uint32_t CS = 0, CI = 256, CP = 512, EV = 768, EW = 1024, FM = 1280, MK = 1312, WAVE0 = 1440, WAVE_BYTES = 96;
    // byte offsets: list scores and ids (two buffers of ls_bytes each), id cache, query
    uint32_t ls, li, ls_bytes, vis, q, total;
    int vis_words, cache_shift;                           // of the id cache
    int rows_per_group;                                   // neighbours a row group scores in a step: 1 or 2
    bool dense;                                           // three workgroups per compute unit, query read from LDS
};

inline GraphLds graph_lds_layout(int d, int elem_bytes, int R, int ef) {
    auto up = [](uint32_t x) { return (x + 15u) & ~15u; };
    const bool inplace = ef > GRAPH_EF_DOUBLE;           // long lists: one buffer, merged in place
    auto lay = [&](uint32_t bits) {
        GraphLds L{};
        uint32_t off = 0;
        L.rp = (uint32_t)((R + ROWS_PER_PASS - 1) / ROWS_PER_PASS * ROWS_PER_PASS);
        L.cache_bits = bits;
        L.q = off; off = up(off + (uint32_t)d * elem_bytes);
        // score lists are padded to 64 entries; lists of up to 256 entries get buffers of 256, which
        // the scan for the next unexpanded entry then reads without conditions
        const uint32_t ef64 = ef <= GRAPH_DELTA ? (uint32_t)GRAPH_DELTA : ((uint32_t)ef + 63u) & ~63u;
        const uint32_t efi = ef <= GRAPH_DELTA ? (uint32_t)GRAPH_DELTA : (uint32_t)ef;
        L.ls0 = off; off = up(off + 4u * ef64);
        if (inplace) L.ls1 = L.ls0; else { L.ls1 = off; off = up(off + 4u * ef64); }
        L.li0 = off; off = up(off + 4u * efi);
        if (inplace) L.li1 = L.li0; else { L.li1 = off; off = up(off + 4u * efi); }
        L.cs = off; off = up(off + 4u * L.rp);
        L.ci = off; off = up(off + 4u * L.rp);
        L.cpos = off; off = up(off + 4u * L.rp);
        L.cache = off; off = up(off + (4u << bits));
        L.ctl = off; off = up(off + 16u);
        L.adj = off; off = up(off + 2u * 4u * RMAX_LDS);
        L.um = off; off = up(off + 8u * (((uint32_t)ef + 63u) / 64u) + 32u);   // the scans use um[0 .. 3] at any ef
        L.rq = off; off = up(off + 4u * L.rp);
        L.co = off; off = up(off + 4u * L.rp);
        L.total = off;
        return L;
    };
    // Long lists on graphs of at most 32 slots per node: the two-level list.  The large part has one
    // buffer of ef entries, the small part two of GRAPH_DELTA; the adjacency rows read ahead take 32
    // slots each; the words of um double as the position marks of a rebuild; there is no id cache.
    auto lay2 = [&] {
        GraphLds L{};
        L.rp = ROWS_PER_PASS;
        L.cache_bits = 0;                                  // no id cache: the visited set is asked first
        L.two_level = 1;
        L.ls0 = TL_LS0; L.li0 = TL_LI0; L.ls1 = TL_LS1; L.li1 = TL_LI1;
        L.cs = TL_CS; L.ci = TL_CI; L.cpos = TL_CPOS;
        L.ctl = L.cache = TL_CTL;
        L.adj = TL_ADJ;
        L.um = L.rq = L.co = TL_UM;                        // (rq, co: used by the plain loop only)
        L.ms = TL_MS;
        L.mi = up(L.ms + 4u * (uint32_t)ef);
        L.q = up(L.mi + 4u * (uint32_t)ef);
        L.total = up(L.q + (uint32_t)d * elem_bytes);
        return L;
    };
    // (it is the only layout of such lists on such graphs: the software-pipelined loop has no code for
    // a single list of more than 512 entries; with d <= ANN_D_MAX it always fits)
    if (ef > GRAPH_EF_TWO_LEVEL && R <= ROWS_PER_PASS) return lay2();
    // cache slots: a few times the number of nodes a search scores (about 10 ef), at most 2^14;
    // fewer when that lets two workgroups share a compute unit, or when the list needs the room
    uint32_t want = 10;
    while ((1u << want) < 32u * (uint32_t)ef && want < 14) ++want;
    uint32_t bits = want;
    if (lay(11).total <= LDS_MAX / 2)
        while (bits > 11 && lay(bits).total > LDS_MAX / 2) --bits;
    while (bits > 10 && lay(bits).total > LDS_MAX) --bits;
    return lay(bits);
}

inline StepLds graph_step_plan(int cus, int d, int elem_bytes, int B, int ef) {
    auto up = [](uint32_t x) { return (x + 15u) & ~15u; };
    StepLds L{};
    L.rows_per_group = B <= cus ? 2 : 1;
    const uint32_t entries = ef <= GRAPH_DELTA ? (uint32_t)GRAPH_DELTA : ((uint32_t)ef + 63u) & ~63u;
    uint32_t off = up(StepLds::WAVE0 + GRAPH_WAVES * StepLds::WAVE_BYTES);
    L.ls_bytes = 4u * entries;
    L.ls = off; off = up(off + 2u * L.ls_bytes);
    L.li = off; off = up(off + 2u * L.ls_bytes);
    L.q = off; off = up(off + (uint32_t)d * elem_bytes);
    L.vis = off;
    // id cache: a few times the number of nodes a search scores (about 10 ef)
    int bits = 10;
    while ((1u << bits) < 32u * (uint32_t)ef && bits < 13) ++bits;
    L.vis_words = 1 << bits;
    L.cache_shift = 32 - bits;
    L.total = up(off + 4u * (uint32_t)L.vis_words);
    // More queries than two workgroups per compute unit hold at once, and a layout small enough for three: the form
    // that reads the query from LDS and runs three per compute unit.
    L.dense = B > GRAPH_DENSE_MIN_B && 3 * (size_t)L.total <= LDS_MAX;
    return L;
}

// graph_frontier_kernel (graphs of at most 32 slots per node)
constexpr int FRONTIER_MOST = 63;                         // most neighbours a step scores
constexpr int FRONTIER_VIS_LDS = 0, FRONTIER_VIS_GLOBAL = 1;              // where the visited set is
constexpr int FRONTIER_SPARE = 512, FRONTIER_SPARE_MIN = 280, FRONTIER_SPARE_TIGHT = 124;   // places beyond ef, at least; where room is what counts; tight
// Whether a step of graph_frontier_kernel touches the adjacency rows of the queue's next nodes ahead.  Of eight waves the last one, which does so, seldom
// has a row to score: without, 200 k x 768 fp16, R = 32, B = 1, ef = 64, 256, 512, 1024, 2048 3.0, 3.3, 4.2, 5.5, 6.8 % longer (six queries each), B = 256, ef = 128,
// 512, 2048 3.2, 4.4, 6.3 %, 200 k x 256, B = 32 4.0, 5.1, 7.9 %.  Two workgroups of four waves keep the memory path busy with rows: with / without, us,
// 200 k x 768, R = 32, B = 512, ef = 256 710 / 702 and 693 / 677, 200 k x 384, B = 1000, ef = 200 784 / 779 and 818 / 803.
constexpr bool frontier_ahead(int waves) { return waves == 8; }

struct FrontierLds {
    // fixed byte offsets: keys of a step's neighbours (twice), a place to order them in, where they are by hash (twice), counts of
    // the waves, then the scratch of every wave
    static constexpr int HASH_BITS = 7, HASHES = 1 << HASH_BITS;
    static constexpr uint32_t CK = 0, SORTED = 1024, HASH = 1536, CTL = HASH + 8 * HASHES, WAVES = CTL + 80, WAVE_BYTES = 544;
    // byte offsets: expanded nodes and pool, visited bits, query
    uint32_t keys, vis, q, total;
    int cap, spare, vis_words, vis_mode;                  // places of the array; how many above ef a bound may leave in it
    int waves, width, per_cu;                             // variant: waves of a workgroup, expansions a step tries, workgroups per compute unit
    bool tight;                                           // ... that keeps no places for the queue's end
};
// A query has a compute unit to itself: 8 waves, which score all neighbours of a step at once.  More queries: 4 waves, two
// workgroups to a compute unit; beyond what these hold at once three, with the query read from LDS.  200 k x 768, R = 32, ef = 192, us,
// one / two / three workgroups: B = 256 427 / 605 / -; 512 794 / 662 / 720; 1024 1424 / 1206 / 1071.  (Three where little room is left
// for the array find bounds all the time: 1 M x 768, B = 1024, ef = 4096 18.8 ms by two, 20.3 by three.)
// width: trying 8 expansions instead of 4 costs a step some 500 clocks and pays where steps commit more than three: where a
// search covers most of its graph (200 k x 768, B = 256, ef = 2048 2480 / 2580 us with 4 / 8; 60 k x 384, ef = 4096 3240 / 2770), and
// with the maturity exit, which most queries leave while nearly every expansion stands (200 k x 384 bf16, B = 256, ef = 256, the kernel as first built, 312 / 257).
inline bool frontier_layout(int64_t N, int d, int elem_bytes, int ef, int waves, int per_cu, int width, int spare_min, FrontierLds &L) {
    auto up = [](uint32_t x) { return (x + 15u) & ~15u; };
    L = FrontierLds{};
    L.waves = waves;
    L.per_cu = per_cu;
    L.width = width;
    const int64_t room = (int64_t)(LDS_MAX / per_cu) & ~15, words = visited_words(N);
    uint32_t off = up(FrontierLds::WAVES + waves * FrontierLds::WAVE_BYTES);
    L.q = off; off = up(off + (uint32_t)d * elem_bytes);
    L.vis = off;
    if (off + words * 4 + 8 * ((int64_t)ef + spare_min) <= room) {
        L.vis_mode = FRONTIER_VIS_LDS;
        L.vis_words = (int)words;
    } else {
        L.vis_mode = FRONTIER_VIS_GLOBAL;
    }
    off = up(off + 4u * (uint32_t)L.vis_words);
    L.keys = off;
    // The more places beyond ef, the rarer a bound has to be found; all that a search of a short list scores fits.
    int64_t spare = ef / 2 < 1536 ? 1536 : ef / 2 > 4096 ? 4096 : ef / 2;
    const int64_t fit = (room - off) / 8 - ef;
    if (spare > fit) spare = fit < spare_min ? spare_min : fit;
    L.cap = ef + (int)spare;
    L.tight = spare < FRONTIER_SPARE_MIN;
    L.spare = L.tight ? ((int)spare - 72) / 2 : (int)spare / 2 - 136;     // (a bound leaves room for a step and more: see the kernel)
    L.total = up(off + 8u * (uint32_t)L.cap);
    return (int64_t)L.total <= room;
}
inline FrontierLds frontier_plan(int cus, int64_t N, int d, int elem_bytes, int B, int ef, bool exits) {
    const int width = exits || 32 * (int64_t)ef >= N ? 8 : 4;
    auto lay = [&](int waves, int per_cu, FrontierLds &L) {
        return frontier_layout(N, d, elem_bytes, ef, waves, per_cu, width, per_cu == 3 ? 2 * FRONTIER_SPARE : FRONTIER_SPARE, L);
    };
    FrontierLds L;
    if (B > 2 * cus && lay(4, 3, L)) return L;
    if (B > cus && lay(4, 2, L)) return L;
    lay(8, 1, L);
    return L;
}
// The layout that finds room for the visited set in LDS on the largest graphs; false: too large.  (Lists of up to 512 entries left
// more room when they were written out: with counters, so that the same calls need no workspace, a tight array will do.)
inline bool frontier_in_lds(int64_t N, int d, int elem_bytes, int R, int ef, bool counters, FrontierLds &L) {
    auto fits = [&](int spare_min) { return frontier_layout(N, d, elem_bytes, ef, 4, 1, 8, spare_min, L) && L.vis_mode == FRONTIER_VIS_LDS; };
    return R <= GRAPH_STEP_MAX_R && (fits(FRONTIER_SPARE_MIN) || (counters && fits(FRONTIER_SPARE_TIGHT)));
}

// Whether most queries of a search with the maturity exit leave by it.  An average that moves by alpha a sample passes tau after about
// -log(1 - tau) / alpha samples of 1; a search that runs to its end scores up to ef R nodes, and relative qualities beyond 1 shorten the way.  Early
// exits of 450 random calls against samples / (ef R): up to 1 76 to 91 %, 1 to 3 63 %, beyond 3 20 %.
inline bool exit_likely(float tau, float alpha, int R, int ef) { return tau < 1.0f && -logf(1.0f - tau) < 3.0f * ef * R * alpha; }

// Maturity exit: the shortest list that graph_frontier_kernel takes.  Lines drawn through 9260 calls (20 k to 2.5 M nodes, rows of 128 bytes to 4 KB,
// R = 8 to 32, B = 1 to 2000, ef = 8 to 2048), both kernels timed for each.  Time above the better of the two, on average, by these lines / by
// graph_search_kernel alone, in %: queries that leave B = 2 to 8 6 / 31, 9 to 256 0.4 / 68, 257 to 512 0.2 / 60, 513 to 768 0.1 / 67, more 0.3 / 51;
// that stay B = 2 to 8 0.9 / 11, 9 to 256 0.3 / 13, 257 to 512 0.4 / 9, 513 to 768 0.2 / 35, to 1280 0.6 / 18, more 0.4 / 24.  One query is what its own
// walk is (leaves 6 / 21, stays 2 / 29); all together 1.1.
// What moves the lines: R (a step of 63 or 32 neighbours holds the expansions of several narrow rows); the rounds of workgroups (200 k x 768, R = 32,
// ef = 384, queries that stay, this kernel's time over the other's: B = 600 0.83, 1024 1.08, 1990 0.94); the visited set in memory (B = 1024, R = 32,
// ef = 192 1.3 M x 64 1.26, in LDS 200 k x 128 0.96, 40 k x 384, which it covers more of, 0.85); and long rows of a corpus beyond the caches: a step
// scores some neighbours that it drops, at the rate of memory there (B = 1024, R = 32, ef = 512, rows of 1536 bytes 200 k 0.97, 400 k 1.24, 800 k 1.31;
// 768 bytes, 1.3 M, 0.98).
inline bool beyond_caches(int64_t N, int row_bytes) { return row_bytes > 1024 && N * row_bytes > (int64_t)448 << 20; }
inline int frontier_from_leaving(int cus, int64_t N, int row_bytes, int R, int B, bool global) {
    const bool long_rows = row_bytes > 1024, once = B <= 3 * cus;
    if (B == 1) return global ? 144 : R <= 16 ? 48 : row_bytes > 256 ? 112 : 64;
    if (B < 8) return long_rows || global ? 64 : 48;
    if (B <= cus) return R <= 8 ? 72 : R <= 16 ? 56 : R <= 24 ? 40 : 32;
    if (B <= 2 * cus) return R <= 8 ? 72 : R <= 16 ? (long_rows ? 72 : 56) : global ? 64 : long_rows && R <= 24 ? 56 : 40;
    if (beyond_caches(N, row_bytes)) return once ? 96 : 144;
    return !long_rows ? 40 : once ? 56 : R <= 8 ? 120 : 80;
}
inline int frontier_from_staying(int cus, int64_t N, int row_bytes, int R, int B, bool global) {
    const bool long_rows = row_bytes > 1024, far = beyond_caches(N, row_bytes), once = B <= 3 * cus, most = B > 5 * cus;
    if (B == 1 && !global) return 48;
    if (B <= 8) return R <= 8 ? 48 : global ? 160 : R <= 16 ? 72 : 112;
    if (B <= cus) return R <= 8 ? (long_rows ? 72 : 48) : R <= 16 ? (global || far ? 144 : 80) : global || far ? 288 : 144;
    if (B <= 2 * cus) return R <= 8 ? (global ? 144 : 80) : R <= 16 ? (global || far ? 288 : 176) : global ? INT_MAX : far ? 1200 : 288;
    if (R <= 8) return far ? (once ? 64 : most ? 96 : 256) : long_rows && !once ? 80 : 40;
    if (R <= 16) return far ? (once ? 112 : 320) : long_rows && !once ? 144 : 48;
    if (far) return once && R <= 24 ? 600 : INT_MAX;
    if (global) return once ? 176 : most ? 240 : 448;
    return long_rows ? (once ? 144 : 288) : once ? 40 : most ? 56 : 64 + (int)(N / 1536);
}

// Where graph_frontier_kernel is faster than the others (graph_search_kernel, graph_step_kernel, whichever was better), us, others / it:
//   every query a compute unit to itself, R = 32: 200 k x 768 fp16, B = 256 ef = 16 93 / 91, 48 198 / 174, 192 587 / 427, 768 2202 / 1122,
//     4096 7992 / 4101; B = 1 128 / 86, 416 / 226, 1916 / 558 at ef = 48, 192, 768; 60 k x 384 1121 / 510 (ef = 384); 1 M x 768 with the
//     visited set in memory 6196 / 3535 (ef = 2048), 22 838 / 12 592 (8192).  The very shortest lists end before its larger start is
//     paid for (ef = 3: 30.4 / 35.8), and rows of 4 KB, of which a step scores some for nothing, make it later (B = 256, ef = 16
//     134 / 156, 64 360 / 349)
//   two workgroups a compute unit: a step of four waves holds 32 unknown neighbours, little more than one expansion's while the list
//     fills.  200 k x 768, R = 32, B = 300 ef = 64 224 / 244, 96 326 / 348, 128 418 / 394, 192 644 / 562, B = 512 254 / 266, 359 / 373, 442 / 432, 653 / 582;
//     100 k x 256 96 292 / 295, 128 378 / 346; R = 31, whose two rows fit 63 places, 50 k x 128 fp32 64 190 / 179; R = 24 200 k x 768 48 196 / 196,
//     96 354 / 327, 100 k x 256 32 144 / 142, 48 187 / 180; R = 16 8 57 / 59, 12 73 / 71
//   three: once round (B = 700) any but the shortest: 200 k x 768, R = 32 ef = 16 143 / 136, 48 318 / 252, R = 24 64 418 / 289; 100 k x 256 16 133 / 117, 64
//     356 / 230.  More queries, which take turns (B = 1024), have longer rows waiting for the memory path: 200 k x 768, R = 32 24 223 / 245, 48 373 / 378,
//     64 454 / 442, R = 24 24 218 / 209, 48 364 / 350; 100 k x 256, R = 32 24 191 / 188, 64 391 / 321, R = 24 24 194 / 165; R = 16 8 107 / 94
//   rows of 4 KB start later there: 60 k x 1024 fp32, R = 32, B = 300 ef = 128 618 / 646, 160 735 / 711, B = 512 160 794 / 819; B = 700 48 513 / 508, 64 648 /
//     577; B = 1024 96 998 / 1112, 128 1282 / 1305; R = 16, B = 512 16 139 / 169, 48 268 / 270
//   visited set in memory: short lists stay with the id caches, which need no workspace; R = 32, B = 512, 1 M x 768 ef = 600 2215 /
//     2516, 1024 3619 / 3799, 2048 6959 / 6364, 4096 13 421 / 10 524; R = 24 or rows of 256 bytes all of them (700 k, ef = 600 2086 /
//     1983, 1907 / 1812)
//   no counters, visited set in memory, B = 600 / 1024: 0.31 to 0.97 times as long wherever measured (700 to 2048, 200 k to 2.5 M, rows of 128 to 1536 bytes)
//   maturity exit: by the lines above
inline bool frontier_pays(int cus, int64_t N, int row_bytes, int R, int B, int ef, bool counters, bool leaves, const FrontierLds &L) {
    if (R > GRAPH_STEP_MAX_R || L.total > LDS_MAX) return false;
    const bool global = L.vis_mode == FRONTIER_VIS_GLOBAL, own = B <= cus, waits = B > 2 * cus, long_rows = row_bytes > 2560;
    if (counters) return ef >= (leaves ? frontier_from_leaving(cus, N, row_bytes, R, B, global) : frontier_from_staying(cus, N, row_bytes, R, B, global));
    if (global && ef <= GRAPH_EF_TWO_LEVEL) return false;
    if (own) return ef >= (row_bytes > 2048 ? 72 : R > 16 ? 12 : 8);
    if (R <= 16) return ef >= (long_rows ? (waits ? 16 : 36) : waits ? 8 : 12);
    if (global) return waits || R <= 24 || row_bytes <= 512 || ef >= 1400;
    const bool once = B <= 3 * cus, mid_rows = row_bytes > 1024;
    if (waits) return ef >= (once ? (long_rows ? 64 : 16) : long_rows ? (B <= 6 * cus ? 136 : 96) : mid_rows && R > 24 ? 64 : 24);
    if (R <= 24) return ef >= (long_rows ? 128 : mid_rows ? 72 : 40);
    return ef >= (long_rows ? 200 : mid_rows ? 128 : R < GRAPH_STEP_MAX_R ? 64 : 96);
}

// Where graph_step_kernel is faster than graph_search_kernel, among the calls that graph_frontier_kernel does not take: lists of
// up to 512 entries without counters on graphs whose visited set does not fit LDS beside them.  A step costs two to three expansions of the
// other kernel, so what decides is how many expansions it commits: the neighbours a step holds (63 for a batch that leaves
// every query a compute unit, else 32) against the unseen ones that an expansion brings.  Those get fewer as a search covers
// more of the graph, so the line runs along N / ef, the nodes of the graph per entry of the list, and lies higher for narrow
// graphs and for batches that wait for a place anyway (the mean over the queries counts there, not the slowest).  Time of the
// one-by-one loop / time in steps:
//   more queries than two workgroups per compute unit hold, R = 32: 200 k, ef = 192 to 512, B = 600 1.0 to 1.2; 1 M 0.96 to 1.08; about
//     two full rounds of places (B = 800 to 1100) gain least: 200 k 0.89 to 1.05, 1 M 0.78 to 0.84; B = 2048 200 k 1.05 to 1.43,
//     1 M 0.71 to 1.0.  R = 16: 1.0 to 2.1 at any of these N
//   up to two queries 1.0 to 4.4 (0.8 at worst: it depends on the query); rows of more than 2 KB not
inline bool graph_step_pays(int cus, int64_t N, int row_bytes, int R, int B, int ef) {
    if (R > GRAPH_STEP_MAX_R || ef > GRAPH_EF_TWO_LEVEL) return false;
    if (B <= 2) return ef >= 320 && row_bytes <= 2048;
    if (B <= 2 * cus || ef < 192) return false;
    if (R <= 16) return true;
    const bool two_rounds = B >= 3 * cus && 2 * B <= 9 * cus;
    const int64_t reach = two_rounds ? (R <= 24 ? 800 : 400) : R <= 24 ? 3000 : B > GRAPH_DENSE_MIN_B ? 1024 : 1600;
    return ef * reach >= N;                               // nodes per list entry up to which steps pay
}

}  // namespace ann
