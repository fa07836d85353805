// Which kernel a GEMM of the bf16 model runs in, by its sizes and rows: host arithmetic only, free of any device state, so
// that a machine without a GPU can check what a shape takes (ee_debug_gemm_route).
#pragma once
#include <algorithm>
#include <cstddef>

#include "ee.h"

namespace ee {

// A GEMM cut along its contraction (pf_part_kernel in ee_prefill.hip): the k-tiles of all result tiles (256 columns x mtl
// row tiles) stand behind each other and every workgroup takes `unit` of them.
struct PartGeom {
    int n_tiles, n_wgN, n_wgM, m_tiles, KT, unit, mtl;
};

namespace route {

constexpr int CUS = 256;
constexpr int PANEL = 16;  // 16-column weight tiles per result tile of the prompt phase's GEMMs and of the cut (256 columns)

// ---- decode steps, few rows: the rows are staged in LDS

constexpr int lds_row_stride(int K) { return 2 * K + 32; }  // elements; +64 B staggers the banks of two rows
inline size_t lds_rows_bytes(int T, int K) { return (size_t)T * lds_row_stride(K) * 2; }

// Waves per workgroup of a decode GEMM (bf16); merges: its input is merged from attention partials while being staged;
// packed: its rows come in operand order.
inline int step_waves(int T, int K, int N, bool packed, bool merges) {
    const int kt = K / 32;
    // One workgroup or less per CU: more waves, shorter chains, where the chains are long enough.  Us with 4 and 8 waves (event
    // pairs, which add about 3 us; spread 0.5), 1, 2 and 3 rows: 64 k-tiles, 64 workgroups (down) 7.3 / 6.6, 9.1 / 8.2, 9.4 /
    // 8.9; 128 (O, KV range unsplit) 8.5 / 8.2, 8.5 / 7.8, 9.2 / 8.8; 256 (gate|up) 8.7 / 8.6, 8.5 / 8.1, 9.1 / 8.6.  48
    // k-tiles: 96 workgroups (down) 8.0 / 8.2, 7.6 / 7.8, 8.3 / 8.4.  32 to 40 k-tiles lose with one row: Q|K|V, 192
    // workgroups 7.2 / 7.6, 8.1 / 8.2, 8.2 / 8.2, 240 7.6 / 8.0; gate|up, 128 7.1 / 7.4; O, 64 7.4 / 7.7, 8.3 / 8.6.
    if (kt > 48 && kt <= 64 && T <= 3 && N / 16 <= CUS && !merges && !packed) return 8;
    if (kt <= 64 || T > 32) return 4;   // (packed rows: rows_shape has the last word)
    if (kt <= 128 || T > 16) return 8;  // (16 waves of 1024 threads leave 128 registers each: one row tile only)
    return 16;
}

// Which rows are staged.  Every workgroup stages all of them for its one column tile, so what a second and third row cost
// grows with their bytes and with the rounds of workgroups: two or three rows of up to 36 KB (2 rows at K = 4096), or
// of all the LDS where the launch is a single round (the down projection).  Us per step, staged / rows_kernel: 7B widths,
// 4 layers, 2 sequences 456 / 489, 3 (48 KB) 503 / 497, 4 526 / 502; 1.3B widths, 8 layers, 3 sequences 451 / 482, 4 503 /
// 488, 8 647 / 521; 30B widths, 4 layers, 2 sequences (53 KB) 988 / 962, 3 1061 / 966; 768 wide, 12 layers, 4 sequences
// 474 / 405, 16 624 / 407.
constexpr size_t LDS_MAX_BYTES = 72 * 1024;      // one row, workgroups of up to 8 waves
constexpr size_t LDS_MAX_BYTES_16 = 140 * 1024;  // 16 waves have the CU to themselves whatever their LDS use
constexpr size_t LDS_FEW_BYTES = 36 * 1024;

inline bool rows_staged(int T, int K, int N) {
    if (T > 3) return false;
    const size_t b = lds_rows_bytes(T, K), all = step_waves(T, K, N, false, false) == 16 ? LDS_MAX_BYTES_16 : LDS_MAX_BYTES;
    if (T == 1 || N / 16 <= CUS) return b <= all;
    return b <= LDS_FEW_BYTES;
}

// The rows of a head.  They are packed for this one launch, which a projection's rows are not (their producer writes them
// so), so up to four stay staged, from 24 k-tiles on and with workgroups of up to 8 waves (K up to 4096).  What staging adds
// to a head and its packing, us, vocabulary 32000 | 50304: 4 rows, 768 wide -0.8 | -2.3; 1024 -3.0 | -5.8; 1536 -3.5 | -7.5;
// 2048 -3.8 | -8.1; 2560 -0.2 | -4.3; 3072 +2.5 | -0.7; 4096 -2.5 | -4.3; 3 rows, 3072 wide -0.5 | -7.0; 4096 -1.8 | -4.7.
// Beyond: 4 rows, 256 and 512 wide +3, +4; 6 rows, 2048 wide +5.6 | +8.1; 5120 wide (16 waves), 2 rows +5.5 | +3.3.
inline bool head_staged(int T, int K) {
    if (rows_staged(T, K, 3 * K)) return true;
    return T <= 4 && K >= 24 * 32 && step_waves(T, K, 3 * K, false, false) <= 8 && lds_rows_bytes(T, K) <= LDS_MAX_BYTES;
}

// ---- decode steps of one sequence: is the front of the next segment (packing, Q|K|V, attention) enqueued behind an exit's head,
// before the decision is known?  A token that stays saves the host's round trip, about 6 us at any width and row count (2 to 9
// from 2048 wide on, 2 to 15 at 768).  For one that leaves the front ran for nothing, and what of it outlasts the host's own
// time delays the next step, by about, at 1 | 2 | 4 | 8 | 16 rows (contexts 300 and 1200): 768 wide 0 | 7 | 0 | 1 | 8 us; 2048
// wide 8 | 3 | 13 | 16 | 22; 4096 wide 6 | 12 | 21 | 24 | 30; 6656 wide 38 | 43 | 50 | 50 | 58; 32 rows 9, 22, 37, 57.  The line (16
// rows, 4 rows at 4096 wide) is where a front thrown away costs about three times what a kept one saves, so that it pays while
// no more than one token in four leaves at the exit.  (6656 wide, 1 and 2 rows: one in seven.)
constexpr int FRONT_MAX_ROWS = 16, FRONT_MAX_ELEMS = 4 * 4096 + 1024;
inline bool front_ahead(int dtype, int T, int d) { return dtype != EE_BF16 || (T <= FRONT_MAX_ROWS && T * d <= FRONT_MAX_ELEMS); }

// ---- decode steps, many rows: rows_kernel, in passes of up to 64 rows

// ee_config::gemm_min_workgroups: 0 stands for 512, and from there on it changes nothing
inline bool default_min_wgs(int min_wgs) { return min_wgs < 1 || min_wgs >= 512; }

constexpr int PASS_ROWS = 64;  // the largest row tile count rows_kernel is built for

inline int row_tiles(int T) { return T <= 16 ? 1 : (T <= 32 ? 2 : 4); }

// Column tiles per workgroup of a launch of many rows.  One workgroup is resident per CU, so the launch runs in rounds of
// 256 workgroups (fewer where the test hook ee_config::gemm_min_workgroups asks for it), and per k-tile a workgroup takes
// in its G weight tiles and the rows' operands in two terms: rounds x (G + 2 mt) is what the launch costs (64 rows at the
// 7B width: Q|K|V, 768 tiles, 3 tiles per workgroup; gate|up, 1376 tiles, 6).
inline int tiles_per_wg(int mt, int n_tiles, int min_wgs) {
    const int cus = default_min_wgs(min_wgs) ? CUS : (min_wgs / 2 > 0 ? min_wgs / 2 : 1);
    int best = 1;
    long cost = -1;
    for (int g = 1; g <= 6; ++g) {
        const long c = (long)((n_tiles + g - 1) / g + cus - 1) / cus * (g + 2 * mt);
        if (cost < 0 || c < cost) cost = c, best = g;
    }
    return best;
}

// Ring slots per wave of rows_kernel: as many as the registers hold next to the accumulators (512 per lane with one wave per
// SIMD, 256 with two, 128 with four).
constexpr int rows_ring(int waves, int mt, int tiles) {
    const int d = ((waves == 4 ? 290 : waves == 8 ? 190 : 84) - 4 * tiles * mt) / (4 * (tiles + 2 * mt));
    return d < 2 ? 2 : d > 8 ? 8 : d;
}

// Does rows_kernel refill a ring slot between the MFMAs of the next one (or in a burst behind its own)?  Four row tiles with
// one wave per SIMD only: that wave waits half of its time for the memory pipeline to take a load, and in a burst of G + 2 MT
// of them its matrix core waits too.  Us a full-depth step, burst / between: 4 waves (gate|up at 4096 wide, Q|K|V and gate|up
// at 6656), 33 | 48 | 64 rows: 4096 wide, 8 layers 1376 / 1351 | 1443 / 1418 | 1524 / 1504 (gate|up 51.8 / 48.5 us), 6656 wide,
// 6 layers 2039 / 2032 | 2090 / 2082 | 2207 / 2199.  8 waves cover each other's waits and lose by it: 2048 wide, 8 layers 700 /
// 707 | 724 / 729 | 761 / 769, 3072 wide 998 / 1001 | 1016 / 1021 | 1066 / 1072, 5120 wide, 4 layers 1118 / 1135 | 1176 / 1189
// | 1203 / 1219.
constexpr bool rows_loads_between(int waves, int mt) { return mt == 4 && waves == 4; }

// The launch of up to 64 packed rows.
struct RowsShape {
    int mt, tiles, waves;  // row tiles, column tiles per workgroup, waves
};

inline RowsShape rows_shape(int T, int K, int N, int min_wgs) {
    RowsShape r{row_tiles(T), 0, step_waves(T, K, N, true, false)};
    r.tiles = tiles_per_wg(r.mt, N / 16, min_wgs);
    if (r.waves == 16 && r.tiles >= 3) r.waves = 8;  // (1024 threads leave 128 registers per lane: two tiles at most)
    // Four row tiles: two waves per SIMD cover each other's waits for the memory pipeline.  Us a pass of two steps, 4 and 8
    // waves: 64 sequences, 768 wide, 12 layers 1519 / 1377; 2048 wide, 8 layers 1809 / 1675, 40 sequences 1672 / 1533; 4096
    // wide (Q|K|V, three tiles), 8 layers 4397 / 4343.  Five and six tiles keep one wave per SIMD: at the 256 registers of
    // two, six tiles spill 34 (4096 wide 4456), and 8 partial sums of five fill the LDS.
    if (r.mt == 4) r.waves = r.tiles <= 4 ? 8 : 4;
    return r;
}

// ---- GEMMs cut along their contraction

constexpr int PART_TILES = 256;

// Geometry of the cut of an N x K matrix over M rows: every workgroup an even share, but no fewer than eight k-tiles (a
// part costs its writing and reading) and no more parts than fit `bytes`.  False: it cannot be cut so (a share of the whole
// contraction is no cut).
inline bool part_geom(int N, int K, int M, size_t bytes, PartGeom* g) {
    g->mtl = M <= 64 ? 4 : 8;
    g->KT = K / 32;
    g->n_tiles = N / 16;
    g->n_wgN = (g->n_tiles + PANEL - 1) / PANEL;
    g->n_wgM = (M + g->mtl * 16 - 1) / (g->mtl * 16);
    g->m_tiles = (M + 15) / 16;
    const long tiles = (long)g->n_wgN * g->n_wgM;
    if (tiles > PART_TILES || g->n_tiles % 2) return false;
    const long wgs = std::min<long>(CUS, (long)(bytes / ((size_t)PANEL * g->mtl * 1024)) - tiles);
    if (wgs < 1) return false;
    const long u = (tiles * g->KT + wgs - 1) / wgs;
    g->unit = (int)std::max<long>(u, 8);
    return g->unit < g->KT;
}

inline int part_wgs(const PartGeom& g) { return (g.n_wgN * g.n_wgM * g.KT + g.unit - 1) / g.unit; }

// What the cut and its sum take, in microseconds, next to a launch without it: what a CU takes in, at gbps64 (64-row tiles) or
// gbps128 (128-row tiles) GB/s, bounds the cut; the sum reads all parts back and writes M x N values, those of Q|K|V at 340 a
// nanosecond (it writes V one 2-byte element at a time, as the cache keeps V transposed), others at 560.  Constants common to
// both ways to launch are left out, so those of the two rules below are differences.  All fitted to the times of whole
// prompts and steps with each of the four GEMMs cut and not, in all combinations.
inline float cut_us(int kernel, const PartGeom& g, int M, float gbps64, float gbps128) {
    const int parts = part_wgs(g) + g.n_wgN * g.n_wgM;
    return g.unit * (16 + 2 * g.mtl) / (g.mtl == 4 ? gbps64 : gbps128) + parts * 16 * g.mtl / 5300.0f +
           (float)M * (g.n_tiles * 16) / (kernel == EE_K_QKV ? 340e3f : 560e3f);
}

// Decode steps: does the cut, at 60 and 100 GB/s, beat rows_kernel, which takes, per k-tile and round, G KB of weights and 2 mt KB
// of rows, both at 92 GB/s with four row tiles and 8 waves, else the weights at 55 and the rows at 120, and for each further pass of
// up to 64 rows 1 us more (with RMS scales in front 3)?  Up to 32 rows rows_kernel takes in less and needs no second launch.
// Us that cutting one GEMM adds to a layer at 33 | 64 rows: 4096 wide Q|K|V +3 | +6, O -2 | -3, gate|up +2 | +4, down -16 | -15;
// 2048 wide +4 | +5, +1 | +2, +7 | +7, -6 | -7; 6656 wide +4 | +6, -6 | -5, -10 | -7, -28 | -29; 1024 wide all but down (-2 |
// -1) lose.  From 66 rows on rows_kernel streams the weights twice, and what wins at 1024 wide is down (-5), at 2048 wide all but
// gate|up (-3, -3, +1, -15), from 3072 wide on all four; with the scratch of a model for just so many rows (fewer workgroups) less:
// 66 | 96 rows, 2048 wide +5 | -4, -3 | -5, +21 | +5, -12 | -18; 4096 wide +1 | -9, -5 | -9, 0 | -12, -30 | -36.  Of 650
// such points the rule is wrong by 1 us or more at nine, by 3 us at most.
inline bool step_cut(int kernel, int N, int K, int T, int min_wgs, size_t bytes, PartGeom* g) {
    if (T <= 32 || !default_min_wgs(min_wgs)) return false;
    const bool resid = kernel == EE_K_OPROJ || kernel == EE_K_DOWN;
    float us = -3.8f;
    for (int r0 = 0; r0 < T; r0 += PASS_ROWS) {
        const RowsShape r = rows_shape(std::min(T - r0, PASS_ROWS), K, N, 0);
        const int rounds = ((N / 16 + r.tiles - 1) / r.tiles + CUS - 1) / CUS;
        us += rounds * (K / 32) * (r.mt == 4 && r.waves == 8 ? (r.tiles + 2 * r.mt) / 92.0f : r.tiles / 55.0f + 2 * r.mt / 120.0f);
        if (r0) us += resid ? 1.0f : 3.0f;
    }
    return part_geom(N, K, T, bytes, g) && cut_us(kernel, *g, T, 60.0f, 100.0f) < us;
}

// The head of 33 to 64 rows in panels of 256 columns (a vocabulary of at least half as many panels as there are CUs; 64 rows,
// 50304 words, 4096 wide: 128 -> 98 us).
inline bool head_panels(int T, int V, int min_wgs) { return T > 32 && T <= PASS_ROWS && default_min_wgs(min_wgs) && V >= 128 * 256; }

// ---- decode attention

constexpr int ATT_ROWS = 16;  // rows of a query tile: consecutive positions of one sequence

// Positions of K and V behind a launch: those its sequences have, and those its query tiles read (each tile all up to its last row).
struct KvReads {
    size_t distinct = 0, read = 0;
    void add(int first, int rows) {  // a sequence whose rows are the positions first .. first + rows - 1
        for (int r = 0; r < rows; r += ATT_ROWS) read += first + std::min(r + ATT_ROWS, rows);
        if (rows > 0) distinct += first + rows;
    }
};

// Are K and V read past the caches?  The 256 MB behind the L2s hold them until they are read again where that comes soon enough:
// what counts is their bytes over the `layers` that lie between (with exits on, those up to the end of this segment: a token may
// leave there and the next one begins), not those of one layer.  % that reading them past the caches adds to a step, by
// those bytes: 63 to 330 MB -0.7 to +2.8, nearly all slower (7B widths, 1 sequence, 32 layers, 306 MB +0.4; 8, first exit behind 2
// layers, 253 MB +2.8), 380 to 530 MB between -2.8 and +1.5, 20 of 26 points faster (16 sequences, 1.3B widths, first exit behind 6 layers, 384 MB
// -2.6; 7B widths, behind 2, 506 MB -1.0; one, 32 layers, 518 MB 0.0 and +0.2), 750 MB and more 0 to -6 (7B widths, 16
// sequences, 16 layers, 4.0 GB -2.7; 1.3B widths, 24 layers, 3.0 GB -4.2, 6.0 GB -6.0, first exit behind 6 of them, 1.5 GB -5.7; 30B
// widths, 16, 4 layers, 3.3 GB -3.9; the worst, 64 contexts of 100, +0.5).
// Query tiles of one sequence read the same positions at about the same time, and the caches serve the second, unless there is
// too much between them as well.  read / distinct 1.1 to 1.5: -0.4 to -4.4.  2 (17 to 32 rows a sequence): 86 to 244 MB a layer
// +0.5 to +3.6, one point of nine faster (-0.9); 250 to 500 MB between -5.1 and +1.8, ten of 14 faster.  3 (33 to 41 rows): +0.2
// to +7.5 at 60 to 530 MB a layer.
inline bool kv_past_caches(const KvReads& r, int d, int layers) {
    const size_t layer = r.distinct * d * 4;
    return 2 * r.read <= 3 * r.distinct ? layer * layers >= (size_t)384 << 20 : r.read <= 2 * r.distinct && layer >= (size_t)256 << 20;
}

// ---- prompt phase

// Row tiles per workgroup of a GEMM that is not cut, 8 or 4.  A CU works through about ceil(workgroups / 256) tiles
// (whether one after another or two side by side), each for a time proportional to its rows: take the cheaper, 128 rows on
// a tie (half the activation traffic from L2).
inline int prompt_row_tiles(int N, int M) {
    const long n_wgN = (N + 255) / 256;
    const long r8 = (n_wgN * ((M + 127) / 128) + CUS - 1) / CUS * 8;
    const long r4 = (n_wgN * ((M + 63) / 64) + CUS - 1) / CUS * 4;
    return r4 < r8 ? 4 : 8;
}

// Prompt phase: is the cut, at 54 and 50 GB/s, faster than a workgroup per result tile, which takes in `rounds` x KT x (16 + 2 mtl) KB per CU, at
// 77 GB/s with 64-row tiles and 55 with 128-row tiles, and 1/70 us per 64-row tile or 15 us with 128-row tiles (0.3 us per
// k-tile on short contractions)?  Us that cutting one GEMM adds to a layer: 4096 wide, 64 | 99 | 256 | 512 rows: Q|K|V -31 |
// -19 | +6 | -7, O -40 | -30 | -26 | -15, gate|up -17 | -2 | -19 | +1, down -115 | -94 | -90 | -59; 2048 wide, 65 | 384 | 640
// rows: -13 | +3 | +18, -14 | -10 | -4, -4 | -9 | +18, -44 | -41 | -28.
inline bool prompt_cut(int kernel, int N, int K, int M, size_t bytes, PartGeom* g) {
    const bool resid = kernel == EE_K_OPROJ || kernel == EE_K_DOWN;
    // (With more than four row tiles of a few column panels the ranges of one panel's row tiles no longer run side by side,
    // so its weights are fetched again: 640 rows at the 7B widths, 80 tiles, the cut loses by 16 us for O and for down.)
    if (resid && (N + 255) / 256 * ((M + 127) / 128) > 64) return false;
    // (Short contractions: with 128-row tiles 16 and 20 k-tiles gain 1 or lose up to 6 us by it and 24 gain 2 to 3, with 64-row
    // tiles 12 lose 0 to 3, 16 and 20 gain 0 to 2 and 24 gain 2 to 4.)
    if (K < (M <= 64 ? 22 : 32) * 32 || !part_geom(N, K, M, bytes, g)) return false;
    const int mtl = prompt_row_tiles(N, M);
    const long direct_tiles = (long)g->n_wgN * ((M + mtl * 16 - 1) / (mtl * 16));
    const long rounds = (direct_tiles + CUS - 1) / CUS;
    const float us = rounds * g->KT * (16 + 2 * mtl) / (mtl == 4 ? 77.0f : 55.0f) + (mtl == 4 ? direct_tiles / 70.0f : std::min(15.0f, 0.3f * g->KT));
    return cut_us(kernel, *g, M, 54.0f, 50.0f) < us + (kernel == EE_K_QKV ? 2.0f : resid ? 1.0f : -1.0f);
}

// Scratch that the cuts of a prompt phase of up to `max_rows` rows per pass can use.  (What is cut, and how, changes with
// the number of 64-row tiles.)
inline size_t prompt_part_bytes(int d, int F, int max_rows) {
    const int N[4] = {3 * d, d, 2 * F, d}, K[4] = {d, d, d, F}, kernel[4] = {EE_K_QKV, EE_K_OPROJ, EE_K_SWIGLU, EE_K_DOWN};
    size_t need = 0;
    for (int i = 0; i < 4; ++i)
        for (int M = 1; M <= max_rows; M += 64) {
            PartGeom g;
            if (prompt_cut(kernel[i], N[i], K[i], M, (size_t)1 << 40, &g))
                need = std::max(need, (size_t)(part_wgs(g) + g.n_wgN * g.n_wgM) * PANEL * g.mtl * 1024);
        }
    return need;
}

}  // namespace route
}  // namespace ee
