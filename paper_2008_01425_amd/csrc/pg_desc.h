// Descriptor records shared by the host planner and the gfx950 kernels.
//
// Notation follows the paper: workers i, edges e = (a, b), layers l with X^l in R^{p x q},
// rank r_l, projection state Q_e^l (q x r_l), P_e^l = D_e Q_e (p x r_l), Phat = orth(P).
// A worker multiplies its matrix ONCE per sweep by the stacked columns of all its incident
// edges ("Linearity", Section 3.1): R = deg(i) * r_l stacked columns j = slot * r_l + k.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define PG_BOTH __host__ __device__
#else
#define PG_BOTH
#endif

namespace pg {

constexpr int kMaxCols = 16;   // largest R = deg(i) * r_l one pass supports
constexpr int kThreads = 256;  // work-group size of the column-owner and combine kernels (4 wavefronts)
constexpr int kRowThreads = 64;  // narrow row-owner kernels: one wavefront per tile
constexpr int64_t kLightBytes = 64ll << 20;  // parameter bytes (all workers) up to which the narrow row kernels block 4 rows, not 8
// Parameter bytes (all workers) above which passes stream them past the caches, where the rows suit
// it (see streams()).  Measured with one matrix of 4608 columns cut to size, streamed / plain: up to 4
// stacked columns 1.04 (round) and 0.97 (run) at 208 MB, 1.01 and 0.93 at 302 MB, 0.97 and 0.88 at
// 377 MB; 8 columns 1.03 at 472 MB, 0.98 at 604 MB; 16 columns 1.00 at 377 MB, 0.97 at 604 MB.
constexpr int64_t kStreamBytes = 320ll << 20;
constexpr int64_t kStreamBytesWide = 512ll << 20;  // 8-16 stacked columns
// Share of the elements that has to lie in layers that gain from streamed passes (from runs that write every
// second round).  The hint goes with the launch, not the layer: it gains 3-5 % on rows that suit it and
// costs 5-20 % on the others, so about three quarters break even.
constexpr double kStreamShare = 0.75;
// Runs that write every second round: at most this many stacked columns, and this much LDS for a
// peeking column kernel's work-group (Phat and the pending coefficients of a row block).
// Measured on VGG-16 shapes, ring of 16, ten rounds a call: rank 1 (2 stacked columns) 5.55 -> 4.50 ms; at 4
// columns 4 rows per lane group gain 7 % and 8 rows, which spill, lose 12 %.
constexpr int kLazyCols = 4;
constexpr int kLazyColLds = 64 * 1024;
// Narrow kernels: rows of at least this many floats may be moved four at a time whatever q is (see
// row_body, and gains_units_of_four() in the planner for which are).  Shorter ones are a few vectors
// at most and go by the widest one that divides q.
constexpr int kAnyAlignCols = 16;
constexpr int64_t kOddLongBytes = 40ll << 20;    // parameter bytes (all workers) from which long rows of odd length are ...
constexpr int64_t kOddLongBytes4 = 128ll << 20;  // ... at 4 stacked columns, unless the set is light or a row fits one step
// Share of the elements in such rows from which the kernels that carry a body for them are launched.
// Measured, those kernels / the ones without on matrices of 576 (4608, 32, 152) columns beside some of
// 577 (4607, 27, 153), 8 to 300 MB, ring of 8, round, SGD round and run at ranks 1 and 2: no such rows
// 0.98-1.03; share 0.003: 0.94-1.04; 0.01: 0.80-1.05; 0.05: 0.75-1.04; all rows: 0.49-1.08.
constexpr double kOddShare = 0.01;
constexpr int kVecClassPairs = 1024;  // (worker, vector layer) pairs from which vector layers get kernels of their own
constexpr int kWideCols = 8;     // from this many compiled columns on, row tiles stage Q in LDS
constexpr int kWideLdsBytes = 48 * 1024;  // LDS budget of a wide row tile's Q slice
constexpr int kColLdsBytes = 48 * 1024;   // LDS budget of a (vector) column tile's Phat slice
constexpr int kMfmaRowBlocks = 2;  // matrix-core row tiles: blocks of 16 rows per wavefront
constexpr int kMfmaRowCols = 16;    // stacked columns from which row passes run on the matrix cores
constexpr int kMfmaSegCols = 2048;  // matrix-core row tiles: longest column segment
constexpr int kMfmaTileCols = 256;  // matrix-core column tiles: columns per tile (four wavefronts)

// One stacked column of a (worker, layer) pair.
struct ColDesc {
    int64_t q_off;   // float offset of the Q column (edge, layer, k) in the state buffer
    int64_t ph_off;  // float offset of the Phat column (edge, layer, k) in the workspace
    float coef;      // +w_e when the worker is the edge's first endpoint, -w_e otherwise:
                     // X_i -= coef * Phat Q'^T   (Eq. (2); equal and opposite on the two ends)
    int32_t pad;
};

// One (worker, layer) pair.
struct PairDesc {
    int32_t worker, p, q, R;
    int64_t x_off;     // float offset of the layer inside a worker buffer (rows are ld floats apart)
    int64_t pw_off;    // double offset of this pair's partial products X_i S: [seg][j][row]
    int64_t qw_off;    // double offset of this pair's partial products X_i^T T: [blk][j][c]
    int32_t col0;      // first ColDesc of the pair (R consecutive entries)
    int32_t lpr;       // row-owner kernels: lanes that share one row (power of two <= 64)
    int32_t nseg;      // row-owner kernels: column segments a row is split into
    int32_t seg_len;   // floats per segment (multiple of lpr * V; the last one may be shorter)
    int32_t lg;        // column-owner kernel: lanes side by side over columns (power of two <= 64)
    int32_t nblk;      // column-owner kernel: row blocks
    int32_t blk_rows;  // rows per block
    int32_t V;         // floats per access to X: 4, 2 or 1.  The largest that divides q, or 4 where the planner
                       // chose units of four: any rows from kAnyAlignCols on in the narrow kernels, padded rows in the wide ones
    int32_t wc;        // matrix-core row tiles: wavefronts side by side over the column steps (1, 2 or 4)
    int32_t ld;        // floats from one row of the layer to the next in a worker buffer (>= q)
};

// Row-owner tile: rows [row0, row0 + nrows) x column segment seg of one pair.
struct RowTile {
    int32_t pair, row0, nrows, seg;
};

// Column-owner tile: columns [c0, c0 + lg * V) x row block blk of one pair.
struct ColTile {
    int32_t pair, c0, blk, pad;
};

// One (edge, layer): where its partial products, Phat, state and flags live.
struct EdgeLayerDesc {
    int32_t p, q, r, nseg;
    int32_t nblk, pad;
    int64_t pwa_off, pwb_off;  // double offsets of this edge's column 0, segment 0, in worker a / b
    int64_t pwa_seg, pwb_seg;  // stride between segments (R_a * p, R_b * p)
    int64_t qwa_off, qwb_off;  // double offsets of this edge's column 0, block 0, in worker a / b
    int64_t qwa_blk, qwb_blk;  // stride between blocks (R_a * q, R_b * q)
    int64_t pd_off;            // double offset of the Gram-Schmidt scratch: r columns of p
    int64_t ph_off;            // float offset of Phat: r columns of p
    int64_t q_off;             // float offset of the state block: r columns of q
    int64_t flag_off;          // int32 index of the r dropped-column flags
};

// Row chunk of one (edge, layer) for the two-kernel orthonormalisation of tall layers; the
// chunks of an (edge, layer) are consecutive tiles.
struct OrthTile {
    int32_t el, row0, nrows, chunk, nchunks, pad;
};
constexpr int kOrthTallRows = 4096;   // layers taller than this are orthonormalised chunk by chunk
constexpr int kCombPRows = 2048;      // rows per work-group of the p-side combine of single iterations
constexpr int kOrthChunkRows = 1024;  // rows per chunk (one work-group of 256 threads)

// Edge kernels (sets of small layers): one work-group holds the difference of the two workers' matrices of
// one (edge, layer) in registers, kEdgeUnits units of four floats of one row per thread.
constexpr int kEdgeThreads[] = {256, 512};  // work-group sizes; a set takes the smallest that its layers fit
constexpr int kEdgeUnits = 9;
constexpr int kEdgeMaxRank = 4;
// Elements of a layer up to which they are taken.  Time of the streaming kernels over theirs, 60 drawn sets: largest layer 1400 to
// 7200 elements 1.3-3.5, 8300 to 12700 1.2-2.0, above 14000 0.8-1.1 (a work-group is then longer at it than the launches it saves);
// 100 x 100, ring of 8, ten rounds 138 -> 115 us, three layers of 64 x 32 and less, ring of 4, one round 20.0 -> 10.2 us.
constexpr int kEdgeSize = 12800;
// (Edge, layer) pairs, one work-group each, up to which they are taken: streaming kernels over theirs, 400 drawn sets of up to 4000 layers, round and
// single iteration (worst twentieth / median): up to 2048 pairs 1.43 / 2.0 and 1.07 / 1.5, 3000 to 5000 1.16 / 1.29 and 0.87 / 0.95,
// above 10000 0.66 / 0.92 and 0.62 / 0.78.
constexpr int kEdgeTiles = 2048;
// Runs: a round's update goes into the next round's edge kernel up to one pair per CU, and where that work, done once per edge, is less than the
// launch it saves.  Run of five with it / without it, times of the streaming kernels over both (median): up to 64 pairs 2.05 / 1.57, 128 to 256
// 2.06 / 1.87, 256 to 512 2.26 / 2.73, 2000 1.2 / 1.7.
constexpr int kEdgeRunTiles = 256;
constexpr int kEdgeRunCost = 150;                   // see edge_run_cost()
constexpr int64_t kEdgeRunBytes = 32ll << 20;       // most of the second buffer that it takes
constexpr int kEdgeLdsBytes = 152 * 1024;
constexpr int kEdgeSumBytes = 72 * 1024;    // of that, column sums of the wavefronts
constexpr int kApplyUnits = 4;  // units of four floats per thread of the update kernel that goes with them
struct EdgeTile {
    int32_t p, q, r, ld;
    int32_t wa, wb;          // the edge's workers
    int32_t tc_shift;        // log2 of the threads side by side over the units of a row
    int32_t own;             // bit 0 (1): this work-group stores worker a's (b's) matrix when it applies a pending update
    int32_t col_a, Ra, col_b, Rb;  // the two workers' stacked columns of this layer
    int64_t x_off, q_off, ph_off, flag_off;
};
// Units of a thread whose column sums an edge kernel exchanges at once.
PG_BOTH inline int edge_units_at_once(int tc_shift, int nt) {
    const int groups = tc_shift <= 6 ? nt / 64 : nt >> tc_shift;  // wavefronts with the same columns
    const int fit = kEdgeSumBytes / (groups * 32 << tc_shift);
    return fit < 1 ? 1 : fit;
}
// LDS sections of an edge kernel's work-group, byte offsets: sums of the wavefronts; P [r][ps] in double (ps = p in whole
// units of four); the right vectors [r][vs], zeros behind q; the threads' entries of the unit vectors; single iterations:
// unit vectors in R^q and the vectors in R^p.  At first the operands of a pending update (R vectors of each side in all).
struct EdgeLds {
    int red, p, v, ph, u, pst, bytes;
};
PG_BOTH inline EdgeLds edge_lds(int p, int q, int r, int tc_shift, int nt, int R) {
    const int vs = (q + 3) & ~3, ps = (p + 3) & ~3;
    const int groups = tc_shift <= 6 ? nt / 64 : nt >> tc_shift;
    int units = edge_units_at_once(tc_shift, nt), all = ((vs >> 2) + (1 << tc_shift) - 1) >> tc_shift;
    if (units > all) units = all;
    EdgeLds o;
    o.red = 0;
    int red = units * groups * 32 << tc_shift;
    const int part = tc_shift > 6 ? r * (1 << (tc_shift - 6)) * ps * 8 : 0;  // row sums of the wavefronts of a row
    if (red < part) red = part;
    if (red < R * (vs + ps) * 4) red = R * (vs + ps) * 4;
    o.p = red;
    o.v = o.p + r * ps * 8;
    o.ph = o.v + r * vs * 4;
    o.u = o.ph + r * nt * 4;
    o.pst = o.u + r * vs * 4;
    o.bytes = o.pst + r * ps * 4;
    return o;
}
// Update tile: units [first, first + kThreads * kApplyUnits) of one pair, counted row by row.
struct ApplyTile {
    int32_t pair, first;
};

// Tile of the update kernel for workers with different numbers of columns: rows [row0, row0 + nrows) and units (four columns)
// [unit0, unit0 + nunits) of one pair, 2^tc_shift threads side by side over the units, kMixedRows rows per thread at a time.
constexpr int kMixedRows = 4;
constexpr int kMixedTileBytes = 32 * 1024, kMixedTiles = 1024;  // most parameter bytes of a tile, tiles to aim at
struct MixedTile {
    int32_t pair, row0, nrows, unit0, nunits, tc_shift;
};

// Edge sweeps: one (edge, layer).
constexpr int kSweepMaxRank = 4;
constexpr int kSweepGram = 10;         // Gram sums per row block (rank 4)
constexpr int kSweepVectorRows = 512;  // vectors up to this length are one wavefront's
constexpr int kSweepExactSize = 10000; // elements up to which a layer is walked twice (rows under four floats: rows x rank as well)
constexpr int kSweepExactRows = 2048;  // rows x rank of such a layer with longer rows (its P lies in LDS)
constexpr int64_t kSweepMixedBytes = 160ll << 20;  // parameter bytes (all workers) up to which mixed degrees alone decide
constexpr int kSweepLongRows = 8;      // most rows of a tile whose rows are too long for the registers
constexpr int kSweepLdsBytes = 152 * 1024;
// Sets (bytes read, both ends of every edge) up to which a row block's edges are spread over the dies, so that all of them have work:
// rounds of 70 drawn sets, kept together over spread: up to this limit 0.99-1.07 (mean 1.02), above 0.92-1.08 (mean 0.97).
constexpr double kSweepSpreadBytes = 8.0 * (1 << 20);
struct SweepDesc {
    int32_t p, q, r, ld;
    int32_t wa, wb;          // the edge's workers
    int32_t tc_shift;        // log2 of the threads side by side over the units (four floats) of a row
    int32_t units;           // units per thread, compiled: 1, 2, 3 or 5; 0: rows too long for the registers
    int32_t nblk, flag_off;
    int32_t exact, pad;      // one block, walked twice: the column sums are formed with Phat rounded to float
    int64_t x_off, q_off, ph_off;
    int64_t pe_off, qe_off, g_off; // double offsets of P [k][row], the blocks' D^T P [blk][k][c] and their Gram sums
};
// Rows [row0, row0 + nrows) of one (edge, layer), block blk; blk < 0: nrows vectors, (edge, layer)s el and the next.
struct SweepTile {
    int32_t el, row0, nrows, blk;
};
// Entries [first, first + count) of the p rows of P followed by the q entries of Q' of one (edge, layer).
constexpr int kFinishEntries = 1024;
struct FinishTile {
    int32_t el, first, count;
};

// combine_q tile: 256 consecutive elements of the r*q block of one (edge, layer).
struct CombTile {
    int32_t el, first;
};

}  // namespace pg
