#include "pg_plan.hpp"

#include <algorithm>
#include <cmath>
#include <set>
#include <utility>

#include "../../include/powergossip.h"

namespace pg {

static inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
static inline int pow2_ceil(int v) {
    int r = 1;
    while (r < v) r <<= 1;
    return r;
}

int compiled_cols(int R) {
    int rc = 1;
    while (rc < R) rc <<= 1;
    return rc;
}

int rows_unroll(int RC, bool light) {
    if (RC < kWideCols) return light ? 4 : 8;
    return 4;
}

// Whether streamed passes over this layer gain, given the stacked columns a pass compiles.  A cache
// line that two load instructions share, or that a row fills in part, is fetched (and written) twice
// when it is not kept.  Measured on single matrices of 350-1200 MB, streamed / plain time of a round, an SGD
// round and a run of two to four rounds:
//   1-4 columns  q % 32 == 0: 0.97-1.00, 0.94-0.97; q = 48, 80, 144: 1.00-1.03, 0.98-1.01;
//                q = 100: 1.04, 1.01; 577: 1.17, 1.11; 4607: 1.04, 1.04; 50: 1.25, 1.15; 12: 1.24, 1.19
//   8 columns    q % 16 == 0: 0.94-1.02; padded rows: q = 72 1.11-1.14, 1.04-1.08; 130: 1.06-1.11, 0.97-1.05;
//                300: 0.96-1.05, 0.92-1.00; 650 and more: 0.94-1.00; unpadded q = 33 to 63: 1.25-1.67
//   16 columns   padded rows: 0.92-1.00; unpadded q = 24, 40, 48: 0.96-1.00; q = 33, 50, 63: 1.01-1.18
bool streams(const LayerInfo &L, int rc) {
    if (rc < kWideCols) return L.q % 32 == 0;
    if (rc < kMaxCols) return L.q % 16 == 0 || L.q >= 256;
    return L.ld % 8 == 0;
}
// Whether runs that write every second round gain on this layer.  Measured as above, time of a run over the plain
// run's: up to 2 columns q = 6 to 24: 1.03-1.19, 32 and more: 0.81-0.98; 4 columns q % 32 == 0: 0.97-1.02,
// q = 12 to 300: 0.98-1.04, 577: 0.94-0.96, 4607: 0.88.
bool gains_behind(const LayerInfo &L, int rc) {
    if (rc <= 2) return L.q >= 32;
    return L.q % 32 == 0 || L.q >= 512;
}

// Whether the narrow kernels gain from units of four floats on this layer's rows (a multiple of four, or not: see
// row_body).  They make a quarter of the accesses, but their tiles are four times as wide: a small set has too few
// of them, and the Q-sweep's row blocks get shorter and its partial sums more.  Measured on single
// matrices, time in the dividing width / in units of four, SGD round and run, rings and a tree, ranks 1 and 2:
//   odd q up to 128 (18 to 113): 1.0-1.4 at 1 to 30 MB, 1.1-2.4 above;  175 to 4607: 0.88-1.09 at 1 and 8 MB, 0.71-1.07
//   at 30 MB, 0.98-1.12 at 40 MB, 0.97-1.19 at 55 MB; at 2 columns 0.99-1.13 at 80 MB, 1.07-1.27 at 150 MB; at 4 columns
//   0.90-1.03 at 80 MB (eight rows per lane group from 64 MB on; 235 columns, one step of a wavefront, 1.20 at 77 MB),
//   0.93-1.13 at 150 MB; 1.02-1.48 at 450 MB
//   even q above 128: 0.86-1.04 at 40 and 62 MB, 0.86-1.10 at 150 MB; 300 to 800 MB: 202 to 4606 columns 1.00-1.24
//   at 2 stacked columns, 130 columns 0.94; at 4 stacked columns 510 to 4606 columns 0.93-1.09, 130 to 310 0.86-1.06
// Workers with few columns in a layer that others take in wide kernels keep the tiles of those (trees at ranks 2 to 4, 3
// to 120 MB, SGD round and run): 8 columns, odd q 37 to 117: 0.95-1.10, 135 and 155: 0.90-1.01, 175 to 513: 0.97-1.32, even
// 62 to 254: 0.89-1.03, 510: 1.00-1.09; 16 columns, odd q 37 to 513: 0.71-1.02, 801 to 8191: 0.97-1.07, even: 0.83-1.00.
bool gains_units_of_four(const LayerInfo &L, int rc, double total_bytes, const Plan &P) {
    if (L.q % 4 == 0 || L.q < kAnyAlignCols) return false;
    const bool odd = L.q % 2 != 0;
    if (rc >= kMaxCols) return odd && L.q >= 768;
    if (rc >= kWideCols) return odd ? L.q <= 128 || L.q >= 168 : L.q >= 400;
    if (L.q <= 128) return true;
    if (!odd) return P.large && L.q >= (rc <= 2 ? 192 : 512);
    return total_bytes >= (double)(rc <= 2 || P.light || L.q <= 256 ? kOddLongBytes : kOddLongBytes4);
}
// The wide kernels, on padded rows.  Measured over 600 drawn sets, time in the dividing width / in units of four:
// odd q 0.94-2.1 (49 of 53 above 1).  Even q in light sets: 8 columns 70 to 342 columns 0.88-0.98, 510 to 5222 columns
// 1.04-1.22; 16 columns 174 to 2434 columns 0.94-1.04; in larger sets 1.03-1.11 (2906 to 4942 columns, 73 to 602 MB; 650
// columns, 850 MB: SGD round 2.87 -> 2.74 ms).
bool gains_wide_units(const LayerInfo &L, int rc, const Plan &P) {
    return L.q % 2 != 0 || !P.light || (rc < kMaxCols && L.q >= 512);
}

// Whether a layer fits the edge kernels with `nt` threads, and then the threads side by side over a row's units
// (log2): as many as the rows leave, no more than a row has units.
static bool edge_split(const LayerInfo &L, int nt, int &tc_shift) {
    if (L.r > kEdgeMaxRank || L.p > nt) return false;
    const int nv = (L.q + 3) / 4;
    tc_shift = 0;
    while ((int64_t)L.p << (tc_shift + 1) <= nt && (1 << tc_shift) < nv) ++tc_shift;
    return (nv + (1 << tc_shift) - 1) >> tc_shift <= kEdgeUnits && edge_lds(L.p, L.q, L.r, tc_shift, nt, 0).bytes <= kEdgeLdsBytes;
}

// What applying a pending update of R columns, both ends together, adds to an edge kernel, in units of 1/30 us: vectors staged four at a time, a loop of
// loads each, and a multiply-add per column and unit.  (Least squares over 388 sets, us: 0.39 per staging step, 0.034 per column and unit; the launch that it
// saves 5.2.  Single rows of 4000 to 6000 floats and work-groups with 16 or more columns lost up to 1.7 times.)
static int edge_run_cost(const LayerInfo &L, int nt, int tc_shift, int R) {
    const int nv = (L.q + 3) / 4, units = (nv + (1 << tc_shift) - 1) >> tc_shift;
    const int stage = (R + 3) / 4 * ((std::max(L.p, L.q) + nt - 1) / nt);
    return 12 * stage + R * units;
}

// Whether a set gains from edge sweeps.  They read the parameters once per power step where the streaming kernels read them twice, and
// three launches make a round where those need five, and on a graph of mixed degrees five kinds of row and column kernels one after the other.
// Against that stand their work per edge instead of per worker and, at higher ranks, column sums that leave few wavefronts per SIMD.
// Time of the streaming kernels over that of the sweeps, 400 drawn sets of 0.1 to 950 MB, single rounds and SGD rounds:
//   rank 1                            1.1-1.5, a few sets of three workers or few row blocks 0.75-1.0; VGG-16 on a ring of 16 1.10
//   rank 2, q up to 900               1.1-1.6;  q above 900: 0.6-1.0 (VGG-16 0.90)
//   rank 3 and 4, q up to 512         1.1-1.6;  q above 512: 0.3-1.1 (4 x 4 torus, 650 columns, 2.8 GB: 0.78)
//   mixed degrees (trees, hubs)       rank 1 and 2 1.2-2.3, ranks 3 and 4 1.1-1.8; above 160 MB with long rows at rank 2 and more 0.66-1.1
static bool gains_sweeps(const Plan &P, size_t max_deg, double total_bytes) {
    size_t min_deg = max_deg;
    for (const auto &inc : P.incident)
        if (!inc.empty()) min_deg = std::min(min_deg, inc.size());
    double heavy = 0.0;
    for (const LayerInfo &L : P.layers)
        if ((L.r >= 3 && L.q > 512) || (L.r == 2 && L.q > 900)) heavy += (double)L.p * L.q;
    const bool mixed = min_deg < max_deg && total_bytes <= (double)kSweepMixedBytes;
    return mixed || heavy <= 0.25 * P.elems_per_worker;
}
// Threads side by side over a row's units (log2) and units per thread of the edge sweeps: the split that covers the row with the
// fewest idle units, of those the one with the most units per thread.  Five units are compiled at rank 1 only: their sums in double are
// 40 registers per column, at rank 3 and 4 more than half of what a thread has; at rank 2 they have not been tried.
static bool sweep_split(const LayerInfo &L, int nt, int rank, int max_units, SweepDesc &d) {
    const int nv = (L.q + 3) / 4;
    int best = 0;
    d.exact = (int64_t)L.p * L.q <= kSweepExactSize && (int64_t)L.p * L.r <= (L.q < 4 ? kSweepExactSize : kSweepExactRows);
    for (int units : {1, 2, 3, 5}) {
        if (units > 3 && (rank > 1 || max_units < 5)) break;
        if (d.exact && units != 1 && units != 3) continue;
        int sh = 0;
        while ((units << sh) < nv) ++sh;
        if ((1 << sh) > nt) continue;
        if (best == 0 || units << sh <= best) {
            best = units << sh;
            d.tc_shift = sh;
            d.units = units;
        }
    }
    if (best == 0) d.tc_shift = d.units = d.exact = 0;
    return best > 0;
}
// Rows a work-group takes per step (see sweep_tile).
static int sweep_step_rows(const LayerInfo &L, int nt, int rank, const SweepDesc &d) {
    if (L.q < 4) return nt;
    if (d.units == 0) return 1;
    const int m = d.exact ? (d.units == 1 ? 2 : 1) : d.units == 1 ? 4 : d.units == 5 || (d.units == 3 && rank > 2) ? 1 : 2;
    return (nt >> d.tc_shift) * m;
}

// Time of a power step, us, with the edge sweeps and with the streaming kernels, and what a run of the latter saves per round by its fused pass.
// Least squares (of the logarithm) over 2200 drawn sets of 0.04 MB to 4 GB -- rings, trees, tori, stars, hypercubes, complete graphs and circulants of degree
// up to 23, rows of 1 to 80000 floats, up to 4000 layers, 2 to 40 workers -- each called both ways: 80 % of the estimates lie within 20 % for the sweeps,
// within 30 % for the streaming kernels.
struct StepTimes {
    double sweep, stream, fused;
};
static StepTimes step_times(const Plan &P) {
    const int k = P.max_layer_rank <= 1 ? 0 : P.max_layer_rank <= 2 ? 1 : 2, nt = P.sweep_threads;
    StepTimes T;
    // The sweep: the work-groups of a die side by side on its 32 CUs (two of 256 threads each, one of 512), then the longest alone.  Work in units of
    // four floats that one thread takes.
    std::vector<double> load(8, 0.0);
    double longest = 0.0, sums = 0.0, long_rows = 0.0;
    int blocks = 0;
    for (size_t i = 0; i < P.sweep_tiles.size(); ++i) {
        const SweepTile &t = P.sweep_tiles[i];
        if (t.nrows <= 0) continue;
        double work = 8.0;
        if (t.blk >= 0) {
            const SweepDesc &d = P.sweep_descs[t.el];
            const LayerInfo L{d.p, d.q, d.r, 0, 0, d.ld, 0};
            const int rows = sweep_step_rows(L, nt, P.max_layer_rank, d);
            const double units = d.q < 4 ? 1.0 : d.units ? (double)rows / (nt >> d.tc_shift) * d.units : d.q / (4.0 * nt);
            work += (t.nrows + rows - 1) / rows * units * (d.exact ? 2 : 1);
        }
        load[i & 7] += work;
        longest = std::max(longest, work);
    }
    for (const SweepDesc &d : P.sweep_descs) {
        blocks = std::max(blocks, d.nblk);
        if (d.q >= 4 && d.units == 0) long_rows += 8e-6 * d.p * d.q;
        else sums += 16e-6 * d.nblk * d.r * d.q;
    }
    const double all = *std::max_element(load.begin(), load.end()) / (nt == 256 ? 64 : 32), wide = nt == 256 ? 1.0 : 1.36;
    const double per_unit[] = {0.24, 0.38, 0.64}, alone[] = {0.14, 0.25, 0.49}, per_block[] = {0.11, 0.12, 0.26}, per_slot[] = {1.4, 1.4, 4.0};
    T.sweep = 7.0 + wide * (per_unit[k] * all + alone[k] * longest) + per_slot[k] * (double)P.sweep_tiles.size() / 512 +  // sweep
              per_block[k] * blocks + 0.6 * sums + 0.2 * long_rows;                                                       // finish, MB
    // The streaming kernels: launches of every class, the longest tile of each, the partial sums, both reads.
    int widest = 1, segments = 1, rblocks = 1;
    double tiles = 0.0;
    for (const RowClass &rc : P.row_classes) {
        double most = 0.0;
        for (const RowTile &t : rc.tiles) {
            const PairDesc &pd = P.pairs[t.pair];
            const double w = pd.q == 1 ? t.nrows / 64.0 : (double)t.nrows * std::min(pd.seg_len, pd.q) / (64.0 * pd.V);
            most = std::max(most, rc.RC >= kWideCols && pd.q > 1 ? w / 4 : w);
        }
        tiles += most;
        widest = std::max(widest, rc.RC);
    }
    for (const EdgeLayerDesc &d : P.els) {
        segments = std::max(segments, d.nseg);
        rblocks = std::max(rblocks, d.nblk);
    }
    const double read = (widest < kWideCols ? 0.16 : widest == kWideCols ? 0.12 : 0.15) * 4e-6 * P.pass_elems;
    const size_t launches = P.row_classes.size() + P.col_classes.size();
    T.stream = 6.3 + 4.4 * launches + 0.17 * tiles + 0.14 * segments + 0.27 * rblocks + 2.4e-6 * P.part_bytes + 2.0 * read;
    T.fused = 4.4 * P.row_classes.size() + 0.4 * read;
    return T;
}
// What the streaming kernels' time has to be of the sweeps'.  2477 other drawn sets that the rule above takes, single rounds and runs of two and of five,
// faster or slower by more than 4 % (10 %) in every call, or in some: all of them with the sweeps, 214 (126) slower; with the sets that these lines leave
// on the streaming kernels, 93 (35) slower and 103 (68) left that would have been faster; at 0.95 and 1.2, 68 (20) and 275 (199).  Sets of few workers, whose
// streaming passes are short, and of many edges per worker are overrated by the estimate.
constexpr double kSweepGain = 0.85, kSweepGainFew = 1.0;
static bool sweeps_are_faster(const Plan &P) {
    const StepTimes T = step_times(P);
    int workers = 0;
    for (const auto &inc : P.incident) workers += !inc.empty();
    const double need = workers <= 4 || P.n_edges >= 4 * workers ? kSweepGainFew : kSweepGain;
    // (where runs write every second round, they and single rounds stay with the streaming kernels: what is left are SGD rounds)
    return P.steps * T.stream - (P.lazy ? 0.0 : T.fused) >= need * P.steps * T.sweep;
}

int build_plan(Plan &P, int n_workers, int n_edges, const int32_t *edges, const float *edge_w,
               int n_layers, const int32_t *rows, const int32_t *cols, int rank, int power_steps,
               const Tuning &tune) {
    if (n_workers < 1 || n_edges < 0 || n_layers < 1 || rank < 1 || power_steps < 1) return PG_ERR_ARG;
    if ((n_edges > 0 && (!edges || !edge_w)) || !rows || !cols) return PG_ERR_ARG;

    P.n = n_workers;
    P.n_edges = n_edges;
    P.n_layers = n_layers;
    P.rank = rank;
    P.steps = power_steps;
    P.mfma_cols = tune.mfma_cols;
    P.edges.assign(edges, edges + 2 * (size_t)n_edges);
    P.edge_w.assign(edge_w, edge_w + n_edges);

    // ---- topology (graph G and mixing weights W, assumption A4) ----
    std::set<std::pair<int, int>> seen;
    P.incident.assign(n_workers, {});
    std::vector<double> wsum(n_workers, 0.0);
    for (int e = 0; e < n_edges; ++e) {
        int a = edges[2 * e], b = edges[2 * e + 1];
        if (a < 0 || b < 0 || a >= n_workers || b >= n_workers || a == b) return PG_ERR_TOPOLOGY;
        if (!seen.insert({std::min(a, b), std::max(a, b)}).second) return PG_ERR_TOPOLOGY;
        float w = edge_w[e];
        if (!std::isfinite(w) || w < 0.0f) return PG_ERR_ARG;
        wsum[a] += w;
        wsum[b] += w;
        P.incident[a].push_back(e);
        P.incident[b].push_back(e);
    }
    for (int i = 0; i < n_workers; ++i)
        if (wsum[i] > 1.0 + 1e-6) return PG_ERR_ARG;  // the self-weight W_ii would be negative

    size_t max_deg = 0;
    for (int i = 0; i < n_workers; ++i) max_deg = std::max(max_deg, P.incident[i].size());

    // ---- layers: every weight and bias is its own matrix (Section 2) ----
    P.layers.resize(n_layers);
    int64_t off = 0;
    P.elems_per_worker = 0;
    P.message_floats = 0;
    for (int l = 0; l < n_layers; ++l) {
        int p = rows[l], q = cols[l];
        if (p < 1 || q < 1) return PG_ERR_SHAPE;
        LayerInfo &L = P.layers[l];
        L.p = p;
        L.q = q;
        L.r = std::min(rank, std::min(p, q));
        P.max_layer_rank = std::max(P.max_layer_rank, L.r);
        P.max_rows = std::max(P.max_rows, p);
        L.V = (q % 4 == 0) ? 4 : (q % 2 == 0 ? 2 : 1);
        // Row stride.  With 8 or more stacked columns a tile's wavefronts work side by side on
        // 64-column (256-byte) pieces of the same rows; when rows start at arbitrary addresses every
        // piece ends inside a 128-byte line that the neighbouring wavefront touches at another time,
        // and the line crosses the memory interface twice (measured on 650-float rows: a third more
        // bytes read, a quarter more written).  Rows of such layers start on line boundaries.
        const int per_pass = std::min<int>((int)max_deg, std::max(1, kMaxCols / L.r));  // edges one pass takes
        const bool shared_rows = compiled_cols(std::max(1, per_pass * L.r)) >= kWideCols;
        L.ld = (shared_rows && q >= 64) ? (int)round_up(q, 32) : q;
        L.x_off = off;
        off = round_up(off + (int64_t)p * L.ld, 32);
        P.elems_per_worker += (double)p * q;
        P.message_floats += (size_t)L.r * ((size_t)p + q);
    }
    P.param_floats = (size_t)off;
    for (int l = 0; l < n_layers; ++l)
        if (P.layers[l].r > kMaxCols) return PG_ERR_ARG;  // one edge's columns must fit one pass

    // ---- projection state: edge-major, then layer, r_l columns of q_l floats ----
    P.q_off.resize((size_t)n_edges * n_layers);
    P.ph_off.resize((size_t)n_edges * n_layers);
    P.flag_off.resize((size_t)n_edges * n_layers);
    int64_t qo = 0, pho = 0, flo = 0, pdo = 0;
    std::vector<int64_t> pd_off((size_t)n_edges * n_layers);
    for (int e = 0; e < n_edges; ++e)
        for (int l = 0; l < n_layers; ++l) {
            const LayerInfo &L = P.layers[l];
            size_t id = (size_t)e * n_layers + l;
            P.q_off[id] = qo;
            qo = round_up(qo + (int64_t)L.q * L.r, 4);
            P.ph_off[id] = pho;
            pho = round_up(pho + (int64_t)L.p * L.r, 4);
            pd_off[id] = pdo;
            pdo += (int64_t)L.p * L.r;
            P.flag_off[id] = flo;
            flo += L.r;
        }
    P.qstate_floats = (size_t)qo;
    P.pstate_floats = (size_t)pho;

    // ---- tile sizes: the byte targets suit workloads that fill the chip many times over; small
    // parameter sets are cut finer so that every SIMD still gets a tile ----
    Tuning tn = tune;
    const double total_bytes = 4.0 * n_workers * P.elems_per_worker;
    {
        const double slots = 4096.0;  // 256 CUs x 4 SIMDs x a few wavefronts
        P.light = tune.light < 0 ? total_bytes <= (double)kLightBytes : tune.light != 0;
        bool wide = false;  // some worker has 8 or more stacked columns in a pass
        double streamed = 0.0, behind = 0.0, elems = 0.0;
        for (const LayerInfo &L : P.layers) {
            const int per_pass = std::min<int>((int)max_deg, std::max(1, kMaxCols / L.r));
            const int rc = compiled_cols(std::max(1, per_pass * L.r));
            const double n_el = (double)L.p * L.q;
            wide = wide || rc >= kWideCols;
            elems += n_el;
            if (streams(L, rc)) streamed += n_el;
            if (gains_behind(L, rc)) behind += n_el;
        }
        P.large = tune.stream < 0 ? total_bytes > (double)(wide ? kStreamBytesWide : kStreamBytes) : tune.stream != 0;
        P.stream = tune.stream < 0 ? P.large && streamed >= kStreamShare * elems : tune.stream != 0;
        P.lazy = tune.lazy < 0 ? P.large && behind >= kStreamShare * elems : tune.lazy != 0;
        tn.row_tile_bytes = (int)std::max((P.light ? 4.0 : 8.0) * 1024, std::min((double)tune.row_tile_bytes, total_bytes / slots));
        tn.col_tile_bytes = (int)std::max(32.0 * 1024, std::min((double)tune.col_tile_bytes, 4.0 * total_bytes / slots));
        tn.wide_tile_bytes = (int)std::max(32.0 * 1024, std::min((double)tune.wide_tile_bytes, 4.0 * total_bytes / slots));
        tn.mcol_tile_bytes = (int)std::max(64.0 * 1024, std::min((double)tune.mcol_tile_bytes, 8.0 * total_bytes / slots));
    }

    // ---- workspace sections, given the doubles of the P- and Q-partials ----
    int64_t orth_chunks = 0;  // tall layers: row chunks for the two-kernel orthonormalisation (36 Gram sums per chunk)
    {
        bool tall = false;
        for (const LayerInfo &L : P.layers) tall = tall || L.p > kOrthTallRows;
        if (tall)
            for (const LayerInfo &L : P.layers) orth_chunks += (int64_t)n_edges * ((L.p + kOrthChunkRows - 1) / kOrthChunkRows);
    }
    auto sections = [&](int64_t pwo, int64_t qwo) {
        size_t o = 0;
        P.ws_pw = o;
        o = (size_t)round_up(o + (size_t)pwo * 8, 256);
        P.ws_qw = o;
        o = (size_t)round_up(o + (size_t)qwo * 8, 256);
        P.ws_pd = o;
        o = (size_t)round_up(o + (size_t)pdo * 8, 256);
        P.ws_ph = o;
        o = (size_t)round_up(o + (size_t)pho * 4, 256);
        P.ws_flag = o;
        o = (size_t)round_up(o + (size_t)flo * 4, 256);
        P.ws_gpart = o;
        o = (size_t)round_up(o + (size_t)orth_chunks * 36 * 8, 256);
        // unit vectors in R^q of Algorithm 2's odd iterations (state layout)
        P.ws_uq = o;
        o = (size_t)round_up(o + (size_t)qo * 4, 256);
        P.ws_bytes = std::max<size_t>(o, 256);
    };

    // ---- per-layer launch geometry ----
    struct Geo {
        int lpr, nseg, seg_len, rows_iter_base;  // row-owner
        int wc;                                  // matrix-core row tiles: wavefronts across the column steps
        bool wide;                               // row-owner: many stacked columns, Q slice in LDS
        bool mrow;                               // row-owner: matrix-core tiles
        bool units;                              // wide kernels: units of four floats
        int lg, nblk, blk_rows;                  // column-owner
    };
    std::vector<Geo> geo(n_layers);
    // The geometry under the settings `t` for rows of odd length; sets the workspace sections.
    auto lay_out = [&](const Tuning &t) {
        double odd = 0.0;  // elements in rows that units of four floats speed up
        for (LayerInfo &L : P.layers) {
            const int per_pass = std::min<int>((int)max_deg, std::max(1, kMaxCols / L.r));
            const int rc = compiled_cols(std::max(1, per_pass * L.r));
            const bool gains = t.odd_rows < 0 ? gains_units_of_four(L, rc, total_bytes, P)
                                              : t.odd_rows != 0 && L.q >= kAnyAlignCols;
            L.Vn = gains ? 4 : L.V;
            if (L.Vn > L.V) odd += (double)L.p * L.q;
        }
        P.odd_rows = t.odd_rows < 0 ? odd >= kOddShare * P.elems_per_worker && odd > 0.0 : t.odd_rows != 0;
        if (!P.odd_rows)
            for (LayerInfo &L : P.layers) L.Vn = L.V;
        // Wide kernels in units of four floats on padded rows.  Every vector width is a launch of its own,
        // so in a small set whose other layers need another width anyway the split costs more than the
        // wider accesses save (11 workers, 115 MB, eight layers of odd lengths: 447 -> 475 us per SGD
        // round); in large ones, or where all rows are padded, it pays.  For the same reason a layer that gains nothing
        // by itself goes along with others that are moved in units of four anyway (143 x 32, 378 x 182, 72 x 345 and 83 x 36
        // on a 3x3 torus at rank 3, one round: 60 us with a launch of its own for the even rows, 39 us without).
        bool all_padded = true, some_units = false;
        for (const LayerInfo &L : P.layers) {
            const int per_pass = std::min<int>((int)max_deg, std::max(1, kMaxCols / L.r));
            const int rc = compiled_cols(std::max(1, per_pass * L.r));
            all_padded = all_padded && L.ld % 4 == 0;
            if (rc >= kWideCols && L.ld % 4 == 0) some_units = some_units || L.q % 4 == 0 || gains_wide_units(L, rc, P);
        }
        const bool wide_units = tune.mfma_cols && (t.wide_units < 0 ? some_units && (P.large || all_padded) : t.wide_units != 0);
        constexpr int kColUnroll = 8;
        for (int l = 0; l < n_layers; ++l) {
            const LayerInfo &L = P.layers[l];
            Geo &g = geo[l];
            // The row blocking depends on the stacked column count; size for the best-connected worker.
            // (a worker with more than kMaxCols stacked columns takes several passes of whole edges)
            const int per_pass = std::min<int>((int)max_deg, std::max(1, kMaxCols / L.r));
            int rc_max = compiled_cols(std::max(1, per_pass * L.r));
            g.wide = rc_max >= kWideCols;
            const int Vg = g.wide ? L.V : L.Vn;
            const int nv = (L.q + Vg - 1) / Vg;  // vector loads per row
            // Row passes on the matrix cores pay from 16 stacked columns on (measured: at 8 the vector
            // kernels' P-sweep is the faster one) and address a layer with 32-bit byte offsets.
            g.mrow = tune.mfma_rows && rc_max >= tune.mfma_row_cols && (int64_t)L.p * L.ld < ((int64_t)1 << 30);
            // Lanes per row: a whole wavefront for few stacked columns; 16 for many, where the
            // per-row lane reduction (RC values per row) would otherwise rival the products.
            g.lpr = std::min((g.wide && !g.mrow) ? 16 : 64, pow2_ceil(nv));
            g.units = g.wide && wide_units && L.ld % 4 == 0;
            const int wide_V = g.units ? 4 : Vg;  // width of the wide kernels' accesses to X
            int chunk = g.lpr * wide_V;  // floats one lane group covers per step
            int nchunks = (L.q + chunk - 1) / chunk;
            int seg_chunks;
            if (!g.wide) {
                // one wavefront per tile: column segments keep a tile near the byte target when a
                // single row is long
                int rows_iter = (64 / g.lpr) * rows_unroll(rc_max, P.light);
                int64_t chunk_bytes = (int64_t)rows_iter * chunk * 4;
                seg_chunks = (int)std::max<int64_t>(1, tn.row_tile_bytes / chunk_bytes);
                g.rows_iter_base = 64 / g.lpr;
            } else if (g.mrow) {
                // matrix cores: steps of 64 columns; a row is cut only when it is very long
                chunk = 64;
                nchunks = (L.q + chunk - 1) / chunk;
                seg_chunks = kMfmaSegCols / chunk;
                g.rows_iter_base = 64 / g.lpr;  // for this layer's workers with few stacked columns
            } else {
                // four wavefronts per tile share the Q slice in LDS: RC * seg_len floats must fit
                seg_chunks = std::max(1, kWideLdsBytes / (rc_max * 4) / chunk);
                g.rows_iter_base = (kThreads / 64) * (64 / g.lpr);
            }
            g.nseg = (nchunks + seg_chunks - 1) / seg_chunks;
            seg_chunks = (nchunks + g.nseg - 1) / g.nseg;
            g.nseg = (nchunks + seg_chunks - 1) / seg_chunks;
            g.seg_len = seg_chunks * chunk;
            g.wc = 1;
            if (g.mrow) g.wc = seg_chunks >= 4 ? 4 : (seg_chunks >= 2 ? 2 : 1);

            // Column-owner kernel: lanes side by side over columns; pick the lane-group width that
            // wastes the fewest lanes on the ragged end of a row (ties go to the wider group).
            int best = 64;
            double best_util = -1;
            for (int lg : {64, 32, 16}) {
                int lgc = std::min(lg, pow2_ceil(nv));
                int groups = (nv + lgc - 1) / lgc;
                double util = (double)nv / ((double)groups * lgc);
                if (util > best_util + 0.05) {
                    best_util = util;
                    best = lgc;
                }
            }
            // With many stacked columns the kernel is bound by arithmetic and LDS reads of Phat, and
            // one row per wavefront (all 64 lanes side by side) with shorter row blocks measures best.
            const bool col_heavy = rc_max >= 16;
            if (col_heavy && (double)nv / ((double)((nv + 63) / 64) * 64) > 0.6) best = std::min(64, pow2_ceil(nv));
            g.lg = best;
            int row_groups = 4 * (64 / g.lg);
            int64_t row_bytes = (int64_t)g.lg * (t.long_blocks ? L.V : Vg) * 4;
            int64_t want = std::max<int64_t>(1, tn.col_tile_bytes / row_bytes);
            int64_t unit = (int64_t)row_groups * kColUnroll;
            if (g.wide && tune.mfma_cols) {
                // four wavefronts per tile of kMfmaTileCols columns
                want = std::max<int64_t>(16, tn.mcol_tile_bytes / (kMfmaTileCols * 4));
                unit = 16;
            }
            int64_t br = round_up(want, unit);
            if (!(g.wide && tune.mfma_cols)) {
                // the vector column kernel stages the block's Phat slice in LDS: (rows + 1) x columns floats
                const int64_t cap = kColLdsBytes / (4 * rc_max) - 1;
                if (br > cap) br = cap >= unit ? cap / unit * unit : cap;
            }
            if (br >= L.p) br = L.p;
            g.blk_rows = (int)br;
            g.nblk = (L.p + g.blk_rows - 1) / g.blk_rows;
        }
        // every edge brings r columns to the partials of both its ends
        int64_t pw = 0, qw = 0;
        for (int l = 0; l < n_layers; ++l) {
            const int64_t c2 = 2 * (int64_t)n_edges * P.layers[l].r;
            pw += geo[l].nseg * c2 * P.layers[l].p;
            qw += geo[l].nblk * c2 * P.layers[l].q;
        }
        sections(pw, qw);
    };
    lay_out(tune);
    // Units of four floats on rows of odd length change the segments and row blocks and with them the
    // number of partial sums, mostly upwards.  A problem that does not fit the static workspace that
    // way is planned with longer row blocks if it fits then, next with the widths that divide its rows
    // (54126 x 1162 on a ring of 8 at rank 2: 56.0 MB, 30.1 MB with the dividing widths; 23961 x 626 on
    // a ring of 20 at rank 2: 36.7 MB with those, 31.9 MB with units of four and longer blocks).
    if (tune.odd_rows < 0 && tune.wide_units < 0 && P.ws_bytes > (size_t)PG_STATIC_WORKSPACE_BYTES) {
        Tuning other[5] = {tune, tune, tune, tune, tune};
        other[0].long_blocks = true;
        other[1].odd_rows = other[1].wide_units = 0;
        other[2].odd_rows = 1;
        other[3].odd_rows = 1;
        other[3].long_blocks = true;
        for (const Tuning &t : other) {  // the last one, where none fits: as at first
            lay_out(t);
            if (P.ws_bytes <= (size_t)PG_STATIC_WORKSPACE_BYTES) break;
        }
    }

    // ---- (worker, layer) pairs with their stacked columns ----
    // A worker multiplies its matrix by the columns of all its incident edges in one pass when
    // they number at most kMaxCols; otherwise its edges are split into groups of whole edges,
    // one PairDesc (one pass over the matrix) per group.
    P.pairs.clear();
    P.pair_first.assign((size_t)n_layers * n_workers, 0);
    P.pair_count.assign((size_t)n_layers * n_workers, 0);
    P.max_groups = 1;
    P.cols.clear();
    int64_t pwo = 0, qwo = 0;
    // per (layer, worker, incident slot): which group the edge is in, and its first column there
    std::vector<std::vector<std::pair<int, int>>> slot_home((size_t)n_layers * n_workers);
    for (int l = 0; l < n_layers; ++l) {
        const LayerInfo &L = P.layers[l];
        const Geo &g = geo[l];
        const int epg = std::max(1, kMaxCols / L.r);  // edges per group
        for (int i = 0; i < n_workers; ++i) {
            const auto &inc = P.incident[i];
            const size_t li = (size_t)l * n_workers + i;
            const int ngroups = std::max<int>(1, ((int)inc.size() + epg - 1) / epg);
            P.pair_first[li] = (int)P.pairs.size();
            P.pair_count[li] = ngroups;
            P.max_groups = std::max(P.max_groups, ngroups);
            slot_home[li].resize(inc.size());
            for (int gi = 0; gi < ngroups; ++gi) {
                const int s0 = gi * epg, s1 = std::min<int>((int)inc.size(), s0 + epg);
                PairDesc pd;
                pd.worker = i;
                pd.p = L.p;
                pd.q = L.q;
                pd.R = (s1 - s0) * L.r;
                pd.x_off = L.x_off;
                pd.pw_off = pwo;
                pd.qw_off = qwo;
                pd.col0 = (int)P.cols.size();
                pd.lpr = g.lpr;
                pd.nseg = g.nseg;
                pd.seg_len = g.seg_len;
                pd.lg = g.lg;
                pd.nblk = g.nblk;
                pd.blk_rows = g.blk_rows;
                pd.V = L.V;
                pd.wc = g.wc;
                pd.ld = L.ld;
                pwo += (int64_t)g.nseg * pd.R * L.p;
                qwo += (int64_t)g.nblk * pd.R * L.q;
                for (int sl = s0; sl < s1; ++sl) {
                    const int e = inc[sl];
                    slot_home[li][sl] = {(int)P.pairs.size(), (sl - s0) * L.r};
                    for (int k = 0; k < L.r; ++k) {
                        ColDesc c;
                        size_t id = (size_t)e * n_layers + l;
                        c.q_off = P.q_off[id] + (int64_t)k * L.q;
                        c.ph_off = P.ph_off[id] + (int64_t)k * L.p;
                        c.coef = (P.edges[2 * e] == i) ? P.edge_w[e] : -P.edge_w[e];
                        c.pad = 0;
                        P.cols.push_back(c);
                    }
                }
                P.pairs.push_back(pd);
                P.pair_group.push_back(gi);
                P.pair_layer.push_back(l);
            }
        }
    }

    // ---- (edge, layer) records ----
    P.els.resize((size_t)n_layers * n_edges);
    P.comb_tiles.clear();
    for (int l = 0; l < n_layers; ++l) {
        const LayerInfo &L = P.layers[l];
        const Geo &g = geo[l];
        for (int e = 0; e < n_edges; ++e) {
            EdgeLayerDesc &d = P.els[(size_t)l * n_edges + e];
            int a = P.edges[2 * e], b = P.edges[2 * e + 1];
            auto home = [&](int w) {
                const auto &inc = P.incident[w];
                const int sl = (int)(std::find(inc.begin(), inc.end(), e) - inc.begin());
                return slot_home[(size_t)l * n_workers + w][sl];
            };
            const std::pair<int, int> ha = home(a), hb = home(b);
            const PairDesc &pa = P.pairs[ha.first];
            const PairDesc &pb = P.pairs[hb.first];
            const int ja = ha.second, jb = hb.second;
            size_t id = (size_t)e * n_layers + l;
            d.p = L.p;
            d.q = L.q;
            d.r = L.r;
            d.nseg = g.nseg;
            d.nblk = g.nblk;
            d.pad = 0;
            d.pwa_off = pa.pw_off + (int64_t)ja * L.p;
            d.pwb_off = pb.pw_off + (int64_t)jb * L.p;
            d.pwa_seg = (int64_t)pa.R * L.p;
            d.pwb_seg = (int64_t)pb.R * L.p;
            d.qwa_off = pa.qw_off + (int64_t)ja * L.q;
            d.qwb_off = pb.qw_off + (int64_t)jb * L.q;
            d.qwa_blk = (int64_t)pa.R * L.q;
            d.qwb_blk = (int64_t)pb.R * L.q;
            d.pd_off = pd_off[id];
            d.ph_off = P.ph_off[id];
            d.q_off = P.q_off[id];
            d.flag_off = P.flag_off[id];
            int64_t total = (int64_t)L.r * L.q;
            for (int64_t f = 0; f < total; f += kThreads)
                P.comb_tiles.push_back({(int32_t)((size_t)l * n_edges + e), (int32_t)f});
        }
    }

    sections(pwo, qwo);
    P.orth_tiles.clear();
    if (orth_chunks > 0) {
        for (size_t el = 0; el < P.els.size(); ++el) {
            const int p = P.els[el].p;
            const int nch = (p + kOrthChunkRows - 1) / kOrthChunkRows;
            for (int ch = 0; ch < nch; ++ch)
                P.orth_tiles.push_back({(int32_t)el, ch * kOrthChunkRows,
                                        std::min(kOrthChunkRows, p - ch * kOrthChunkRows), ch, nch, 0});
        }
    }

    // ---- tiles, grouped by kernel instantiation, in address order ----
    P.row_classes.clear();
    P.col_classes.clear();
    P.isolated_pairs.clear();
    P.isolated_elems = 0;
    P.pass_elems = 0;
    // many stacked columns: one class (one kernel instantiation) per vector width
    // (tiles of different column groups of one matrix must not update it at the same time: every
    // group index has launches of its own)
    auto row_class = [&](int RC, int V, bool mfma, int group, bool vec) -> size_t {
        if (RC < kWideCols) V = 0;
        for (size_t k = 0; k < P.row_classes.size(); ++k)
            if (P.row_classes[k].RC == RC && P.row_classes[k].V == V && P.row_classes[k].mfma == mfma &&
                P.row_classes[k].group == group && P.row_classes[k].vec == vec)
                return k;
        P.row_classes.push_back({RC, V, mfma, {}, 0, 0, 0, group, false, vec});
        return P.row_classes.size() - 1;
    };
    auto col_class = [&](int RC, int V, bool vec) -> size_t {
        if (RC < kWideCols) V = 0;
        for (size_t k = 0; k < P.col_classes.size(); ++k)
            if (P.col_classes[k].RC == RC && P.col_classes[k].V == V && P.col_classes[k].vec == vec) return k;
        P.col_classes.push_back({RC, V, {}, 0, 0, 0, vec});
        return P.col_classes.size() - 1;
    };
    // Vector layers (biases, normalisation scales) are a sliver of the bytes; as tiles of the matrix
    // kernels they run at those kernels' low occupancy, one short latency-bound wavefront after the
    // other.  Where there are many of them they get launches of their own with a kernel that needs
    // few registers; where there are few, another launch would cost more than it saves.
    int64_t vec_pairs = 0;
    for (int l = 0; l < n_layers; ++l)
        if (P.layers[l].q == 1)
            for (int i = 0; i < n_workers; ++i) vec_pairs += P.pair_count[(size_t)l * n_workers + i];
    const bool split_vec = tune.vec_kernels >= 2 || (tune.vec_kernels == 1 && vec_pairs >= kVecClassPairs);
    for (int l = 0; l < n_layers; ++l) {
        const LayerInfo &L = P.layers[l];
        const Geo &g = geo[l];
        for (int i = 0; i < n_workers; ++i)
          for (int gi = 0; gi < P.pair_count[(size_t)l * n_workers + i]; ++gi) {
            int pair = P.pair_first[(size_t)l * n_workers + i] + gi;
            const PairDesc &pd = P.pairs[pair];
            if (pd.R == 0) {  // isolated worker: nothing to multiply, no gossip term
                P.isolated_pairs.push_back(pair);
                P.isolated_elems += (double)L.p * L.q;
                continue;
            }
            int RC = compiled_cols(pd.R);
            const bool mrow = g.mrow && RC >= kWideCols;
            // Layers with padded rows are read and written four floats at a time by the wide kernels
            // whatever q is; a row's last unit may reach into the padding (zeroed, never stored).
            const bool wide4 = RC >= kWideCols && g.units;
            const int Vr = wide4 ? 4 : (RC < kWideCols ? L.Vn : L.V);
            const int Vc = wide4 ? 4 : L.V;
            P.pairs[pair].V = Vr;
            const bool vec = split_vec && L.q == 1 && RC < kWideCols;
            RowClass &rc = P.row_classes[row_class(RC, Vr, mrow, gi, vec)];
            rc.pad = rc.pad || (RC >= kWideCols && L.q % Vr != 0);
            int rows_iter = g.rows_iter_base * rows_unroll(RC, P.light);
            int tile_rows;
            if (RC < kWideCols) {
                int iters = 1;
                if (g.nseg == 1) {
                    int64_t bytes_iter = (int64_t)rows_iter * L.q * 4;
                    iters = (int)std::max<int64_t>(1, tn.row_tile_bytes / bytes_iter);
                }
                tile_rows = rows_iter * iters;
                // the vector kernel: one step (four entries per lane) per tile, so that a long vector
                // is several short independent tiles and not one latency-bound loop
                if (vec) tile_rows = 256;
            } else if (mrow) {
                tile_rows = 16 * kMfmaRowBlocks * (4 / g.wc);
            } else {
                // enough rows that staging the Q slice (RC rows' worth of traffic) is amortised
                int64_t seg_bytes = (int64_t)std::min(g.seg_len, L.q) * 4;
                int64_t want = std::max<int64_t>(8 * RC, tn.wide_tile_bytes / seg_bytes);
                tile_rows = (int)(round_up(want, rows_iter));
                rc.max_seg = std::max(rc.max_seg, g.seg_len);
            }
            for (int r0 = 0; r0 < L.p; r0 += tile_rows)
                for (int sg = 0; sg < g.nseg; ++sg)
                    rc.tiles.push_back({pair, r0, std::min(tile_rows, L.p - r0), sg});
            rc.elems += (double)L.p * L.q;
            P.pass_elems += (double)L.p * L.q;

            ColClass &cc = P.col_classes[col_class(RC, Vc, vec)];
            int cw = (RC >= kWideCols && tune.mfma_cols) ? kMfmaTileCols : g.lg * Vr;
            for (int b = 0; b < g.nblk; ++b)
                for (int c0 = 0; c0 < L.q; c0 += cw) cc.tiles.push_back({pair, c0, b, 0});
            cc.elems += (double)L.p * L.q;
            cc.max_rows = std::max(cc.max_rows, g.blk_rows);
        }
    }
    // Runs that write every second round: narrow kernels only, one power step, one column group, and the
    // second Phat buffer lies in the column-by-column Gram-Schmidt's scratch.
    P.lazy = P.lazy && !P.light && P.steps == 1 && P.max_groups == 1 && P.ws_ph - P.ws_pd >= P.pstate_floats * sizeof(float);
    for (const RowClass &rc : P.row_classes) P.lazy = P.lazy && rc.RC <= kLazyCols && !rc.vec;
    for (const ColClass &cc : P.col_classes)
        P.lazy = P.lazy && cc.RC <= kLazyCols && !cc.vec && lazy_col_lds(cc.max_rows, cc.RC) <= (size_t)kLazyColLds;
    // ---- sets of small layers: edge kernels ----
    P.ws_static_bytes = P.ws_bytes;
    P.part_bytes = 8.0 * (double)(pwo + qwo);
    P.edge_tiles.clear();
    P.apply_tiles.clear();
    P.edge_elems = 0;
    P.edge = tune.edge != 0 && n_edges > 0 && P.max_groups == 1 && (tune.edge > 0 || (int64_t)n_edges * n_layers <= kEdgeTiles);
    for (const LayerInfo &L : P.layers) P.edge = P.edge && (tune.edge > 0 || (int64_t)L.p * L.q <= kEdgeSize);
    std::vector<int> shift(n_layers);
    bool fits = false;
    for (int nt : kEdgeThreads) {
        P.edge_threads = nt;
        fits = nt >= tune.edge_threads;
        for (int l = 0; l < n_layers && fits; ++l) fits = edge_split(P.layers[l], nt, shift[l]);
        if (fits) break;
    }
    P.edge = P.edge && fits;
    if (P.edge) {
        std::vector<int> order(n_layers);
        for (int l = 0; l < n_layers; ++l) order[l] = l;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
            return (int64_t)P.layers[a].p * P.layers[a].q > (int64_t)P.layers[b].p * P.layers[b].q;
        });
        for (int l : order) {
            const LayerInfo &L = P.layers[l];
            P.edge_lds = std::max(P.edge_lds, edge_lds(L.p, L.q, L.r, shift[l], P.edge_threads, 0).bytes);
            P.edge_run_lds = std::max(P.edge_run_lds, edge_lds(L.p, L.q, L.r, shift[l], P.edge_threads, 2 * (int)max_deg * L.r).bytes);
            for (int e = 0; e < n_edges; ++e) {
                const int a = P.edges[2 * e], b = P.edges[2 * e + 1];
                const size_t id = (size_t)e * n_layers + l;
                const PairDesc &pa = P.pairs[P.pair_first[(size_t)l * n_workers + a]], &pb = P.pairs[P.pair_first[(size_t)l * n_workers + b]];
                const int own = (P.incident[a][0] == e ? 1 : 0) | (P.incident[b][0] == e ? 2 : 0);
                P.edge_tiles.push_back({L.p, L.q, L.r, L.ld, a, b, shift[l], own, pa.col0, pa.R, pb.col0, pb.R,
                                        L.x_off, P.q_off[id], P.ph_off[id], P.flag_off[id]});
                P.edge_elems += 2.0 * L.p * L.q;
            }
            for (int i = 0; i < n_workers; ++i) {
                const int pair = P.pair_first[(size_t)l * n_workers + i];
                if (P.pairs[pair].R == 0) continue;
                P.apply_cols = std::max(P.apply_cols, compiled_cols(P.pairs[pair].R));
                const int units = L.p * ((L.q + 3) / 4);
                for (int u = 0; u < units; u += kThreads * kApplyUnits) P.apply_tiles.push_back({pair, u});
            }
        }
        P.edge_run = P.edge_run_lds <= kEdgeLdsBytes;
        if (tune.edge <= 0) {
            P.edge_run = P.edge_run && P.edge_tiles.size() <= (size_t)kEdgeRunTiles &&
                         4 * (int64_t)n_workers * (int64_t)P.param_floats <= kEdgeRunBytes;
            for (int l = 0; l < n_layers; ++l)
                P.edge_run = P.edge_run && edge_run_cost(P.layers[l], P.edge_threads, shift[l], 2 * (int)max_deg * P.layers[l].r) <= kEdgeRunCost;
        }
        if (P.edge_run) {
            P.ws_y = P.ws_bytes;
            P.ws_ph2 = (size_t)round_up(P.ws_y + (size_t)n_workers * P.param_floats * 4, 256);
            P.ws_bytes = (size_t)round_up(P.ws_ph2 + P.pstate_floats * 4, 256);
        }
    }

    // ---- edge sweeps ----
    P.sweep = !P.edge && tune.sweep != 0 && n_edges > 0 && P.max_layer_rank <= kSweepMaxRank &&
              (tune.sweep > 0 || gains_sweeps(P, max_deg, total_bytes));
    std::vector<SweepDesc> geometry(n_layers);
    if (P.sweep) {
        // work-groups of 256, or of 512 where more than a quarter of the elements lie in rows that need those; of the rows
        // that do not fit either the finishing kernel forms the column sums
        for (int nt : {512, 256}) {
            double too_long = 0.0;
            for (int l = 0; l < n_layers; ++l) {
                if (!sweep_split(P.layers[l], nt, P.max_layer_rank, tune.sweep_units, geometry[l])) too_long += (double)P.layers[l].p * P.layers[l].q;
                P.sweep = P.sweep && (int64_t)P.layers[l].p * P.layers[l].ld < ((int64_t)1 << 30);
            }
            if (nt == 256 && (tune.sweep_threads > nt || too_long > 0.25 * P.elems_per_worker)) break;
            P.sweep_threads = nt;
        }
        for (int l = 0; l < n_layers; ++l) sweep_split(P.layers[l], P.sweep_threads, P.max_layer_rank, tune.sweep_units, geometry[l]);
    }
    if (P.sweep) {
        // Row blocks: two work-groups per CU take the whole set where it is small enough, at most 1.5 MB each.  The blocks' column sums
        // cost r / rows of the traffic and the time to add them up, so a block has 16 r rows, unless that leaves fewer
        // blocks than CUs; then 8 r, then 4 r.  (Rounds of 70 drawn sets over this: always 16 r 0.98-1.40, always 8 r 0.89-1.11, 4 r 0.86-1.16.)
        const int nt = P.sweep_threads;
        const double connected = (double)std::count_if(P.incident.begin(), P.incident.end(), [](const std::vector<int> &e) { return !e.empty(); });
        P.sweep_elems = P.elems_per_worker * connected;
        const double all = 8.0 * n_edges * P.elems_per_worker;
        const size_t room = P.ws_pd - P.ws_pw, others = P.ws_bytes - room;
        auto long_rows = [&](int l) { return P.layers[l].q >= 4 && geometry[l].units == 0; };  // leave no column sums
        P.sweep_long_elems = 0;
        for (int l = 0; l < n_layers; ++l)
            if (long_rows(l)) P.sweep_long_elems += (double)P.layers[l].p * P.layers[l].q * connected;
        std::vector<int> blk_rows(n_layers), nblk(n_layers);
        int64_t pe = 0, qe = 0, gr = 0;
        int least = 16, max_cols = 1;
        for (const LayerInfo &L : P.layers) max_cols = std::max(max_cols, L.q);
        for (; least > 4; least /= 2) {
            int64_t tiles = 0;
            for (const LayerInfo &L : P.layers) tiles += (int64_t)n_edges * ((L.p + least * L.r - 1) / (least * L.r));
            if (tiles >= 256) break;
        }
        // Most bytes of sums: what the static workspace leaves; where a set is beyond that anyway, a quarter of the parameters.
        const size_t fixed = (size_t)PG_STATIC_WORKSPACE_BYTES - 512;
        const size_t most = P.ws_bytes <= (size_t)PG_STATIC_WORKSPACE_BYTES ? (others < fixed ? fixed - others : 0)
                                                                            : std::max(room, (size_t)(P.sweep_elems));
        for (double target = std::max(16.0 * 1024, std::min((double)tune.sweep_tile_bytes, all / 512));; target *= 1.25) {
            pe = qe = gr = 0;
            for (int l = 0; l < n_layers; ++l) {
                const LayerInfo &L = P.layers[l];
                const int step = sweep_step_rows(L, nt, P.max_layer_rank, geometry[l]);
                int64_t rows_l = std::max<int64_t>((int64_t)(target / (8.0 * L.q)), least * L.r);
                rows_l = std::max(rows_l, std::min<int64_t>(16 * L.r, (L.p + 15) / 16));
                if (long_rows(l)) rows_l = std::min<int64_t>(kSweepLongRows, std::max<int64_t>(1, (int64_t)(target / (8.0 * L.q))));
                if ((L.q == 1 && L.p <= kSweepVectorRows) || geometry[l].exact) rows_l = L.p;
                rows_l = std::min<int64_t>(round_up(rows_l, step), L.p);
                nblk[l] = (int)((L.p + rows_l - 1) / rows_l);
                blk_rows[l] = nblk[l] == 1 ? L.p : (int)std::min<int64_t>(round_up((L.p + nblk[l] - 1) / nblk[l], step), L.p);
                nblk[l] = (L.p + blk_rows[l] - 1) / blk_rows[l];
                pe += (int64_t)n_edges * L.r * L.p;
                if (!long_rows(l)) qe += (int64_t)n_edges * nblk[l] * L.r * L.q;
                gr += (int64_t)n_edges * nblk[l] * kSweepGram;
            }
            const size_t need = (size_t)(pe + qe + gr) * 8;
            if (need <= most) break;
            if (target > 8.0 * P.max_rows * (double)max_cols) {  // no longer blocks to be had
                P.sweep = false;
                break;
            }
        }
        if (P.sweep) {
            if ((size_t)(pe + qe + gr) * 8 > room) sections(pwo, std::max(qwo, pe + qe + gr - pwo));
            P.ws_static_bytes = P.ws_bytes;
            P.sweep_descs.clear();
            P.sweep_tiles.clear();
            P.finish_tiles.clear();
            std::vector<std::vector<SweepTile>> die(8);
            std::vector<double> load(8, 0.0);
            int next_die = 0;
            int64_t at_p = 0, at_q = pe, at_g = pe + qe;
            auto vector = [&](int l) { return P.layers[l].q == 1 && P.layers[l].p <= kSweepVectorRows; };
            auto add = [&](int l, int e) {
                const LayerInfo &L = P.layers[l];
                const int a = P.edges[2 * e], b = P.edges[2 * e + 1];
                const size_t id = (size_t)e * n_layers + l;
                SweepDesc d = geometry[l];
                d.p = L.p;
                d.q = L.q;
                d.r = L.r;
                d.ld = L.ld;
                d.wa = a;
                d.wb = b;
                d.nblk = nblk[l];
                d.flag_off = (int32_t)P.flag_off[id];
                d.pad = 0;
                d.x_off = L.x_off;
                d.q_off = P.q_off[id];
                d.ph_off = P.ph_off[id];
                d.pe_off = at_p;
                d.qe_off = at_q;
                d.g_off = at_g;
                at_p += (int64_t)L.r * L.p;
                if (!long_rows(l)) at_q += (int64_t)nblk[l] * L.r * L.q;
                at_g += (int64_t)nblk[l] * kSweepGram;
                const int el = (int)P.sweep_descs.size();
                P.sweep_descs.push_back(d);
                const int entries = long_rows(l) ? kThreads : kFinishEntries;
                for (int f = 0; f < L.p + L.q; f += entries) P.finish_tiles.push_back({el, f, entries});
                // LDS: see sweep_body
                const int vs = 4 * d.units << d.tc_shift;
                const int sums = nt * d.units * 32;
                const int plain = L.r * vs * 4 + 2 * (nt / 64) * 4 * kSweepMaxRank * 8 + (d.exact && L.q >= 4 ? L.r * L.p * 8 : 0);
                if (!vector(l)) {
                    P.sweep_lds = std::max(P.sweep_lds, std::max(plain, sums));
                }
                return el;
            };
            for (int l = 0; l < n_layers; ++l) {
                if (vector(l)) continue;
                const int first = (int)P.sweep_descs.size();
                for (int e = 0; e < n_edges; ++e) add(l, e);
                for (int b = 0; b < nblk[l]; ++b) {
                    const int row0 = b * blk_rows[l], nrows = std::min(blk_rows[l], P.layers[l].p - row0);
                    const double bytes = 8.0 * nrows * P.layers[l].q;
                    int to = (int)(std::min_element(load.begin(), load.end()) - load.begin());
                    for (int e = 0; e < n_edges; ++e) {
                        if (!P.large && all <= kSweepSpreadBytes) to = next_die++ & 7;
                        die[to].push_back({first + e, row0, nrows, b});
                        load[to] += bytes;
                    }
                }
            }
            const int first_vector = (int)P.sweep_descs.size();
            for (int l = 0; l < n_layers; ++l)
                if (vector(l))
                    for (int e = 0; e < n_edges; ++e) add(l, e);
            const int waves = nt / 64, nvec = (int)P.sweep_descs.size() - first_vector;
            for (int v = 0; v < nvec; v += waves) {
                size_t to = 0;
                for (size_t k = 1; k < 8; ++k)
                    if (die[k].size() < die[to].size()) to = k;
                die[to].push_back({first_vector + v, 0, std::min(waves, nvec - v), -1});
            }
            size_t slots = 0;
            for (auto &v : die) slots = std::max(slots, v.size());
            for (size_t s = 0; s < slots; ++s)
                for (int k = 0; k < 8; ++k) P.sweep_tiles.push_back(s < die[k].size() ? die[k][s] : SweepTile{0, 0, 0, 0});
            P.sweep = P.sweep_lds <= kSweepLdsBytes && (tune.sweep > 0 || sweeps_are_faster(P));
        }
        if (!P.sweep) {  // as if there were none
            sections(pwo, qwo);
            P.ws_static_bytes = P.ws_bytes;
            P.sweep_descs.clear();
            P.sweep_tiles.clear();
            P.finish_tiles.clear();
        }
    }

    // ---- update of sets with several kinds of row kernels, in one launch ----
    // Row launches over time of this one, whole calls (random trees of 3 to 21 workers, a torus and a ring with several layers):
    //   rank 2 to 4, two or more kinds, up to 25 MB   1.1-2.5 (361 x 45, tree of 9: 32.8 -> 23.1 us; 50 x 5760, tree of 21, run of 5: 500 -> 251)
    //   rank 2, 64 MB 1.04;  ragged layers of 131 MB, rank 3: 322 -> 292
    //   rank 1                                        0.91-1.12: the row kernels' few columns suit them better
    //   one kind of row kernel                        0.78-0.91
    // Tiles: with 32 KB for every set 103 x 194 on a tree of 10 took 37 us against 31; about a thousand tiles mend that.  Long rows are
    // cut as well: whole rows of 70001 columns left five work-groups per worker with all the work (780 us against 324).
    P.mixed_tiles.clear();
    // Behind edge kernels: more than eight columns.  Calls with a kernel that holds all 16 columns of a unit over calls with this one, 72 sets: SGD round and
    // single iteration 1.16, up to 1.5; round 0.87-1.12.
    const bool one_update = P.edge ? P.apply_cols > kWideCols
                                   : P.sweep && P.max_groups == 1 && tune.mixed != 0 &&
                                         (tune.mixed > 0 || (rank >= 2 && P.row_classes.size() > 1 && total_bytes <= (double)kSweepMixedBytes));
    if (one_update) {
        const double bytes = std::min((double)kMixedTileBytes, total_bytes / kMixedTiles);
        for (int l = 0; l < n_layers; ++l) {
            const LayerInfo &L = P.layers[l];
            const int units = (L.q + 3) / 4, parts = (units + kThreads - 1) / kThreads, width = (units + parts - 1) / parts;
            int sh = 0;
            while ((1 << sh) < width) ++sh;
            const int step = (kThreads >> sh) * kMixedRows;
            const int steps = (int)std::max(1.0, bytes / ((double)step * width * 16));
            const int64_t rows_t = std::min<int64_t>((int64_t)step * steps, L.p);
            for (int i = 0; i < n_workers; ++i) {
                const int pair = P.pair_first[(size_t)l * n_workers + i];
                if (P.pairs[pair].R == 0) continue;
                for (int64_t r0 = 0; r0 < L.p; r0 += rows_t)
                    for (int u0 = 0; u0 < units; u0 += width)
                        P.mixed_tiles.push_back({pair, (int32_t)r0, (int32_t)std::min<int64_t>(rows_t, L.p - r0), u0, std::min(width, units - u0), sh});
            }
        }
    }
    return PG_OK;
}

}  // namespace pg
