// Host-only check of the planner (no HIP): for a list of problems, every (worker, layer) pair
// with edges is covered exactly once by its row tiles (rows x column segments) and by its
// column tiles (columns x row blocks), tiles respect what their kernel family assumes, and the
// workspace sections hold the partial sums.  Prints "ok <name>" per problem; exit status 1 on
// the first violation.  Built and run by tests/test_host_api.py.
#include <cstdio>
#include <cstdint>
#include <algorithm>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../include/powergossip.h"
#include "../paper_2008_01425_amd/csrc/pg_plan.hpp"

using namespace pg;

#define REQUIRE(cond, ...)                       \
    do {                                         \
        if (!(cond)) {                           \
            printf("FAIL %s: ", name);           \
            printf(__VA_ARGS__);                 \
            printf(" [%s]\n", #cond);            \
            return 1;                            \
        }                                        \
    } while (0)

static void ring(int n, std::vector<int32_t> &e) {
    for (int i = 0; i < n; ++i) {
        e.push_back(i);
        e.push_back((i + 1) % n);
    }
}
static void torus(int R, int C, std::vector<int32_t> &e) {
    for (int r = 0; r < R; ++r)
        for (int c = 0; c < C; ++c) {
            int v = r * C + c;
            e.push_back(v);
            e.push_back(r * C + (c + 1) % C);
            e.push_back(v);
            e.push_back(((r + 1) % R) * C + c);
        }
}

static int check(const char *name, int n, const std::vector<int32_t> &e, const std::vector<float> &ew,
                 const std::vector<int32_t> &rows, const std::vector<int32_t> &cols, int rank, int steps,
                 const Tuning &tune) {
    Plan P;
    int rc = build_plan(P, n, (int)ew.size(), e.data(), ew.data(), (int)rows.size(), rows.data(), cols.data(),
                        rank, steps, tune);
    REQUIRE(rc == PG_OK, "build_plan returned %d", rc);
    const int L = (int)rows.size();

    // ---- row tiles: per (pair, segment) the row intervals tile [0, p) ----
    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> rcover;
    for (const RowClass &c : P.row_classes)
        for (const RowTile &t : c.tiles) {
            REQUIRE(t.pair >= 0 && t.pair < (int)P.pairs.size(), "row tile pair %d", t.pair);
            const PairDesc &pd = P.pairs[t.pair];
            REQUIRE(compiled_cols(pd.R) == c.RC, "pair %d with R=%d in class RC=%d", t.pair, pd.R, c.RC);
            // accesses as wide as the row length allows, or four floats wide
            REQUIRE(pd.V == 4 || pd.q % 4 != 0, "rows of %d floats in units of %d", pd.q, pd.V);
            REQUIRE(pd.V >= 2 || pd.q % 2 != 0, "rows of %d floats in units of %d", pd.q, pd.V);
            // wider ones: in narrow kernels where the set is planned for it, from 16 columns on (the last unit is
            // moved back to the row's end); in wide kernels on rows padded to whole units
            if (pd.q % pd.V != 0 && c.RC < kWideCols) REQUIRE(P.odd_rows && pd.V == 4 && pd.q >= 16 && pd.seg_len % 4 == 0, "narrow rows of %d floats in units of %d", pd.q, pd.V);
            if (pd.q % pd.V != 0 && c.RC >= kWideCols) REQUIRE(c.pad && pd.V == 4 && pd.ld % 4 == 0, "wide rows of %d floats (stride %d) in units of %d", pd.q, pd.ld, pd.V);
            REQUIRE(t.nrows >= 1 && t.row0 >= 0 && t.row0 + t.nrows <= pd.p, "row tile rows %d+%d of %d", t.row0, t.nrows, pd.p);
            REQUIRE(t.seg >= 0 && t.seg < pd.nseg && (int64_t)t.seg * pd.seg_len < pd.q, "segment %d", t.seg);
            if (c.RC >= kWideCols) REQUIRE(c.V == pd.V, "class V=%d, layer V=%d", c.V, pd.V);
            if (c.vec) REQUIRE(pd.q == 1 && c.RC < kWideCols && t.nrows <= 256, "vector tile: q=%d, RC=%d, %d rows", pd.q, c.RC, t.nrows);
            if (tune.vec_kernels == 2 && c.RC < kWideCols) REQUIRE(c.vec == (pd.q == 1), "vector layer outside the vector classes (q=%d)", pd.q);
            if (tune.vec_kernels == 0) REQUIRE(!c.vec, "vector class although switched off");
            if (c.mfma) {
                REQUIRE(pd.wc == 1 || pd.wc == 2 || pd.wc == 4, "wc=%d", pd.wc);
                REQUIRE(pd.seg_len % 64 == 0, "seg_len=%d", pd.seg_len);
                REQUIRE(t.nrows <= 16 * kMfmaRowBlocks * (4 / pd.wc), "matrix-core tile of %d rows, wc=%d", t.nrows, pd.wc);
                REQUIRE((int64_t)pd.p * pd.q < ((int64_t)1 << 30), "layer too large for 32-bit offsets");
            } else if (c.RC >= kWideCols) {
                REQUIRE((int64_t)c.RC * pd.seg_len * 4 <= kWideLdsBytes, "Q slice of %d x %d floats", c.RC, pd.seg_len);
                REQUIRE(c.max_seg >= pd.seg_len, "max_seg");
                REQUIRE(pd.seg_len % (pd.lpr * pd.V) == 0, "seg_len %d, lpr %d, V %d", pd.seg_len, pd.lpr, pd.V);
            } else {
                REQUIRE(pd.lpr >= 1 && pd.lpr <= 64 && (pd.lpr & (pd.lpr - 1)) == 0, "lpr=%d", pd.lpr);
                REQUIRE(pd.seg_len % pd.V == 0, "seg_len %d V %d", pd.seg_len, pd.V);
            }
            rcover[{t.pair, t.seg}].push_back({t.row0, t.row0 + t.nrows});
        }
    // ---- column tiles: per (pair, row block) the column intervals tile [0, q) ----
    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> ccover;
    for (const ColClass &c : P.col_classes)
        for (const ColTile &t : c.tiles) {
            REQUIRE(t.pair >= 0 && t.pair < (int)P.pairs.size(), "col tile pair %d", t.pair);
            const PairDesc &pd = P.pairs[t.pair];
            REQUIRE(compiled_cols(pd.R) == c.RC, "pair %d with R=%d in column class RC=%d", t.pair, pd.R, c.RC);
            REQUIRE(t.blk >= 0 && t.blk < pd.nblk && (int64_t)t.blk * pd.blk_rows < pd.p, "row block %d", t.blk);
            if (c.vec) REQUIRE(pd.q == 1 && c.RC < kWideCols, "vector column tile: q=%d, RC=%d", pd.q, c.RC);
            if (tune.vec_kernels == 2 && c.RC < kWideCols) REQUIRE(c.vec == (pd.q == 1), "vector layer outside the vector column classes (q=%d)", pd.q);
            const int cw = (c.RC >= kWideCols && P.mfma_cols) ? kMfmaTileCols : pd.lg * pd.V;
            REQUIRE(t.c0 >= 0 && t.c0 < pd.q && t.c0 % cw == 0, "column tile at %d, width %d", t.c0, cw);
            if (!(c.RC >= kWideCols && P.mfma_cols)) {
                REQUIRE(c.max_rows >= pd.blk_rows, "max_rows");
                REQUIRE((int64_t)(pd.blk_rows + 1) * c.RC * 4 <= kColLdsBytes, "Phat slice of %d rows x %d columns", pd.blk_rows, c.RC);
            }
            ccover[{t.pair, t.blk}].push_back({t.c0, std::min(pd.q, t.c0 + cw)});
        }
    auto tiles_exactly = [](std::vector<std::pair<int, int>> v, int end) {
        std::sort(v.begin(), v.end());
        int at = 0;
        for (auto &iv : v) {
            if (iv.first != at) return false;
            at = iv.second;
        }
        return at == end;
    };
    int64_t pw_need = 0, qw_need = 0;
    REQUIRE((int)P.pair_first.size() == L * n && (int)P.pair_count.size() == L * n, "pair index tables");
    int next_pair = 0;
    for (int l = 0; l < L; ++l)
        for (int i = 0; i < n; ++i) {
            const int first = P.pair_first[l * n + i], count = P.pair_count[l * n + i];
            REQUIRE(first == next_pair && count >= 1 && count <= P.max_groups, "groups of layer %d worker %d", l, i);
            next_pair += count;
            int Rsum = 0;
            for (int gi = 0; gi < count; ++gi) {
                const int pair = first + gi;
                const PairDesc &pd = P.pairs[pair];
                REQUIRE(pd.p == rows[l] && pd.q == cols[l] && pd.worker == i, "pair %d fields", pair);
                REQUIRE(P.pair_group[pair] == gi && P.pair_layer[pair] == l, "pair %d group/layer", pair);
                REQUIRE(pd.R <= kMaxCols && pd.R % P.layers[l].r == 0, "R=%d of pair %d", pd.R, pair);
                REQUIRE(pd.ld >= pd.q && (pd.ld == pd.q || pd.ld % 32 == 0), "row stride %d of pair %d", pd.ld, pair);
                Rsum += pd.R;
                if (pd.R == 0) {
                    REQUIRE(count == 1, "empty group beside others");
                    REQUIRE(!rcover.count({pair, 0}) && !ccover.count({pair, 0}), "tiles for a worker without edges");
                    continue;
                }
                REQUIRE((int64_t)pd.nseg * pd.seg_len >= pd.q && (int64_t)(pd.nseg - 1) * pd.seg_len < pd.q, "segments of pair %d", pair);
                REQUIRE((int64_t)pd.nblk * pd.blk_rows >= pd.p && (int64_t)(pd.nblk - 1) * pd.blk_rows < pd.p, "blocks of pair %d", pair);
                for (int sg = 0; sg < pd.nseg; ++sg)
                    REQUIRE(tiles_exactly(rcover[{pair, sg}], pd.p), "rows of pair %d (layer %d, worker %d), segment %d", pair, l, i, sg);
                for (int b = 0; b < pd.nblk; ++b)
                    REQUIRE(tiles_exactly(ccover[{pair, b}], pd.q), "columns of pair %d, block %d", pair, b);
                REQUIRE(pd.pw_off == pw_need && pd.qw_off == qw_need, "partial-sum offsets of pair %d", pair);
                pw_need += (int64_t)pd.nseg * pd.R * pd.p;
                qw_need += (int64_t)pd.nblk * pd.R * pd.q;
            }
            REQUIRE(Rsum == (int)P.incident[i].size() * P.layers[l].r, "stacked columns of layer %d worker %d", l, i);
        }
    REQUIRE(next_pair == (int)P.pairs.size(), "pair count");
    // a row class holds tiles of one column group only (groups of one matrix never share a launch)
    for (const RowClass &c : P.row_classes)
        for (const RowTile &t : c.tiles) REQUIRE(P.pair_group[t.pair] == c.group, "tile of group %d in class of group %d", P.pair_group[t.pair], c.group);
    REQUIRE(P.orth_tiles.empty() || P.ws_uq >= P.ws_gpart + P.orth_tiles.size() * 36 * 8, "Gram sums do not fit their section");
    REQUIRE(P.ws_qw >= P.ws_pw + (size_t)pw_need * 8, "P partial sums do not fit their section");
    REQUIRE(P.ws_pd >= P.ws_qw + (size_t)qw_need * 8, "Q partial sums do not fit their section");
    REQUIRE(P.ws_bytes >= P.ws_uq, "workspace size");
    // ---- sweeps do not take a problem beyond the static workspace, and beyond that add at most a quarter of the parameters ----
    {
        Plan S;
        Tuning plain = tune;
        plain.edge = plain.sweep = 0;
        build_plan(S, n, (int)ew.size(), e.data(), ew.data(), L, rows.data(), cols.data(), rank, steps, plain);
        const size_t limit = S.ws_bytes <= (size_t)PG_STATIC_WORKSPACE_BYTES ? (size_t)PG_STATIC_WORKSPACE_BYTES : S.ws_bytes + (size_t)(n * S.elems_per_worker);
        REQUIRE(P.ws_static_bytes <= limit, "workspace %zu, %zu without sweeps, parameters %.0f", P.ws_static_bytes, S.ws_bytes, 4.0 * n * S.elems_per_worker);
        // the second buffer of runs on edge kernels, with one of the unit vectors
        if (tune.edge <= 0) REQUIRE(P.ws_bytes - P.ws_static_bytes <= (size_t)kEdgeRunBytes + 512 + 4 * P.pstate_floats, "workspace %zu, single rounds %zu", P.ws_bytes, P.ws_static_bytes);
        if (!P.sweep && !P.edge) REQUIRE(P.ws_bytes == S.ws_bytes && P.sweep_tiles.empty() && P.finish_tiles.empty(), "workspace %zu, %zu without sweeps", P.ws_bytes, S.ws_bytes);
    }
    // ---- one-launch update: every element of every pair with columns once ----
    if (!P.mixed_tiles.empty()) {
        std::vector<int64_t> covered(P.pairs.size(), 0);
        std::vector<std::set<std::pair<int, int>>> corners(P.pairs.size());
        for (const MixedTile &t : P.mixed_tiles) {
            const PairDesc &pd = P.pairs[t.pair];
            REQUIRE(t.nrows > 0 && t.nunits > 0 && t.row0 >= 0 && t.unit0 >= 0 && t.row0 + t.nrows <= pd.p && t.unit0 + t.nunits <= (pd.q + 3) / 4, "update tile of pair %d", t.pair);
            REQUIRE(t.tc_shift >= 0 && (1 << t.tc_shift) <= kThreads, "%d threads on a row", 1 << t.tc_shift);
            REQUIRE(corners[t.pair].insert({t.row0, t.unit0}).second, "update tile of pair %d twice", t.pair);
            covered[t.pair] += (int64_t)t.nrows * t.nunits;
        }
        for (size_t i = 0; i < P.pairs.size(); ++i)
            REQUIRE(covered[i] == (P.pairs[i].R ? (int64_t)P.pairs[i].p * ((P.pairs[i].q + 3) / 4) : 0), "update of pair %zu", i);
    }
    // ---- edge sweeps: the blocks of every (edge, layer) tile [0, p), each once; vectors once; entries of the results once; sums fit ----
    if (P.sweep) {
        std::map<int, std::vector<std::pair<int, int>>> scover, fcover;
        REQUIRE(P.sweep_tiles.size() % 8 == 0, "slots of eight");
        for (const SweepTile &t : P.sweep_tiles) {
            if (t.nrows == 0) continue;
            if (t.blk < 0) {
                REQUIRE(t.nrows <= P.sweep_threads / 64, "%d vectors in a tile", t.nrows);
                for (int k = 0; k < t.nrows; ++k) {
                    REQUIRE(t.el + k < (int)P.sweep_descs.size() && P.sweep_descs[t.el + k].q == 1 && P.sweep_descs[t.el + k].nblk == 1, "vector %d", t.el + k);
                    scover[t.el + k].push_back({0, P.sweep_descs[t.el + k].p});
                }
                continue;
            }
            const SweepDesc &d = P.sweep_descs[t.el];
            REQUIRE(t.blk < d.nblk && t.nrows > 0, "block %d of %d", t.blk, d.nblk);
            if (d.exact) REQUIRE(d.nblk == 1 && (d.q < 4 || d.units == 1 || d.units == 3), "exact layer: %d blocks, %d units", d.nblk, d.units);
            if (d.q >= 4 && d.units == 0) REQUIRE(t.nrows <= kSweepLongRows, "%d long rows", t.nrows);
            if (d.q >= 4 && d.units > 0) REQUIRE((4 * d.units << d.tc_shift) >= d.q && (1 << d.tc_shift) <= P.sweep_threads, "%d floats over %d x %d units", d.q, d.units, 1 << d.tc_shift);
            scover[t.el].push_back({t.row0, t.row0 + t.nrows});
        }
        for (const FinishTile &t : P.finish_tiles) fcover[t.el].push_back({t.first, std::min(t.first + t.count, P.sweep_descs[t.el].p + P.sweep_descs[t.el].q)});
        REQUIRE(P.sweep_descs.size() == (size_t)L * P.n_edges, "%zu (edge, layer)s", P.sweep_descs.size());
        const int64_t room = (int64_t)(P.ws_pd - P.ws_pw) / 8;
        for (int el = 0; el < (int)P.sweep_descs.size(); ++el) {
            const SweepDesc &d = P.sweep_descs[el];
            REQUIRE(tiles_exactly(scover[el], d.p), "rows of (edge, layer) %d", el);
            REQUIRE(tiles_exactly(fcover[el], d.p + d.q), "entries of (edge, layer) %d", el);
            const int64_t left = d.q >= 4 && d.units == 0 ? 0 : (int64_t)d.nblk * d.r * d.q;  // long rows leave no column sums
            REQUIRE(d.pe_off + (int64_t)d.r * d.p <= room && d.qe_off + left <= room &&
                    d.g_off + (int64_t)d.nblk * kSweepGram <= room, "sums of (edge, layer) %d", el);
        }
        REQUIRE(P.sweep_lds <= kSweepLdsBytes, "%d bytes of LDS", P.sweep_lds);
    }
    if (P.edge) {
        REQUIRE(P.edge_tiles.size() == (size_t)L * P.n_edges && P.edge_lds <= kEdgeLdsBytes, "edge tiles");
        for (const EdgeTile &t : P.edge_tiles)
            REQUIRE(((int64_t)t.p << t.tc_shift) <= P.edge_threads && (4 * kEdgeUnits << t.tc_shift) >= t.q, "%d x %d over %d threads", t.p, t.q, P.edge_threads);
        std::map<int, std::vector<std::pair<int, int>>> acover;
        for (const ApplyTile &t : P.apply_tiles) {
            const int units = P.pairs[t.pair].p * ((P.pairs[t.pair].q + 3) / 4);
            acover[t.pair].push_back({t.first, std::min(units, t.first + kThreads * kApplyUnits)});
        }
        for (auto &a : acover) REQUIRE(tiles_exactly(a.second, P.pairs[a.first].p * ((P.pairs[a.first].q + 3) / 4)), "units of pair %d", a.first);
    }
    if (name[0] != 'r' || name[1] != 'a') printf("ok %s\n", name);  // the random problems stay quiet
    return 0;
}

// Which sets have their passes streamed, and which runs write every second round (`one` layer shape besides
// an optional second).
static int check_paths(const char *name, int n, const std::vector<int32_t> &e, const std::vector<int32_t> &rows,
                       const std::vector<int32_t> &cols, int rank, int steps, bool stream, bool lazy) {
    Plan P;
    std::vector<float> w(e.size() / 2, 0.2f);
    int rc = build_plan(P, n, (int)w.size(), e.data(), w.data(), (int)rows.size(), rows.data(), cols.data(), rank, steps, Tuning());
    REQUIRE(rc == PG_OK, "build_plan returned %d", rc);
    REQUIRE(P.stream == stream, "streamed: %d", P.stream);
    REQUIRE(P.lazy == lazy, "writes every second round: %d", P.lazy);
    for (const ColClass &c : P.col_classes)
        if (P.lazy) REQUIRE(lazy_col_lds(c.max_rows, c.RC) <= 64 * 1024 && c.RC <= 4 && !c.vec, "peeking column kernel of %d rows", c.max_rows);
    printf("as expected: %s\n", name);
    return 0;
}

int main() {
    int bad = 0;
    std::vector<Tuning> tunings(4);
    tunings[0].sweep = 1;
    tunings[0].mixed = 1;
    tunings[1].edge = 1;
    tunings[3].edge = 0;
    tunings[3].sweep = 1;
    tunings[1].mfma_rows = false;
    tunings[1].vec_kernels = 0;
    tunings[2].mfma_rows = false;
    tunings[2].mfma_cols = false;
    tunings[3].vec_kernels = 2;
    for (const Tuning &tn : tunings) {
        std::vector<int32_t> e;
        ring(4, e);
        bad |= check("tiny", 4, e, std::vector<float>(4, 1 / 3.f), {64, 32, 16}, {32, 16, 1}, 1, 1, tn);
        e.clear();
        ring(16, e);
        bad |= check("vgg16 r=2", 16, e, std::vector<float>(16, 1 / 3.f),
                     {64, 64, 128, 128, 256, 256, 256, 512, 512, 512, 512, 512, 512, 10},
                     {27, 576, 576, 1152, 1152, 2304, 2304, 2304, 4608, 4608, 4608, 4608, 4608, 512}, 2, 1, tn);
        e.clear();
        torus(4, 4, e);
        bad |= check("lstm", 16, e, std::vector<float>(32, 0.2f), {33278, 2600, 2600, 2600, 2600},
                     {650, 650, 650, 650, 650}, 4, 2, tn);
        e.clear();
        torus(8, 8, e);
        {
            std::vector<int32_t> r, c;
            for (int i = 0; i < 161; ++i) {
                r.push_back(64 + i * 13 % 2000);
                c.push_back(i % 3 == 0 ? 1 : (i % 5 == 0 ? 147 : 64 * (1 + i % 70)));
            }
            bad |= check("resnet50-like", 64, e, std::vector<float>(128, 0.2f), r, c, 2, 2, tn);
        }
        e.clear();
        ring(3, e);
        bad |= check("odd shapes", 3, e, std::vector<float>(3, 1 / 3.f), {1, 7, 33278, 5, 4099}, {1, 3, 650, 100003, 68}, 3, 1, tn);
        // star with a chord, rank 4: 16, 8, 8, 4 and 4 stacked columns in every layer; one worker without edges
        e = {0, 1, 0, 2, 3, 0, 0, 4, 2, 1};
        bad |= check("mixed degrees", 6, e, {0.2f, 0.2f, 0.2f, 0.2f, 0.15f},
                     {50, 17, 100, 9, 33, 16, 1, 300, 2}, {131, 70, 64, 3, 200, 65, 40, 5000, 9}, 4, 2, tn);
        e.clear();
        torus(3, 3, e);
        bad |= check("torus 3x3 rank 2", 9, e, std::vector<float>(18, 0.2f), {120, 33, 40, 2600}, {260, 12, 1, 63}, 2, 1, tn);
        bad |= check("extreme aspect ratios", 9, e, std::vector<float>(18, 0.2f), {5, 300001, 1, 2, 70001, 33278},
                     {100003, 3, 1, 65537, 1, 1}, 4, 1, tn);
        // more than 16 stacked columns: rank 8 (two groups of two edges), rank 6 (two of two), rank 16 (four of one)
        bad |= check("torus 3x3 rank 8", 9, e, std::vector<float>(18, 0.2f), {120, 33, 40, 8, 700}, {260, 12, 1, 100, 650}, 8, 2, tn);
        bad |= check("torus 3x3 rank 6", 9, e, std::vector<float>(18, 0.2f), {120, 33, 5}, {260, 12, 64}, 6, 1, tn);
        bad |= check("torus 3x3 rank 16", 9, e, std::vector<float>(18, 0.2f), {120, 16, 40}, {260, 300, 1}, 16, 1, tn);
    }
    // seeded random problems: graphs with isolated and high-degree workers, layer shapes from 1 x 1 to
    // very tall and very wide, ranks 1..16, every kernel-family setting
    uint64_t state = 0x9E3779B97F4A7C15ull;
    auto rnd = [&](int lo, int hi) {  // uniform in [lo, hi]
        state ^= state << 13;
        state ^= state >> 7;
        state ^= state << 17;
        return lo + (int)(state % (uint64_t)(hi - lo + 1));
    };
    int nrandom = 0;
    for (int trial = 0; trial < 240 && !bad; ++trial) {
        const int n = rnd(1, 12);
        std::vector<int32_t> e;
        std::vector<int> deg(n, 0);
        for (int a = 0; a < n; ++a)
            for (int b = a + 1; b < n; ++b)
                if (rnd(0, 99) < (trial % 3 == 0 ? 70 : 25)) {
                    if (rnd(0, 1)) { e.push_back(a); e.push_back(b); } else { e.push_back(b); e.push_back(a); }
                    ++deg[a]; ++deg[b];
                }
        const int ne = (int)e.size() / 2;
        const int dmax = std::max(1, *std::max_element(deg.begin(), deg.end()));
        std::vector<float> w(ne, 1.0f / dmax);
        std::vector<int32_t> r, c;
        const int nl = rnd(1, 6);
        for (int l = 0; l < nl; ++l) {
            switch (rnd(0, 5)) {
                case 0: r.push_back(rnd(1, 40)); c.push_back(rnd(1, 40)); break;
                case 1: r.push_back(rnd(1, 90000)); c.push_back(1); break;
                case 2: r.push_back(rnd(1, 8)); c.push_back(rnd(1, 120000)); break;
                case 3: r.push_back(rnd(1, 40000)); c.push_back(rnd(1, 12)); break;
                default: r.push_back(rnd(16, 3000)); c.push_back(rnd(16, 5000)); break;
            }
        }
        char label[64];
        snprintf(label, sizeof(label), "random %d", trial);
        bad |= check(label, n, e, w, r, c, rnd(1, 16), rnd(1, 3), tunings[trial % tunings.size()]);
        ++nrandom;
    }
    // the same on graphs up to complete ones of 24 workers, with long rows among the layers
    for (int trial = 0; trial < 60 && !bad; ++trial) {
        const int n = rnd(2, 24), kind = trial % 3;
        std::vector<int32_t> e;
        if (kind == 0)
            for (int a = 0; a < n; ++a)
                for (int b = a + 1; b < n; ++b) { e.push_back(a); e.push_back(b); }
        else if (kind == 1 && n > 2)
            ring(n, e);
        else
            for (int a = 1; a < n; ++a) { e.push_back((a - 1) / 3); e.push_back(a); }
        std::vector<float> w(e.size() / 2, 1.0f / n);
        std::vector<int32_t> r, c;
        const int nl = rnd(1, 3);
        for (int l = 0; l < nl; ++l) {
            r.push_back(rnd(0, 2) ? rnd(1, 400) : rnd(1, 4096));
            c.push_back(rnd(0, 2) ? rnd(4000, 80000) : rnd(1, 8000));
        }
        char label[64];
        snprintf(label, sizeof(label), "random long rows %d", trial);
        Tuning forced;
        forced.edge = 0;
        forced.sweep = 1;
        const int rank = rnd(1, 4), steps = rnd(1, 2);
        bad |= check(label, n, e, w, r, c, rank, steps, Tuning());
        bad |= check(label, n, e, w, r, c, rank, steps, forced);
        ++nrandom;
    }
    std::vector<int32_t> r16, t4, t3;
    ring(16, r16);
    torus(4, 4, t4);
    torus(3, 3, t3);
    const std::vector<int32_t> vr = {64, 64, 128, 128, 256, 256, 256, 512, 512, 512, 512, 512, 512, 10, 512},
                               vc = {27, 576, 576, 1152, 1152, 2304, 2304, 2304, 4608, 4608, 4608, 4608, 4608, 512, 1};
    bad |= check_paths("vgg16 rank 1", 16, r16, vr, vc, 1, 1, true, true);
    bad |= check_paths("vgg16 rank 2", 16, r16, vr, vc, 2, 1, true, true);
    bad |= check_paths("vgg16, two power steps", 16, r16, vr, vc, 1, 2, true, false);
    bad |= check_paths("lstm torus rank 4", 16, t4, {33278, 2600, 2600, 2600, 2600}, {650, 650, 650, 650, 650}, 4, 1, true, false);
    bad |= check_paths("small", 16, r16, {512}, {4608}, 1, 1, false, false);
    // rows that are not whole cache lines are not streamed, however large the set
    bad |= check_paths("table of 12 columns", 16, r16, {600000}, {12}, 1, 1, false, false);
    bad |= check_paths("577 columns", 16, r16, {13000}, {577}, 1, 1, false, true);
    bad |= check_paths("577 columns rank 2", 16, r16, {13000}, {577}, 2, 1, false, true);
    bad |= check_paths("100 columns rank 2", 16, r16, {80000}, {100}, 2, 1, false, false);
    bad |= check_paths("63 columns, 8 stacked", 9, t3, {400000}, {63}, 2, 1, false, false);
    bad |= check_paths("100 columns, 8 stacked", 9, t3, {300000}, {100}, 2, 1, false, false);
    bad |= check_paths("100 columns, 16 stacked", 9, t3, {300000}, {100}, 4, 1, true, false);
    bad |= check_paths("50 columns, 16 stacked", 9, t3, {600000}, {50}, 4, 1, false, false);
    // three quarters of the elements decide
    bad |= check_paths("lines beside few odd rows", 16, r16, {4096, 1000}, {4608, 577}, 1, 1, true, true);
    bad |= check_paths("lines beside many odd rows", 16, r16, {2048, 13000}, {4608, 577}, 1, 1, false, true);
    // one long vector or tall narrow layer keeps the whole run writing every round (its row block of the
    // column kernel does not fit beside the pending coefficients)
    bad |= check_paths("a bias of 2800", 16, r16, {4096, 2800}, {4608, 1}, 1, 1, true, false);
    // kernels with the body for rows of odd length: from one element in a hundred on
    auto odd = [&](const char *name, const std::vector<int32_t> &rows, const std::vector<int32_t> &cols, bool want) {
        Plan P;
        std::vector<float> w(16, 0.2f);
        int rc = build_plan(P, 16, 16, r16.data(), w.data(), (int)rows.size(), rows.data(), cols.data(), 1, 1, Tuning());
        REQUIRE(rc == PG_OK, "build_plan returned %d", rc);
        REQUIRE(P.odd_rows == want, "planned for rows of odd length: %d", P.odd_rows);
        printf("as expected: %s\n", name);
        return 0;
    };
    bad |= odd("vgg16 layers", vr, vc, false);
    bad |= odd("whole units only", {100, 40, 3000, 64}, {100, 16, 4, 576}, false);
    bad |= odd("short odd rows", {100, 4000, 900}, {100, 3, 14}, false);
    bad |= odd("one layer of 27 columns", {100, 64}, {100, 27}, true);
    bad |= odd("577 columns, 15 MB", {400}, {577}, false);
    bad |= odd("577 columns, 59 MB", {1600}, {577}, true);
    bad |= odd("109 columns, 1 MB", {160}, {109}, true);
    bad |= odd("1150 columns, 150 MB", {2000}, {1150}, false);
    bad |= odd("1150 columns, 500 MB", {7000}, {1150}, true);
    bad |= odd("130 columns, 500 MB", {60000}, {130}, false);
    bad |= odd("a sliver of 27 columns", {1000, 16}, {1000, 27}, false);
    // a set that units of four floats take beyond the static workspace keeps them where longer row blocks bring it back
    {
        const char *name = "longer blocks before narrower accesses";
        std::vector<int32_t> t54;
        torus(5, 4, t54);
        const std::vector<int32_t> r = {106, 265, 1234, 755, 34, 70, 2198, 4076, 365, 999, 105, 446, 60, 3563, 3749, 2415, 75, 42, 198, 151},
                                   c = {115, 63, 1, 3, 1, 45, 148, 1211, 883, 47, 1197, 3, 1701, 7, 7, 1, 108, 2628, 1, 1};
        Plan P, Q;
        std::vector<float> w(t54.size() / 2, 0.2f);
        Tuning narrow;
        narrow.odd_rows = 1;
        build_plan(Q, 20, (int)w.size(), t54.data(), w.data(), (int)r.size(), r.data(), c.data(), 1, 1, narrow);
        REQUIRE(Q.ws_bytes > (size_t)PG_STATIC_WORKSPACE_BYTES, "%zu bytes", Q.ws_bytes);
        build_plan(P, 20, (int)w.size(), t54.data(), w.data(), (int)r.size(), r.data(), c.data(), 1, 1, Tuning());
        REQUIRE(P.ws_bytes <= (size_t)PG_STATIC_WORKSPACE_BYTES && P.odd_rows, "%zu bytes, units of four %d", P.ws_bytes, P.odd_rows);
        printf("as expected: %s\n", name);
    }
    // which kernels a round takes
    auto path = [&](const char *name, const std::vector<int32_t> &edges, int n, const std::vector<int32_t> &rows, const std::vector<int32_t> &cols,
                    int rank, int steps, const char *want) {
        Plan P;
        std::vector<float> w(edges.size() / 2, 1.0f / n);
        int rc = build_plan(P, n, (int)w.size(), edges.data(), w.data(), (int)rows.size(), rows.data(), cols.data(), rank, steps, Tuning());
        REQUIRE(rc == PG_OK, "build_plan returned %d", rc);
        const std::string got = P.edge ? (P.edge_run ? "edge, runs too" : P.mixed_tiles.empty() ? "edge" : "edge, one update") : P.sweep ? (P.mixed_tiles.empty() ? "sweep" : "sweep, one update") : "stream";
        REQUIRE(got == want, "%s", got.c_str());
        printf("as expected: %s\n", name);
        return 0;
    };
    std::vector<int32_t> r8, r3, t11, c16, c24;
    ring(8, r8);
    ring(3, r3);
    for (int v = 1; v < 11; ++v) { t11.push_back((v - 1) / 3); t11.push_back(v); }
    for (int a = 0; a < 24; ++a)
        for (int b = a + 1; b < 24; ++b) {
            c24.push_back(a); c24.push_back(b);
            if (b < 16) { c16.push_back(a); c16.push_back(b); }
        }
    std::vector<int32_t> nr, nc;  // three convolutions of a small image model's three widths, with their biases
    for (int k = 0; k < 19; ++k) {
        const int ch = k < 7 ? 16 : k < 13 ? 32 : 64;
        nr.insert(nr.end(), {ch, ch, ch});
        nc.insert(nc.end(), {k == 0 ? 27 : 9 * ch, 1, 1});
    }
    bad |= path("vgg16 layers, rank 1", r16, 16, vr, vc, 1, 1, "sweep");
    bad |= path("vgg16 layers, rank 2", r16, 16, vr, vc, 2, 1, "stream");
    bad |= path("100 x 100, ring of 8", r8, 8, {100}, {100}, 1, 1, "edge, runs too");
    bad |= path("small layers, ring of 8, rank 4", r8, 8, {40, 64, 64}, {60, 32, 1}, 4, 1, "edge, runs too");
    // a pending update costs more than a launch: long rows, many columns, more work-groups than CUs
    bad |= path("1 x 5936", r8, 8, {1}, {5936}, 1, 1, "edge");
    bad |= path("122 x 56, 16 columns", t4, 16, {122}, {56}, 4, 1, "edge, one update");
    bad |= path("forty layers of 60 x 64", r8, 8, std::vector<int32_t>(40, 60), std::vector<int32_t>(40, 64), 1, 1, "edge");
    bad |= path("a thousand layers of 8 x 64", r8, 8, std::vector<int32_t>(1000, 8), std::vector<int32_t>(1000, 64), 1, 1, "stream");
    bad |= path("small convolutions, ring of 8", r8, 8, nr, nc, 1, 1, "sweep");
    bad |= path("ragged layers, tree of 11", t11, 11, {510, 77, 1301, 2047, 33, 129, 5, 40001}, {1023, 4099, 333, 255, 1, 2, 70001, 7}, 3, 1, "sweep, one update");
    // rows beyond the registers; a dense graph with much to read per edge, and with little; three workers
    bad |= path("4096 x 70001", r8, 8, {4096}, {70001}, 1, 1, "stream");
    bad |= path("8192 x 20000", r8, 8, {8192}, {20000}, 1, 1, "stream");
    bad |= path("a head of 25088 columns", r16, 16, {4096, 4096, 1000}, {25088, 4096, 4096}, 1, 1, "stream");
    bad |= path("complete graph of 16, 512 x 4608", c16, 16, {512, 512, 512}, {4608, 4608, 4608}, 1, 1, "stream");
    bad |= path("complete graph of 16, 768 x 50257", c16, 16, {768}, {50257}, 1, 1, "stream");
    bad |= path("complete graph of 24, 136 x 23931", c24, 24, {136}, {23931}, 1, 2, "stream");
    bad |= path("complete graph of 24, 55 x 2532", c24, 24, {55}, {2532}, 1, 1, "stream");
    bad |= path("three workers, 100 MB", r3, 3, {3208}, {2644}, 1, 2, "stream");
    bad |= path("three workers, two layers", r3, 3, {2210, 40}, {950, 700}, 1, 2, "stream");
    // wide kernels: which floats per access the padded layers get
    auto widths = [&](const char *name, const std::vector<int32_t> &edges, int n, const std::vector<int32_t> &rows,
                      const std::vector<int32_t> &cols, int rank, int want) {
        Plan P;
        std::vector<float> w(edges.size() / 2, 0.2f);
        int rc = build_plan(P, n, (int)w.size(), edges.data(), w.data(), (int)rows.size(), rows.data(), cols.data(), rank, 1, Tuning());
        REQUIRE(rc == PG_OK, "build_plan returned %d", rc);
        for (const RowClass &c : P.row_classes)
            if (c.RC >= kWideCols) REQUIRE(c.V == want, "%d floats per access", c.V);
        printf("as expected: %s\n", name);
        return 0;
    };
    bad |= widths("odd rows, 16 columns", t3, 9, {126}, {927}, 4, 4);
    bad |= widths("even rows, 16 columns, small", t3, 9, {241}, {1642}, 4, 2);
    bad |= widths("even rows, 16 columns, 130 MB", t3, 9, {2400}, {1506}, 4, 4);
    bad |= widths("short even rows, 8 columns", t3, 9, {260}, {70}, 2, 2);
    bad |= widths("long even rows, 8 columns", t3, 9, {57}, {5222}, 2, 4);
    bad |= widths("even rows beside whole units", t3, 9, {143, 378, 72, 83}, {32, 182, 345, 36}, 3, 4);
    if (!bad) printf("ok %d random problems\n", nrandom);
    return bad;
}
