// plan_wide_check.cpp -- host-side check of the tables the library plans with:
// ragged tiles (4-wide accesses at element alignment) and split row items.
//
// Replays, on the CPU, the index arithmetic of the kernels over those tables:
// every access inside its buffer, every element stored once, every partial
// sum written once and read only where it was written.  Tiles and items of
// the plain kinds go through plan_check.cpp's own replay.  Built with
// -fsanitize=address,undefined by the test that runs it.
#define main plan_check_main
#include "plan_check.cpp"
#undef main

static void check_ragged_tile(const Plan &pl, const Tile &tl, std::vector<Marks> &elems,
                              std::vector<Marks> &rowp, std::vector<Marks> &colp)
{
    const TensorDesc &td = pl.tensors[static_cast<size_t>(tl.tensor)];
    const int64_t m = td.m, n = td.n, mn = m * n;
    const int V = tl.vec, llog = tl.lanes_log2, L = 1 << llog, G = kWave >> llog;
    const size_t ti = static_cast<size_t>(tl.tensor);
    CHECK(V == kRaggedVec && n >= V && td.vec == 1, "ragged tile of %lld columns, vec %d",
          (long long)n, td.vec);
    CHECK(tl.rpw >= 1 && tl.rpw <= kMaxRowsPerWave, "rpw %d", tl.rpw);
    CHECK(tl.ncols >= 1 && tl.ncols <= L * V && tl.col0 % V == 0, "ncols %d", tl.ncols);
    CHECK(tl.col0 + tl.ncols == n || tl.ncols % V == 0, "partial lane inside a row");
    CHECK(tl.count <= kStreamWaves * tl.rpw && tl.start + tl.count <= m, "row range");
    std::vector<int> lds(static_cast<size_t>(tl.ncols), 0);
    for (int wave = 0; wave < kStreamWaves; ++wave) {
        const int64_t r0 = tl.start + int64_t(wave) * tl.rpw;
        int nr = static_cast<int>(tl.start + tl.count - r0);
        nr = nr < 0 ? 0 : (nr > tl.rpw ? tl.rpw : nr);
        const int nld = (nr + G - 1) >> (6 - llog);
        for (int lane = 0; lane < kWave; ++lane) {
            const int seg = lane >> llog, ccol = (lane & (L - 1)) * V;
            const bool colok = ccol < tl.ncols;
            const int64_t c = colok ? tl.col0 + ccol : tl.col0;
            const int64_t lcol = c < n - V ? c : n - V;
            const int skip = static_cast<int>(c - lcol);
            CHECK(lcol >= 0 && lcol + V <= n && skip >= 0 && skip < V, "column %lld skip %d",
                  (long long)lcol, skip);
            // rows of a load: the wave's own, else its first; the read passes
            // of a wave without rows use the tile's first
            for (int rl = 0; rl < kMaxRowsPerWave + G; ++rl) {
                const int64_t row = rl < nr ? r0 + rl : nr > 0 ? r0 : tl.start;
                CHECK(row * n + lcol + V <= mn, "load past the tensor");
            }
            for (int ld = 0; ld < nld; ++ld) {
                const int rl = ld * G + seg;
                if (!colok || rl >= nr) continue;
                for (int i = skip; i < V; ++i)
                    elems[ti].hit((r0 + rl) * n + lcol + i, "element");
            }
            if (wave == 0 && lane < L && colok)
                for (int i = skip; i < V; ++i) {
                    const int j = ccol - skip + i;
                    CHECK(j >= 0 && j < tl.ncols, "column slot %d of %d", j, tl.ncols);
                    if (j >= 0 && j < tl.ncols) lds[static_cast<size_t>(j)] += 1;
                }
            if (lane < nr) rowp[ti].hit(int64_t(tl.cb) * pad4(m) + r0 + lane, "rowpart");
        }
    }
    for (int j = 0; j < tl.ncols; ++j) {
        CHECK(lds[static_cast<size_t>(j)] == 1, "column slot %d written %d times", j,
              lds[static_cast<size_t>(j)]);
        colp[ti].hit(colpart_index(tl.col0 + j, tl.stripe, td.nrs), "colpart");
    }
}

static void check_wide_plan(const Plan &pl, int64_t count)
{
    const size_t nt = static_cast<size_t>(count);
    std::vector<Marks> elems(nt), rowp(nt), colp(nt), chunks(nt), rows(nt), cols(nt);
    for (size_t i = 0; i < nt; ++i) {
        const TensorDesc &td = pl.tensors[i];
        elems[i].init(td.m * td.n);
        if (td.kind != KIND_MATRIX) continue;
        rowp[i].init(int64_t(td.ncb) * pad4(td.m));
        colp[i].init(colpart_floats(td.n, td.nrs));
        chunks[i].init(td.nchunk);
        rows[i].init(td.m);
        cols[i].init(td.n);
        CHECK(td.rowpart % 4 == 0 && td.colpart % 4 == 0 &&
                  td.rowpart + int64_t(td.ncb) * pad4(td.m) <= td.colpart &&
                  td.colpart + colpart_floats(td.n, td.nrs) <= td.chunk &&
                  td.chunk + td.nchunk <= pl.ws_floats, "workspace");
    }
    int64_t covered = 0;
    for (const TileGroup &g : pl.groups) {
        CHECK(g.begin == covered && g.count > 0, "groups");
        covered += g.count;
        for (int64_t t = g.begin; t < g.begin + g.count; ++t) {
            const Tile &tl = pl.tiles[static_cast<size_t>(t)];
            CHECK(tl.dtype == g.dtype, "tile dtype vs group");
            if (tl.kind != KIND_MATRIX) continue;
            CHECK(tl.ragged ? g.ragged && g.vec == 4 : tl.vec == 1 || (tl.vec == 4 && g.vec == 4),
                  "tile form vs group");
        }
    }
    CHECK(covered == static_cast<int64_t>(pl.tiles.size()), "groups do not cover tiles");
    for (const Tile &tl : pl.tiles) {
        if (tl.kind != KIND_MATRIX) check_vector_tile(pl, tl, elems);
        else if (tl.ragged) check_ragged_tile(pl, tl, elems, rowp, colp);
        else check_matrix_tile(pl, tl, elems, rowp, colp);
    }
    const int T = 1 << pl.fin_log2, W = T / kWave;
    bool wide = false;
    for (size_t q = 0; q < pl.fin.size(); ++q) {
        const FinItem &it = pl.fin[q];
        const size_t ti = static_cast<size_t>(it.tensor);
        const TensorDesc &td = pl.tensors[ti];
        CHECK((it.kind == FIN_COLS) == (static_cast<int64_t>(q) >= pl.row_items), "item order");
        if (it.kind == FIN_COLS) {
            for (int j = 0; j < it.count; ++j) cols[ti].hit(int64_t(it.start) + j, "column item");
            continue;
        }
        CHECK(it.kind == (td.ncb > kFinWideBlocks ? FIN_ROWS_WIDE : FIN_ROWS), "row item kind");
        wide = wide || it.kind == FIN_ROWS_WIDE;
        for (int j = 0; j < it.count; ++j) rows[ti].hit(int64_t(it.start) + j, "row item");
        CHECK(it.f == td.r && it.len == td.m && it.part == td.rowpart && it.nparts == td.ncb,
              "row item descriptor");
        if (it.kind == FIN_ROWS) {
            for (int w = 0; w < W; ++w)
                if (w * kChunkRows < it.count) chunks[ti].hit(it.chunk - td.chunk + w, "chunk");
            continue;
        }
        CHECK(it.start % kChunkRows == 0 && it.count <= kChunkRows, "split row item");
        chunks[ti].hit(it.chunk - td.chunk, "chunk");
        CHECK(it.chunk == td.chunk + it.start / kChunkRows, "chunk of a split row item");
        const int per = (it.nparts + W - 1) / W, NL = kFinWideLoads(T);
        std::vector<int> seen(static_cast<size_t>(it.nparts), 0);
        for (int w = 0; w < W; ++w) {
            const int b0 = w * per < it.nparts ? w * per : it.nparts;
            const int b1 = b0 + per < it.nparts ? b0 + per : it.nparts;
            for (int cb = b0; cb < b1; cb += NL)
                for (int u = 0; u < NL; ++u) {
                    const int b = cb + u < b1 ? cb + u : b1 - 1;
                    for (int lane = 0; 4 * lane < it.count; ++lane) {
                        const int64_t off = int64_t(b) * pad4(td.m) + it.start + 4 * lane;
                        CHECK(off % 4 == 0 && off + 4 <= int64_t(td.ncb) * pad4(td.m), "rowpart read");
                        for (int j = 0; j < 4 && 4 * lane + j < it.count; ++j)
                            CHECK(rowp[ti].v[static_cast<size_t>(off + j)] == 1, "read before written");
                    }
                    if (cb + u < b1) seen[static_cast<size_t>(b)] += 1;
                }
        }
        for (int b = 0; b < it.nparts; ++b)
            CHECK(seen[static_cast<size_t>(b)] == 1, "block %d read %d times", b,
                  seen[static_cast<size_t>(b)]);
    }
    CHECK(pl.fin_wide == wide, "finalisation form");
    for (size_t i = 0; i < nt; ++i) {
        const TensorDesc &td = pl.tensors[i];
        CHECK(elems[i].all(), "tensor %lldx%lld not covered", (long long)td.m, (long long)td.n);
        if (td.kind != KIND_MATRIX) continue;
        CHECK(rowp[i].all_rows(pad4(td.m), td.m) && chunks[i].all() && rows[i].all() &&
                  cols[i].all(), "%lldx%lld: partials or items incomplete", (long long)td.m,
              (long long)td.n);
        for (int64_t st = 0; st < td.nrs; ++st)
            for (int64_t j = 0; j < td.n; ++j)
                CHECK(colp[i].v[static_cast<size_t>(colpart_index(j, st, td.nrs))],
                      "column partial missing");
    }
}

int main()
{
    std::mt19937_64 rng(99);
    const int64_t ns[] = {2, 3, 4, 5, 7, 9, 27, 33, 63, 129, 253, 255, 256, 257, 259, 384, 509, 513,
                          769, 1000, 1025, 4097, 4353, 5003};
    const int64_t ms[] = {2, 3, 5, 31, 33, 64, 129, 255, 257, 1000, 1025};
    const uintptr_t base = uintptr_t(1) << 40;
    int ragged = 0, split = 0;
    for (int trial = 0; trial < 150; ++trial) {
        const int count = 1 + static_cast<int>(rng() % 5);
        std::vector<rikfad_tensor> ts(static_cast<size_t>(count));
        for (int i = 0; i < count; ++i) {
            rikfad_tensor &t = ts[static_cast<size_t>(i)];
            t = rikfad_tensor{};
            t.m = ms[rng() % (sizeof(ms) / sizeof(ms[0]))];
            t.n = ns[rng() % (sizeof(ns) / sizeof(ns[0]))];
            if (trial % 50 == 7 && i == 0) { t.m = 37; t.n = 50257; }
            if (trial % 50 == 9 && i == 0) { t.m = 50257; t.n = 5; }
            if (trial % 50 == 11 && i == 0) { t.m = 20000; t.n = 33; }
            t.dtype = rng() % 2 ? RIKFAD_BF16 : RIKFAD_FP32;
            const uintptr_t es = t.dtype == RIKFAD_BF16 ? 2 : 4, slot = base + (uintptr_t(i) << 34);
            t.x = reinterpret_cast<void *>(slot + (rng() % 3 ? 0 : es));
            t.g = reinterpret_cast<const void *>(slot + (uintptr_t(1) << 32));
            t.p = reinterpret_cast<float *>(slot + (uintptr_t(2) << 32));
            t.r = reinterpret_cast<float *>(slot + (uintptr_t(3) << 32));
            t.c = reinterpret_cast<float *>(slot + (uintptr_t(3) << 32) + (uintptr_t(1) << 31));
        }
        for (int rpw : {0, 3, 16}) {
            Plan pl;
            std::string err;
            CHECK(plan_rikfad(ts.data(), count, pl, err, rpw, true) == RIKFAD_OK, "%s", err.c_str());
            check_wide_plan(pl, count);
            for (const Tile &tl : pl.tiles) ragged += tl.ragged;
            for (const FinItem &it : pl.fin) split += it.kind == FIN_ROWS_WIDE;
            for (int i = 0; i < count; ++i) {       // every unaligned row of 4 columns or more
                const rikfad_tensor &t = ts[static_cast<size_t>(i)];
                const bool want = t.m > 1 && t.n >= 4 && pl.tensors[static_cast<size_t>(i)].vec == 1;
                for (const Tile &tl : pl.tiles)
                    if (tl.tensor == i) CHECK((tl.ragged != 0) == want, "tile form of %lld columns",
                                              (long long)t.n);
            }
        }
    }
    std::printf("plan_wide_check: %d ragged tiles, %d split items, %d failures\n", ragged, split,
                failures);
    return failures == 0 && ragged > 0 && split > 0 ? 0 : 1;
}
