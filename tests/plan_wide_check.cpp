// plan_wide_check.cpp -- plan_check.cpp's replay over sets that are mostly
// ragged (4-wide accesses at element alignment) or have enough column blocks
// for split row items, in both sizes of the finalisation workgroup.  Built
// with -fsanitize=address,undefined by the test that runs it.
#define main plan_check_main
#include "plan_check.cpp"
#undef main

// Ragged tiles of a set of `count` m x n matrices, all of one storage type, and
// one aligned 8 x 8 matrix of that type if `even`.
static int ragged_tiles(int count, int64_t m, int64_t n, int32_t dtype, bool even = false)
{
    std::vector<rikfad_tensor> ts(static_cast<size_t>(count) + (even ? 1 : 0));
    for (size_t i = 0; i < ts.size(); ++i) {
        rikfad_tensor &t = ts[i];
        const uintptr_t slot = (uintptr_t(1) << 40) + (uintptr_t(i) << 24);
        const bool last = even && i + 1 == ts.size();
        t = rikfad_tensor{};
        t.m = last ? 8 : m;
        t.n = last ? 8 : n;
        t.dtype = dtype;
        t.x = reinterpret_cast<void *>(slot + (last ? 0 : 4));
        t.g = reinterpret_cast<const void *>(slot + (uintptr_t(1) << 21));
        t.p = reinterpret_cast<float *>(slot + (uintptr_t(2) << 21));
        t.r = reinterpret_cast<float *>(slot + (uintptr_t(3) << 21));
        t.c = reinterpret_cast<float *>(slot + (uintptr_t(4) << 21));
    }
    Plan pl;
    std::string err;
    CHECK(plan_rikfad(ts.data(), static_cast<int64_t>(ts.size()), pl, err) == RIKFAD_OK, "%s",
          err.c_str());
    check_plan(pl, static_cast<int64_t>(ts.size()), /*tiny=*/pl.groups.back().vec == 1);
    int ragged = 0;
    for (const Tile &tl : pl.tiles) ragged += tl.ragged;
    return ragged;
}

int main()
{
    // Thousands of ragged tiles of a few elements take one-column tiles, unless
    // the 4-wide kernel has to run for another matrix, the tiles fit in one
    // round, hold more, or would each be two.
    for (int32_t dt : {RIKFAD_FP32, RIKFAD_BF16}) {
        CHECK(ragged_tiles(600, 3, 5, dt) == 0 && ragged_tiles(513, 64, 27, dt) == 0, "tiny tiles");
        CHECK(ragged_tiles(600, 20, 8, dt) == 0, "tiny tiles of misaligned views");
        CHECK(ragged_tiles(600, 3, 5, dt, true) == 600, "an aligned matrix beside them");
        CHECK(ragged_tiles(512, 3, 5, dt) == 512, "one round of tiles");
        CHECK(ragged_tiles(513, 64, 33, dt) == 513, "two one-column tiles for one");
        CHECK(ragged_tiles(513, 500, 4, dt) == 513, "tiles of 2,000 elements");
    }
    // Narrow ragged matrices a little taller than a stripe are shared out evenly.
    for (int64_t m : {192, 300, 384, 448, 600}) {
        rikfad_tensor t{};
        t.m = m;
        t.n = 27;
        t.x = t.p = t.r = t.c = reinterpret_cast<float *>(uintptr_t(1) << 40);
        t.g = t.x;
        std::vector<rikfad_tensor> ts(256, t);      // past the rule for small sets
        Plan pl;
        std::string err;
        CHECK(plan_rikfad(ts.data(), 256, pl, err) == RIKFAD_OK, "%s", err.c_str());
        const int64_t stripes = (m + 255) / 256, per_wave = ((m + stripes - 1) / stripes + 7) / 8;
        for (const Tile &tl : pl.tiles)
            CHECK(tl.ragged && tl.rpw == (per_wave + 7) / 8 * 8 && pl.tensors[0].nrs == stripes,
                  "%lld x 27: %d rows per wave", (long long)m, tl.rpw);
    }
    std::mt19937_64 rng(99);
    const int64_t ns[] = {2, 3, 4, 5, 7, 9, 27, 33, 63, 129, 253, 255, 256, 257, 259, 384, 509, 513,
                          769, 1000, 1025, 4097, 4353, 5003};
    const int64_t ms[] = {2, 3, 5, 31, 33, 64, 129, 255, 257, 1000, 1025};
    const uintptr_t base = uintptr_t(1) << 40;
    int ragged = 0, split[2] = {0, 0};
    for (int trial = 0; trial < 150; ++trial) {
        const int count = (trial % 50 == 13 ? 2 : 1) + static_cast<int>(rng() % 5);
        std::vector<rikfad_tensor> ts(static_cast<size_t>(count));
        for (int i = 0; i < count; ++i) {
            rikfad_tensor &t = ts[static_cast<size_t>(i)];
            t = rikfad_tensor{};
            t.m = ms[rng() % (sizeof(ms) / sizeof(ms[0]))];
            t.n = ns[rng() % (sizeof(ns) / sizeof(ns[0]))];
            if (trial % 50 == 7 && i == 0) { t.m = 37; t.n = 50257; }
            if (trial % 50 == 9 && i == 0) { t.m = 50257; t.n = 5; }
            if (trial % 50 == 11 && i == 0) { t.m = 20000; t.n = 33; }
            if (trial % 50 == 13 && i < 2) { t.m = i ? 259 : 17000; t.n = i ? 6001 : 256; }
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
            CHECK(plan_rikfad(ts.data(), count, pl, err, rpw) == RIKFAD_OK, "%s", err.c_str());
            check_plan(pl, count);
            if (trial % 50 == 13 && rpw == 0)
                CHECK(pl.fin_log2 == kFinLargeLog2, "17000 rows of 256 columns: 256-thread items");
            for (const Tile &tl : pl.tiles) ragged += tl.ragged;
            for (const FinItem &it : pl.fin)
                split[pl.fin_log2 == kFinLargeLog2] += it.kind == FIN_ROWS_WIDE;
        }
    }
    std::printf("plan_wide_check: %d ragged tiles, %d + %d split items, %d failures\n", ragged,
                split[0], split[1], failures);
    return failures == 0 && ragged > 0 && split[0] > 0 && split[1] > 0 ? 0 : 1;
}
