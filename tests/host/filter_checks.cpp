// Host-only checks of the matrix-core filters' planning (api.cpp), built like
// host_checks.cpp, whose stubs and template sets it uses, and run by
// tests/test_host_filter.py.  No GPU: operands are stand-ins that look
// complete.
//
//   filter_checks <iterations> <seed>
//
// For random template sets, frame sizes and pair lists, FP32 (with and without
// the launch of the last columns) and FP64, by rule and for all pairs: every
// pair is filtered once or scored at every offset; each filtered pair's tiles
// are items once; maps and blocks of a chunk lie side by side inside the
// scratch, chunks keep to its limit; LDS sizes suffice; the work items left
// are those of the other pairs, and those of the filtered ones fit the list
// for undecided pairs; the direct form's lists cover every offset once.  The
// ordered records of an FP32 sum stay inside the window and give the segments'
// box sums.  The two-threshold search's filter has a bit for every offset and
// a counter for every tile.  Exit status 0 when every check holds.

#define main host_checks_main
#include "host_checks.cpp"
#undef main

static unsigned long long g_built = 1;

// Operands of every template that look built and complete.
static void stand_ins(sncc_tmpl &tm, const std::shared_ptr<BuildCount> &count) {
  tm.digits32.clear();
  tm.digits_f.clear();
  tm.error_f.clear();
  tm.dense.assign(kDenseForms * (size_t)tm.T, {});
  auto buf = std::make_shared<DenseBuf>();
  buf->count = count;
  buf->ticket = 1;
  for (int t = 0; t < tm.T; ++t) {
    float error = 0.f;
    tm.digits32.push_back(dense_digits32(&tm, t));
    tm.digits_f.push_back(dense_digits_filter(&tm, t, &error));
    tm.error_f.push_back(error);
    for (int digits : {2, 3, 4, 7}) {
      DenseTmpl dt;
      (void)dense_fixed_point(&tm, t, digits, dt);
      dt.frag = &g_built;
      dt.buf = buf;
      tm.dense[kDenseForms * (size_t)t + dense_form(digits)].push_back(dt);
    }
  }
}

// Ranges [first, first + size) must not overlap nor pass `end`.
static void check_ranges(std::vector<std::pair<long long, long long>> r, long long end,
                         const char *what) {
  std::sort(r.begin(), r.end());
  long long at = 0;
  for (const auto &x : r) {
    CHECK(x.first >= at && x.second >= 0, "%s overlap at %lld", what, x.first);
    at = x.first + x.second;
  }
  CHECK(at <= end, "%s end at %lld of %lld", what, at, end);
}

// Tiles of the filter pairs [fp0, fp0 + n) listed in items once each.
static void check_items(const std::vector<FilterPair> &fps, const std::vector<int2> &items,
                        const std::vector<FilterLaunch> &launches, int fp0, int n) {
  std::vector<std::vector<int>> seen(n);
  for (int j = 0; j < n; ++j) seen[j].assign(fps[fp0 + j].a.ntu * fps[fp0 + j].a.ntv, 0);
  for (const FilterLaunch &l : launches) {
    CHECK(l.item0 >= 0 && l.item0 + l.n_items <= (int)items.size(), "launch items");
    CHECK(l.lds <= kTileMaxLds / 2, "LDS %d", l.lds);
    for (int i = l.item0; i < l.item0 + l.n_items; ++i) {
      if (items[i].x < 0) continue;
      CHECK(items[i].x < n, "item's pair");
      if (items[i].x >= n) continue;
      const FilterPair &fp = fps[fp0 + items[i].x];
      CHECK(fp.a.digits == l.digits && fp.a.rv == l.rv, "launch shape");
      CHECK(l.lds >= (2 * kDenseNW * l.rv + fp.a.hb - 1) * fp.a.pitch, "LDS too small");
      CHECK(items[i].y < (int)seen[items[i].x].size(), "tile");
      if (items[i].y < (int)seen[items[i].x].size()) ++seen[items[i].x][items[i].y];
    }
  }
  for (const auto &s : seen)
    for (int c : s) CHECK(c == 1, "tile listed %d times", c);
}

static void check_filter(const sncc_tmpl &tm, FilterPlan &f, const std::vector<char> &use,
                         int n_pairs, const int32_t *pairs, bool fp64, size_t limit, int k,
                         PlanHost *tile, PlanHost *edge) {
  std::vector<int> count(n_pairs, 0);
  long long und[2] = {0, 0};
  for (const FilterChunk &c : f.chunks) {
    std::vector<std::pair<long long, long long>> maps, blocks;
    long long floats = 0;
    for (int j = c.fp0; j < c.fp0 + c.n_fps; ++j) {
      const FilterPair &fp = f.fps[j];
      ++count[fp.pair];
      const long long n = (long long)fp.n_blocks * fp.a.rv * 256;
      CHECK(fp.n_blocks == fp.a.ntu * fp.a.ntv * kDenseNW, "blocks");
      CHECK(fp.a.ntu * (long long)kDenseBU >= fp.a.nu &&
                fp.a.ntv * 2LL * kDenseNW * fp.a.rv >= fp.a.nv, "tiles cover the map");
      maps.emplace_back(fp.map0, n);
      blocks.emplace_back(fp.block0, fp.n_blocks);
      floats += n;
      for (int x = 0; x < 2; ++x) {
        CHECK(fp.n_seq[x] % 8 == 0 && fp.seq0[x] + fp.n_seq[x] <= (int)f.seq.size(), "records");
        const PlanHost *h = x ? edge : tile;
        CHECK(fp.n_items[x] == (h ? h->pairs[fp.pair].item_end - h->pairs[fp.pair].item_begin : 0),
              "items of pair %d", fp.pair);
        und[x] += fp.n_items[x];
      }
    }
    check_ranges(maps, (long long)f.map_floats, "maps");
    check_ranges(blocks, (long long)f.blocks, "blocks");
    CHECK(c.n_fps == 1 || floats <= (long long)limit, "chunk of %lld floats", floats);
    check_items(f.fps, f.items, c.launches, c.fp0, c.n_fps);
  }
  for (int p = 0; p < n_pairs; ++p) {
    CHECK(count[p] == (use[p] ? 1 : 0), "pair %d filtered %d times", p, count[p]);
    CHECK(f.direct[p] == !use[p], "pair %d scored at every offset", p);
  }
  CHECK(f.und_items[0] == und[0] && f.und_items[1] == und[1], "items of undecided pairs");
  CHECK(f.und_queue(0) == 0 && (f.und_queue(0) + kQueueInts) % 2 == 0, "floors' alignment");
  CHECK(f.und_bounds(0) >= kQueueInts + 2 * n_pairs && f.und_queue(1) >= f.und_bounds(0) + 2 &&
            f.und_zero() >= f.und_bounds(1) + 2, "undecided pairs' counters");
  if (fp64) {
    int at = 0;
    for (const SeqPair &q : f.pairs) {
      CHECK(q.chunk0 == at && (long long)q.chunk * q.n_chunks >= (long long)q.nu * q.nv &&
                (long long)q.chunk * (q.n_chunks - 1) < (long long)q.nu * q.nv, "lists");
      at += q.n_chunks;
    }
    CHECK(at == f.n_lists && f.seq_grid >= 1, "lists in all");
    return;
  }
  for (PlanHost *h : {tile, edge}) {
    if (!h) continue;
    drop_items(*h, use);
    std::vector<int> seen(h->items.size(), 0);
    for (int i : h->order) ++seen[i];
    for (size_t i = 0; i < seen.size(); ++i)
      CHECK(seen[i] == (use[h->items[i].pair] ? 0 : 1), "item %zu listed %d times", i, seen[i]);
    CHECK(h->qbeg.back() == (int)h->order.size() && h->grid >= 1, "queues");
  }
}

// The ordered records of template t give the segments' box sums over a window
// of a random table, with areas and c.
static void check_records(std::mt19937_64 &rng, const sncc_tmpl &tm, const PlanHost &ph, int t,
                          int P, const std::vector<SeqRec> &seq, int seq0, int n_seq) {
  const int W = tm.W[t], H = tm.H[t];
  std::vector<uint32_t> s((size_t)(H + 1) * P, 0);
  for (int y = 1; y <= H; ++y) {
    uint32_t row = 0;
    for (int x = 1; x <= W; ++x) {
      row += (uint32_t)(rng() % 256);
      s[(size_t)y * P + x] = s[(size_t)(y - 1) * P + x] + row;
    }
  }
  double got = 0, want = 0, size = 0;
  long long area = 0;
  for (int b = 0; b < n_seq; b += 8) {
    uint32_t prev = 0;
    int slots = 0;
    for (int j = 0; j < 8; ++j) {
      const SeqRec &e = seq[seq0 + b + j];
      CHECK(e.top % 4 == 0 && e.bot % 4 == 0 && e.top >= 0 && e.bot >= 0 &&
                e.top / 4 < (int)s.size() && e.bot / 4 < (int)s.size(), "record in the window");
      if (e.top / 4 >= (int)s.size() || e.bot / 4 >= (int)s.size()) return;
      const uint32_t D = s[e.bot / 4] - s[e.top / 4];
      if (!(e.area_flags & kSeqNoTerm)) {
        CHECK((int)((e.area_flags >> kSeqSlot) & 3) == slots++, "slot");
        if (!(e.area_flags & kSeqZero)) {
          got += (double)(D - prev) * e.c;
          area += e.area_flags & kSeqArea;
        }
      }
      prev = D;
    }
    CHECK(slots == 4, "%d terms in a block", slots);
  }
  for (size_t i = 0; i < tm.segs[t].size(); ++i) {
    const Seg &g = tm.segs[t][i];
    auto at = [&](int y, int x) { return s[(size_t)y * P + x]; };
    const uint32_t F = (at(g.y + g.h, g.x + g.w) - at(g.y + g.h, g.x)) -
                       (at(g.y, g.x + g.w) - at(g.y, g.x));
    want += (double)F * (float)tm.c64[t][i];
    size += std::fabs((double)F * tm.c64[t][i]);
  }
  CHECK(area == (long long)W * H, "areas %lld of %d", area, W * H);
  CHECK(std::fabs(got - want) <= 1e-9 * (size + 1.0), "sum %g for %g", got, want);
  (void)ph;
}

int main(int argc, char **argv) {
  const int iters = argc > 1 ? std::atoi(argv[1]) : 40;
  std::mt19937_64 rng(argc > 2 ? std::strtoull(argv[2], nullptr, 10) : 1);
  auto count = std::make_shared<BuildCount>();
  count->host = &g_built;
  sncc_ctx ctx;
  ctx.num_cu = 256;
  ctx.serial = 1;
  long long n_filtered = 0, n_above = 0;
  for (int i = 0; i < iters; ++i) {
    sncc_tmpl tm;
    const int T = 1 + (int)(rng() % 6);
    if (!make_set(rng, T, i % 4 == 0 ? 300 : 90, tm)) {
      CHECK(false, "fill_templates failed");
      continue;
    }
    stand_ins(tm, count);
    int maxW = 1, maxH = 1;
    for (int t = 0; t < T; ++t) maxW = std::max(maxW, tm.W[t]), maxH = std::max(maxH, tm.H[t]);
    const int M = maxW + (int)(rng() % 900), N = maxH + (int)(rng() % 600);
    int P = 0;
    sncc_sat_pitch(M, &P);
    std::vector<int32_t> pairs;
    const int B = 1 + (int)(rng() % 3), n_pairs = 1 + (int)(rng() % 20);
    for (int p = 0; p < n_pairs; ++p) {
      pairs.push_back((int)(rng() % B));
      pairs.push_back((int)(rng() % T));
    }
    const int k = 1 + (int)(rng() % 64);
    const size_t limit = i % 3 == 0 ? (size_t)1 << 18 : kFilterMapFloats;
    for (const char *form : {"", "1"}) {
      setenv("SNCC_TEST_DENSE", form, 1);
      for (int kind = 0; kind < 3; ++kind) {  // FP32 call, batch with last columns, FP64 call
        PlanHost tile, edge;
        if (kind == 0)
          CHECK(build_one_call_plan(&tm, M, N, P, n_pairs, pairs.data(), k, kSinkTopk, 256,
                                    tile) == SNCC_OK, "plan");
        if (kind == 1) {
          CHECK(build_plan(&tm, 0, M, N, P, n_pairs, pairs.data(), k, kSinkTopk, 256, tile,
                           nullptr, kSplitMain) == SNCC_OK, "main plan");
          int e = -1;
          const TileCfg tc = tile_cfg_of(0);
          for (int c = 0; c < kNumCfgs; ++c) {
            const TileCfg ec = tile_cfg_of(c);
            if (ec.ru == 1 && ec.rv == tc.rv && ec.nw == tc.nw && ec.wgs == tc.wgs) e = c;
          }
          CHECK(build_plan(&tm, e, M, N, P, n_pairs, pairs.data(), k, kSinkTopk, 256, edge,
                           nullptr, kSplitEdge, tc.bu()) == SNCC_OK, "last columns' plan");
        }
        std::vector<char> use =
            filter_pairs(&ctx, &tm, M, N, n_pairs, pairs.data(), k, kind == 2, kind == 1);
        FilterPlan f;
        plan_filter(&ctx, &tm, M, N, P, n_pairs, pairs.data(), k, kind == 2,
                    kind == 2 ? nullptr : &tile, use, f, limit, kind == 1 ? &edge : nullptr);
        n_filtered += (long long)f.fps.size();
        CHECK(!f.missing, "operands missing");
        for (const FilterPair &fp : f.fps)
          for (int x = 0; x < 2 && kind != 2; ++x)
            if (fp.n_seq[x] > 0)
              check_records(rng, tm, x ? edge : tile, pairs[2 * fp.pair + 1], P, f.seq, fp.seq0[x],
                            fp.n_seq[x]);
        check_filter(tm, f, use, n_pairs, pairs.data(), kind == 2, limit, k,
                     kind == 2 ? nullptr : &tile, kind == 1 ? &edge : nullptr);
      }
      // the two-threshold search (its buffers cannot be had here: the plan is
      // complete before them)
      PlanHost fast;
      const std::vector<double> lo(T, 0.4), hi(T, 0.9);
      CHECK(build_plan(&tm, 0, M, N, P, n_pairs, pairs.data(), 1, kSinkCompact, 256, fast,
                       lo.data()) == SNCC_OK, "fast plan");
      AbovePlan a;
      (void)plan_above(&ctx, &tm, fast, N, P, n_pairs, pairs.data(), lo.data(), hi.data(), a);
      CHECK(a.active() || a.n_tiles == 0, "counters without a filter");
      if (!a.active()) continue;
      n_above += (long long)a.fps.size();
      std::vector<std::pair<long long, long long>> words, counters;
      for (int p = 0; p < n_pairs; ++p)
        counters.emplace_back(a.tile0[p], (long long)fast.pairs[p].ntu * fast.pairs[p].ntv);
      check_ranges(counters, a.n_tiles, "counters");
      for (size_t j = 0; j < a.fps.size(); ++j) {
        const FilterPair &fp = a.fps[j];
        CHECK(a.fp_of_pair[fp.pair] == (int)j && fp.block0 == a.tile0[fp.pair] &&
                  fp.n_blocks == fast.pairs[fp.pair].ntv && fp.a.ntu == fast.pairs[fp.pair].ntu,
              "counters of pair %d", fp.pair);
        CHECK(fp.min_count >= 1 && fp.above <= 0.9f, "limits");
        words.emplace_back(fp.map0, (long long)fp.a.ntu * fp.a.ntv * kDenseNW * 64);
      }
      check_ranges(words, (long long)a.words, "bit words");
      check_items(a.fps, a.items, a.launches, 0, (int)a.fps.size());
    }
  }
  count->host = nullptr;
  CHECK(n_filtered > 0 && n_above > 0, "nothing planned");
  printf("filter_checks: %lld filtered pairs, %lld of the two-threshold search, %d failures\n",
         n_filtered, n_above, g_fail);
  return g_fail ? 1 : 0;
}
