// The split of the dK/dV pass (kv_split, add_split in nsp_abi.cpp) on seeded
// random work lists, against the rules it has to keep: every step of every key
// tile in exactly one piece, in order; a tile in several pieces has one slot
// for each, consecutive and its own, and one entry in the sum pass; no more
// shares than compute units and none much longer than the mean; a masked call
// runs exactly the unmasked call's pieces of its items, shared out evenly; the workspace that the
// query asks for and the allocation-free scratch hold the slots.  And the gangs of
// the forward / dQ units: the unit list, or its halves, on queues of about equal
// work, of a kind that changes results only with the whole list, and, on the lists
// of the file that the program is given, well balanced.  Built with g++
// from the library's host sources; prints "split checks ok".
#include "nsp_abi.cpp"

#include <cstdlib>
#include <map>
#include <random>
#include <set>

#define CHECK(c)                                                                 \
  do {                                                                           \
    if (!(c)) {                                                                  \
      std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
      std::exit(1);                                                              \
    }                                                                            \
  } while (0)

namespace {

std::mt19937_64 rng(411);
int uni(int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); }

using Key = std::tuple<int, int, int>;   // item, tile, KV head

void check_list(const nsp_worklist &w, const std::vector<uint8_t> &mask, int *n_split) {
  WlInfo info;
  CHECK(validate_worklist(&w, &info) == NSP_OK);
  const KvSplit sp = kv_split(&w);
  const size_t slot_bytes = nsp::kv_slot_floats(w.head_dim) * sizeof(float);
  CHECK(nsp_varlen_attn_bwd_workspace(&w) == bwd_workspace_bytes(info) + nsp::kKvSlots * slot_bytes);
  HostAttnSched full;
  add_split(full, &w);
  if (sp.pieces.empty()) {
    CHECK(full.kv_wgs.empty() && sp.slots == 0);
    return;
  }
  ++*n_split;
  CHECK(bwd_workspace_bytes(info) + sp.slots * slot_bytes <= nsp::kScratchBytes - nsp::kScratchSchedBytes);
  CHECK(sp.slots <= nsp::kKvSlots);
  // pieces of each tile, in launch-list order of the whole call
  std::map<Key, std::vector<nsp::KvPiece>> tiles;
  int64_t total = 0, longest = 0;
  for (size_t i = 0; i + 1 < sp.share.size(); ++i) {
    int64_t c = 0;
    for (int k = sp.share[i]; k < sp.share[i + 1]; ++k) {
      tiles[Key(sp.pieces[k].item, sp.pieces[k].tile, sp.pieces[k].g)].push_back(sp.pieces[k]);
      c += sp.pieces[k].count + kPieceCost;
    }
    CHECK(c > 0);
    total += c;
    longest = std::max(longest, c);
  }
  CHECK((int)sp.share.size() - 1 <= kAssumedCUs);
  CHECK(longest <= 2 * (total / kAssumedCUs + kPieceCost + kMinPiece));
  std::map<Key, nsp::KvReduce> sums;
  for (const nsp::KvReduce &r : sp.reduce) CHECK(sums.emplace(Key(r.item, r.tile, r.g), r).second);
  std::set<int> slots;
  size_t n_tiles = 0;
  for (int j = 0; j < w.n_items; ++j) {
    const int L = w.cu_seqlens[j + 1] - w.cu_seqlens[j];
    const int nk = (L + 127) / 128, nq = (L + 63) / 64;
    for (int g = 0; g < w.kv_heads[2 * j + 1] - w.kv_heads[2 * j]; ++g) {
      int h0 = -1, h1 = -1;
      for (int i = w.q_heads[2 * j]; i < w.q_heads[2 * j + 1]; ++i)
        if ((int64_t)i * w.hkv_total / w.hq_total == w.kv_heads[2 * j] + g) {
          if (h0 < 0) h0 = i - w.q_heads[2 * j];
          h1 = i - w.q_heads[2 * j] + 1;
        }
      for (int n = 0; n < nk; ++n, ++n_tiles) {
        auto it = tiles.find(Key(j, n, g));
        CHECK(it != tiles.end());
        int64_t at = 0;
        const int steps = h0 < 0 ? 0 : (h1 - h0) * (nq - 2 * n);
        auto r = sums.find(Key(j, n, g));
        CHECK((r != sums.end()) == (it->second.size() > 1));
        for (size_t k = 0; k < it->second.size(); ++k) {
          const nsp::KvPiece &p = it->second[k];
          CHECK(p.first == at && (p.count > 0 || steps == 0));
          CHECK(p.heads == (h0 < 0 ? 0 : (h0 | (h1 << 16))));
          at += p.count;
          if (r == sums.end()) CHECK(p.slot == -1);
          else CHECK(p.slot == r->second.slot + (int)k && p.slot < sp.slots && slots.insert(p.slot).second);
        }
        CHECK(at == steps);
        if (r != sums.end()) CHECK(r->second.count == (int)it->second.size());
      }
    }
  }
  CHECK(n_tiles == tiles.size() && (int)slots.size() == sp.slots);
  // the device lists of the whole and of a masked call
  for (int pass = 0; pass < 2; ++pass) {
    nsp_worklist m = w;
    m.item_mask = pass ? mask.data() : nullptr;
    HostAttnSched s;
    add_split(s, &m);
    CHECK(nsp_varlen_attn_bwd_workspace(&m) == nsp_varlen_attn_bwd_workspace(&w));
    size_t want = 0, sums_want = 0;
    for (const nsp::KvPiece &p : sp.pieces) want += selected(&m, p.item);
    for (const nsp::KvReduce &r : sp.reduce) sums_want += selected(&m, r.item);
    CHECK(s.kv_pieces.size() == want && s.kv_reduce.size() == sums_want);
    int at = 0;
    int64_t own = 0, piece = 0, share = 0;
    for (const int2 &wg : s.kv_wgs) {
      CHECK(wg.x == at && wg.y >= at);
      at = wg.y;
      int64_t c = 0;
      for (int k = wg.x; k < wg.y; ++k) {
        c += s.kv_pieces[k].count + kPieceCost;
        piece = std::max<int64_t>(piece, s.kv_pieces[k].count + kPieceCost);
      }
      own += c;
      share = std::max(share, c);
    }
    // a masked call uses the chip too
    if (pass) CHECK(share <= own / kAssumedCUs + piece && s.kv_wgs.size() <= (size_t)kAssumedCUs);
    CHECK(at == (int)want && s.kv_wgs.size() % 8 == 0);
    for (const nsp::KvPiece &p : s.kv_pieces) {
      CHECK(selected(&m, p.item));
      bool same = false;
      for (const nsp::KvPiece &o : tiles[Key(p.item, p.tile, p.g)]) same |= memcmp(&o, &p, sizeof p) == 0;
      CHECK(same);
    }
  }
}

// What a schedule's passes assume of each other.
void check_passes(const HostAttnSched &s) {
  CHECK(!s.small || (s.dq.kind == nsp::kQHalf && !s.kv_wgs.empty()));
  CHECK(s.kv_wgs.empty() || s.kv_units.empty());
}

void check_gangs(const nsp_worklist &w, int *kinds) {
  const HostAttnSched s = build_attn_schedule(&w, false, true);
  auto key = [](const int4 &u) { return std::make_tuple(u.x, u.y, u.z, u.w); };
  for (const QUnits *q : {&s.fwd, &s.dq}) {
    kinds[q->kind] += 1;
    const int rows = q->kind == nsp::kQWhole ? 256 : 128;
    std::multiset<std::tuple<int, int, int, int>> want, got;
    for (const int4 &u : s.fwd_units)
      for (int p = 0; p < 256 / rows; ++p) {
        const int tile = u.y * (256 / rows) + p, L = w.cu_seqlens[u.x + 1] - w.cu_seqlens[u.x];
        if (tile * rows < L) want.insert(std::make_tuple(u.x, tile, u.z, u.w));
      }
    for (const int4 &u : q->units) got.insert(key(u));
    CHECK(want == got && q->off.size() == 9 && q->off[0] == 0 && q->off[8] == (int)q->units.size());
    int64_t most = 0, total = 0, longest = 0;
    for (int x = 0; x < 8; ++x) {
      CHECK(q->off[x] <= q->off[x + 1]);
      int64_t work = 0;
      for (int k = q->off[x]; k < q->off[x + 1]; ++k) {
        const int L = w.cu_seqlens[q->units[k].x + 1] - w.cu_seqlens[q->units[k].x];
        const int64_t c = (std::min(L, rows * (q->units[k].y + 1)) + 63) / 64 + kUnitCost;
        work += c;
        longest = std::max(longest, c);
      }
      most = std::max(most, work);
      total += work;
    }
    CHECK(most <= total / 8 + longest * kFwdGang * (256 / rows));
  }
  // two key groups, one launch for dK/dV and dQ: decided alike for every mask
  nsp_worklist all = w;
  all.item_mask = nullptr;
  const HostAttnSched f = build_attn_schedule(&all, false, true);
  if (s.fwd_units.empty()) return;
  const HostAttnSched d = build_attn_schedule(&w);   // what the passes take
  check_passes(d);
  check_passes(build_attn_schedule(&w, true));
  CHECK(d.fwd.units.size() == s.fwd.units.size() && d.kv_units.size() == (d.kv_wgs.empty() ? s.kv_units.size() : 0));
  CHECK((f.fwd.kind == nsp::kQKeys) == (s.fwd.kind == nsp::kQKeys));
  CHECK((f.dq.kind == nsp::kQKeys) == (s.dq.kind == nsp::kQKeys));
  CHECK(f.small == s.small && (!s.small || (s.dq.kind == nsp::kQHalf && s.kv_wgs.size() % 8 == 0)));
}

// Whether a pass runs persistent workgroups: more units than the chip holds.
bool persistent(const QUnits &q, int head_dim, bool dq) {
  const int per_cu = q.kind != nsp::kQHalf ? 1 : dq && head_dim == 64 ? 3 : 2;
  return (int)q.units.size() > per_cu * kAssumedCUs && !q.one_shot;
}

// The lists of the GPU tests that stand for persistent passes run them: the kind
// of their forward and dQ units, and whether those and dK/dV are persistent.
void check_tested_lists() {
  struct {
    int L, n, sp, hq, hkv, D, fwd, dq;
    bool q_pers, kv_pers;
  } lists[] = {
      {256, 80, 1, 32, 4, 128, nsp::kQHalf, nsp::kQHalf, false, true},
      {700, 130, 1, 8, 2, 64, nsp::kQHalf, nsp::kQHalf, true, true},
      {700, 130, 1, 8, 2, 128, nsp::kQHalf, nsp::kQHalf, true, true},
      {2560, 14, 1, 8, 2, 128, nsp::kQWhole, nsp::kQWhole, true, true},
      {16384, 2, 8, 16, 2, 128, nsp::kQKeys, nsp::kQKeys, true, false},
  };
  for (auto &t : lists) {
    std::vector<int32_t> cu(1, 0), qh, kvh;
    for (int j = 0; j < t.n; ++j) {
      cu.push_back(cu.back() + t.L);
      qh.insert(qh.end(), {0, t.hq / t.sp});
      kvh.insert(kvh.end(), {0, std::max(1, t.hkv / t.sp)});
    }
    std::vector<uint8_t> mask(t.n, 0);
    mask[0] = 1;
    nsp_worklist w{};
    w.n_items = t.n;
    w.cu_seqlens = cu.data();
    w.q_heads = qh.data();
    w.kv_heads = kvh.data();
    w.hq_total = t.hq;
    w.hkv_total = t.hkv;
    w.head_dim = t.D;
    const HostAttnSched s = build_attn_schedule(&w);
    CHECK(s.fwd.kind == t.fwd && s.dq.kind == t.dq && !s.small);
    CHECK(persistent(s.fwd, t.D, false) == t.q_pers && persistent(s.dq, t.D, true) == t.q_pers);
    CHECK((s.kv_units.size() > (size_t)kAssumedCUs) == t.kv_pers && s.kv_wgs.empty() == t.kv_pers);
    w.item_mask = mask.data();
    const HostAttnSched m = build_attn_schedule(&w);
    CHECK(!persistent(m.fwd, t.D, false) && !persistent(m.dq, t.D, true) && m.kv_units.size() <= (size_t)kAssumedCUs);
  }
}

// Lists of short items and a few long ones: 128-row dQ units at head_dim 64 only
// where the long ones do not end the pass.
void check_long_units() {
  struct {
    int L, n, long_L, n_long, long_hq, hq, hkv, D, dq;
  } lists[] = {
      {100, 150, 9000, 1, 8, 8, 2, 64, nsp::kQWhole},   {100, 150, 9000, 1, 8, 8, 2, 128, nsp::kQHalf},
      {700, 100, 9000, 2, 1, 8, 2, 64, nsp::kQWhole},   {300, 232, 20000, 1, 1, 8, 2, 64, nsp::kQWhole},
      {100, 228, 9000, 1, 1, 8, 2, 64, nsp::kQHalf},    {700, 102, 9000, 2, 4, 32, 4, 64, nsp::kQHalf},
      {100, 695, 20000, 1, 4, 32, 4, 64, nsp::kQHalf},  {700, 102, 9000, 0, 1, 32, 4, 64, nsp::kQHalf},
  };
  for (auto &t : lists) {
    std::vector<int32_t> cu(1, 0), qh, kvh;
    for (int j = 0; j < t.n + t.n_long; ++j) {
      cu.push_back(cu.back() + (j < t.n ? t.L : t.long_L));
      qh.insert(qh.end(), {0, j < t.n ? t.hq : t.long_hq});
      kvh.insert(kvh.end(), {0, t.hkv});
    }
    nsp_worklist w{};
    w.n_items = t.n + t.n_long;
    w.cu_seqlens = cu.data();
    w.q_heads = qh.data();
    w.kv_heads = kvh.data();
    w.hq_total = t.hq;
    w.hkv_total = t.hkv;
    w.head_dim = t.D;
    CHECK(build_attn_schedule(&w).dq.kind == t.dq);
  }
}

// The queues that the forward and dQ passes run end within 1% of an even split by
// the model of a persistent pass, on the lists of a file: name, heads, head_dim,
// items (length, query heads, KV heads, whether the call has them).
void check_balance(const char *path) {
  FILE *f = std::fopen(path, "r");
  CHECK(f);
  char name[64];
  int n = 0, n_lists = 0;
  nsp_worklist w{};
  while (std::fscanf(f, "%63s %d %d %d %d", name, &w.hq_total, &w.hkv_total, &w.head_dim, &n) == 5) {
    std::vector<int32_t> cu(1, 0), qh(2 * n), kvh(2 * n);
    std::vector<uint8_t> mask(n);
    for (int j = 0; j < n; ++j) {
      int L = 0, on = 0;
      CHECK(std::fscanf(f, "%d %d %d %d %d %d", &L, &qh[2 * j], &qh[2 * j + 1], &kvh[2 * j], &kvh[2 * j + 1], &on) == 6);
      cu.push_back(cu.back() + L);
      mask[j] = (uint8_t)on;
    }
    w.n_items = n;
    w.cu_seqlens = cu.data();
    w.q_heads = qh.data();
    w.kv_heads = kvh.data();
    w.item_mask = mask.data();
    const HostAttnSched s = build_attn_schedule(&w);
    for (const QUnits *q : {&s.fwd, &s.dq}) {
      CHECK(q->kind == nsp::kQWhole);
      std::vector<int64_t> steps;
      int64_t total = 0;
      for (const int4 &u : q->units) {
        steps.push_back((std::min(cu[u.x + 1] - cu[u.x], 256 * (u.y + 1)) + 63) / 64);
        total += steps.back();
      }
      const double over = (double)kv_model_makespan(steps, q->off) * kAssumedCUs / (double)total;
      if (over > 1.01) std::fprintf(stderr, "%s: %zu units end at %.4f of an even split\n", name, steps.size(), over);
      CHECK(over <= 1.01);
    }
    ++n_lists;
  }
  std::fclose(f);
  CHECK(n_lists > 0);
}

// Lists near the allocation-free scratch's limits, whose schedules fit with
// 256-row units where the ones with 128-row units do not: of many short items, and
// of two items among empty ones, small enough for one launch (or for key groups).
// Of those a masked call takes the compact schedule too, and the longest such list
// that 256-row units alone allow (items, units and queues, 256 bytes for the
// blocks of a preprocess pass of its own) still fits.
void check_compact() {
  struct { int L, hq, hkv; bool small; } lone[] = {{300, 8, 2, true}, {512, 32, 4, true}, {4096, 4, 1, false}};
  for (auto &c : lone) {
    const int most = 174762;                           // as many empty items as the scratch describes
    std::vector<int32_t> cu(most + 1, c.L + 64), qh(2 * most), kvh(2 * most);
    std::vector<uint8_t> second(most, 0);
    cu[0] = 0;
    cu[1] = c.L;
    second[1] = 1;
    for (int j = 0; j < most; ++j) {
      qh[2 * j + 1] = c.hq;
      kvh[2 * j + 1] = c.hkv;
    }
    nsp_worklist w{};
    w.n_items = 2;
    w.cu_seqlens = cu.data();
    w.q_heads = qh.data();
    w.kv_heads = kvh.data();
    w.hq_total = c.hq;
    w.hkv_total = c.hkv;
    w.head_dim = 128;
    auto items = [](int n) { return align256(n * sizeof(ItemDesc)); };
    const size_t full = attn_blob(build_attn_schedule(&w)).bytes.size() - items(2);
    const size_t least = align256((size_t)16 * c.hq * ((c.L + 255) / 256 + 1)) +
                         align256((size_t)16 * c.hkv * ((c.L + 127) / 128 + 1)) + 2 * 256;
    CHECK(least < full);
    int lo = most, hi = most;                           // the first list whose full schedule is too long, the last that fits
    while (items(lo - 1) + full > nsp::kScratchSchedBytes) --lo;
    while (items(hi) + least > nsp::kScratchSchedBytes) --hi;
    CHECK(lo <= hi);
    for (int n : {lo - 1, lo, hi}) {
      w.n_items = n;
      HostSchedPtr h, m;
      w.item_mask = nullptr;
      CHECK(get_host_schedule(worklist_key("attn", 0, &w, 0), &w, &h) == NSP_OK);
      w.item_mask = second.data();
      CHECK(get_host_schedule(worklist_key("attn", 0, &w, 0), &w, &m) == NSP_OK);
      for (const HostSched *x : {h.get(), m.get()}) {
        check_passes(x->hs);
        CHECK(x->blob.bytes.size() <= nsp::kScratchSchedBytes);
        CHECK(x->hs.small == (n < lo && c.small) && (n < lo || x->hs.dq.kind == nsp::kQWhole));
      }
    }
  }
  std::vector<int32_t> cu(1, 0), heads;
  for (int j = 0; j < 80000; ++j) {
    cu.push_back(cu.back() + 129);
    heads.push_back(0);
    heads.push_back(1);
  }
  nsp_worklist w{};
  w.n_items = 80000;
  w.cu_seqlens = cu.data();
  w.q_heads = w.kv_heads = heads.data();
  w.hq_total = w.hkv_total = 1;
  w.head_dim = 64;
  HostSchedPtr h;
  CHECK(get_host_schedule(worklist_key("attn", 0, &w, 0), &w, &h) == NSP_OK);
  CHECK(attn_blob(build_attn_schedule(&w)).bytes.size() > nsp::kScratchSchedBytes);
  CHECK(h->blob.bytes.size() <= nsp::kScratchSchedBytes);
}

}  // namespace

int main(int argc, char **argv) {
  check_compact();
  check_tested_lists();
  check_long_units();
  if (argc > 1) check_balance(argv[1]);
  int n_split = 0, kinds[3] = {0, 0, 0};
  for (int rep = 0; rep < 400; ++rep) {
    static const int heads[][2] = {{32, 4}, {8, 2}, {16, 16}, {4, 1}, {12, 6}};
    const int *h = heads[uni(0, 4)];
    const int n = uni(1, 6), top = 1 << uni(6, 14);
    std::vector<int32_t> cu(1, 0), qh, kvh;
    std::vector<uint8_t> mask;
    for (int j = 0; j < n; ++j) {
      cu.push_back(cu.back() + (uni(0, 6) ? uni(1, top) : 0));
      const int group = h[0] / h[1];
      const int q0 = uni(0, h[0] - 1), q1 = uni(q0 + 1, h[0]);
      qh.push_back(q0);
      qh.push_back(q1);
      kvh.push_back(uni(0, q0 / group));               // KV heads without query heads among them
      kvh.push_back(uni((q1 - 1) / group + 1, h[1]));
      mask.push_back(uni(0, 1));
    }
    nsp_worklist w{};
    w.n_items = n;
    w.cu_seqlens = cu.data();
    w.q_heads = qh.data();
    w.kv_heads = kvh.data();
    w.hq_total = h[0];
    w.hkv_total = h[1];
    w.head_dim = uni(0, 1) ? 128 : 64;
    check_list(w, mask, &n_split);
    check_gangs(w, kinds);
    w.item_mask = mask.data();
    check_gangs(w, kinds);
  }
  CHECK(n_split > 100 && n_split < 400 && kinds[0] > 50 && kinds[1] > 50 && kinds[2] > 50);
  std::printf("split checks ok (%d of 400 lists split)\n", n_split);
  return 0;
}
