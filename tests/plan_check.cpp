// Runs the host side of the forwards, the fold and vp_ce_backward on the CPU with the kernels
// replaced by recorders, on random problems, and checks what it would have launched.
// Backward: that the residual tiles cover every (vocabulary row, token) once, that the dW and
// dH contractions read each of them once, after it was written and before its buffer is
// written again, that partial sums start from beta = 0 and are all added up, and that every
// buffer lies inside the workspace.  Forwards: that the tiles cover every shard, that the
// partial states lie inside the workspace, for every workspace size that is accepted, and
// that the merge reads as many of them as were written.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <random>
#include <set>

#include "../paper_2609_14306_amd/csrc/vpce_api.cpp"

static std::vector<vpce::StageArgs> launches;
static std::vector<vpce::TransposeArgs> copies;
static std::vector<size_t> copies_before;  // copies made before launch k
static int last_cls, summed;
static std::vector<vpce::FwdArgs> fwds;
static std::vector<vpce::CombArgs> combs;
static std::vector<vpce::FoldArgs> folds;
static char* const kScratch = (char*)(9ll << 44);

// (the tiles' sizes and times are the built library's, which this program is linked with)
namespace vpce {
bool scratch_base(void** p) {
  *p = kScratch;
  return true;
}
bool run_ws_init(unsigned long long*, hipStream_t) { return true; }
bool run_fill_zero(float*, int64_t, hipStream_t) { return true; }
bool run_fwd(int, const FwdArgs& a, hipStream_t) {
  fwds.push_back(a);
  return true;
}
bool run_comb(const CombArgs& a, hipStream_t) {
  combs.push_back(a);
  return true;
}
bool run_state_init(float*, int64_t, hipStream_t) { return true; }
bool run_fold_merge(const FoldArgs& a, hipStream_t) {
  folds.push_back(a);
  return true;
}
bool run_fold_finalize(const FinArgs&, hipStream_t) { return true; }
bool run_count_bad(const int64_t*, int64_t, int64_t, int64_t, unsigned long long*, hipStream_t) { return true; }
bool run_target_logits(int, const TgtArgs&, hipStream_t) { return true; }
bool run_transpose(int, const TransposeArgs& a, hipStream_t) {
  copies.push_back(a);
  return true;
}
bool run_stage(int, int cls, const StageArgs& a, hipStream_t) {
  last_cls = cls;
  launches.push_back(a);
  copies_before.push_back(copies.size());
  return true;
}
bool run_sum_parts(const float*, int n, int64_t, float*, hipStream_t) {
  summed = n;
  return true;
}
}  // namespace vpce

#define CHECK(...)                                                     \
  do {                                                                \
    if (!(__VA_ARGS__)) {                                                       \
      printf("FAILED line %d: %s\n", __LINE__, #__VA_ARGS__);                   \
      return false;                                                   \
    }                                                                 \
  } while (0)

static bool check(const vp_problem& p, int64_t accumulate) {
  launches.clear();
  copies.clear();
  copies_before.clear();
  summed = 1;
  const int64_t T = p.T, d = p.d, eb = p.dtype == VP_BF16 ? 2 : 4, KB = 128 / eb;
  size_t bytes = 0;
  CHECK(vp_ce_workspace_size(&p, nullptr, &bytes) == VP_OK);
  // made-up addresses, far apart; nothing reads them
  char* ws = (char*)(1ll << 44);
  const char* H = (const char*)(2ll << 44);
  float* dH = (float*)(3ll << 44);
  std::vector<const void*> W(p.P);
  std::vector<float*> dW(p.P);
  for (int q = 0; q < p.P; ++q) {
    W[q] = (const void*)((4ll << 44) + ((int64_t)q << 38));
    dW[q] = (float*)((5ll << 44) + ((int64_t)q << 38));
  }
  vp_problem pr = p;
  pr.flags = accumulate ? VP_ACCUMULATE_DW : 0;
  CHECK(vp_ce_backward(&pr, H, W.data(), (const int64_t*)64, (const float*)64, (const float*)64, dH, dW.data(), ws,
                       bytes, nullptr) == VP_OK);
  vp_plan_info info;
  CHECK(vp_ce_plan_info(&pr, &info) == VP_OK);
  CHECK((int64_t)launches.size() == info.stage_launches && info.strips + 1 == info.stage_launches);
  const vpce::BwdTile ft = vpce::bwd_tile(p.dtype, last_cls);
  CHECK(last_cls != 0 || p.dtype == VP_BF16);
  auto inside = [&](const void* a, int64_t n) {
    const char* c = (const char*)a;
    return c >= ws + kHeaderBytes && n >= 0 && c + n <= ws + bytes;
  };
  // per shard: rows still to be written (residual) and contracted, per token chunk
  std::map<std::pair<int, int64_t>, int64_t> written, dw_done, dh_done;  // (shard, t0) -> rows in order
  std::set<std::pair<int64_t, int64_t>> dh_started;                      // (slot, t0)
  std::set<std::pair<int, int64_t>> dw_started;                          // (shard, first row)
  int most_jobs = 1;
  auto shard_of = [&](const vpce::StageSeg& s, int64_t* row) {
    const int q = (int)(((int64_t)(uintptr_t)s.w - (4ll << 44)) >> 38);
    *row = ((int64_t)(uintptr_t)s.w - (4ll << 44) - ((int64_t)q << 38)) / (d * eb);
    return q;
  };
  for (size_t k = 0; k < launches.size(); ++k) {
    const vpce::StageArgs& a = launches[k];
    const int64_t Tc = a.g.Tc, Vr = a.g.Vc, strip = Tc * Vr * eb;
    CHECK(p.dtype != VP_BF16 || Tc <= strip_plan(&p).Tc);  // one chain per dW tile
    CHECK(Tc % ft.bn == 0 && Vr % ft.bm == 0 && a.g.d == d && Tc * Vr < (1ll << 31));
    CHECK(a.g.yt && inside(a.g.yt, T * 4));
    if (a.n_gseg) {
      CHECK(a.n_gseg <= vpce::kMaxSegs && a.g.N > 0 && a.g.N <= Tc && a.g.t0 + a.g.N <= T);
      CHECK(inside(a.g.strip, strip) && inside(a.g.strip_t, strip));
      int64_t row0 = 0;
      for (int i = 0; i < a.n_gseg; ++i) {
        const vpce::StageSeg& s = a.gseg[i];
        int64_t row;
        const int q = shard_of(s, &row);
        CHECK(s.rows > 0 && s.row0 == row0 && row + s.rows <= p.shard_rows[q]);
        int64_t off = 0;
        for (int x = 0; x < q; ++x) off += p.shard_rows[x];
        CHECK(s.gid0 == off + row && s.dw == dW[q] + row * d);
        int64_t& w = written[{q, a.g.t0}];
        CHECK(w == row);
        w += s.rows;
        row0 += round_up(s.rows, ft.bm);
      }
      CHECK(row0 <= Vr && a.g.n_vt * (int64_t)ft.bm == row0);
    }
    if (!a.n_cseg) continue;
    CHECK(k > 0);
    const vpce::StageArgs& b = launches[k - 1];  // wrote the strip
    CHECK(a.n_cseg == b.n_gseg && memcmp(a.cseg, b.gseg, a.n_cseg * sizeof(a.cseg[0])) == 0);
    CHECK(a.c_t0 == b.g.t0 && a.c_N == b.g.N && a.G == b.g.strip && a.Gt == b.g.strip_t);
    if (a.n_gseg) {  // the strip written now lies elsewhere
      for (const void* x : {a.G, a.Gt})
        for (const void* y : {(const void*)a.g.strip, (const void*)a.g.strip_t})
          CHECK(llabs((const char*)x - (const char*)y) >= strip);
    }
    CHECK(a.w_tiles * (int64_t)ft.bn >= a.g.n_vt * 0 + a.cseg[a.n_cseg - 1].row0 + a.cseg[a.n_cseg - 1].rows);
    for (int i = 0; i < a.n_cseg; ++i) {
      int64_t row;
      const int q = shard_of(a.cseg[i], &row);
      const bool first = dw_started.insert({q, row}).second;
      CHECK(a.beta_w == (accumulate || !first ? 1 : 0) || a.c_N == 0);
      dw_done[{q, a.c_t0}] += a.cseg[i].rows;
    }
    // dH jobs: the segments' rows, in order, once
    CHECK(a.n_job >= 1 && a.n_job <= vpce::kMaxJobs);
    most_jobs = std::max(most_jobs, a.n_job);
    int seg = 0;
    int64_t at = 0;
    for (int j = 0; j < a.n_job; ++j) {
      const vpce::StageJob& jb = a.job[j];
      CHECK(jb.seg == seg && jb.n_seg >= 1 && jb.seg + jb.n_seg <= a.n_cseg);
      if (jb.n_seg > 1) {
        CHECK(at == 0);
        seg += jb.n_seg;
      } else {
        CHECK(jb.k0 == at && jb.k0 % KB == 0 && jb.rows > 0);
        at += jb.rows;
        CHECK(at <= a.cseg[seg].rows);
        if (at == a.cseg[seg].rows) {
          ++seg;
          at = 0;
        }
      }
      const bool fresh = dh_started.insert({j, a.c_t0}).second;
      CHECK(jb.beta == (fresh ? 0 : 1));
    }
    CHECK(seg == a.n_cseg && at == 0);
    for (int i = 0; i < a.n_cseg; ++i) {
      int64_t row;
      dh_done[{shard_of(a.cseg[i], &row), a.c_t0}] += a.cseg[i].rows;
    }
    if (last_cls == 3) {
      CHECK(inside(a.Ht, d * round_up(T, 256) * eb) && inside(a.Wt, d * Vr * eb));
      CHECK(copies[0].in == (const void*)H && copies[0].out == a.Ht && copies[0].R == T);
      if (a.c_t0 == 0) {  // its W copied just before this launch
        CHECK(copies_before[k] - copies_before[k - 1] == (size_t)a.n_cseg);
        for (int i = 0; i < a.n_cseg; ++i) {
          const vpce::TransposeArgs& c = copies[copies_before[k - 1] + i];
          CHECK(c.in == a.cseg[i].w && c.R == a.cseg[i].rows && c.R_pad == round_up(c.R, KB));
          CHECK((char*)c.out == (char*)a.Wt + a.cseg[i].row0 * d * eb);
        }
      }
    } else {
      CHECK(copies.empty());
    }
  }
  for (auto* m : {&written, &dw_done, &dh_done})
    for (int q = 0; q < p.P; ++q)
      for (int64_t t0 = 0; t0 < T; t0 += info.Tc) CHECK(((*m)[std::make_pair(q, t0)] == p.shard_rows[q] || p.shard_rows[q] == 0));
  CHECK(summed == most_jobs);
  for (const vpce::StageArgs& a : launches) {
    if (!a.n_cseg) continue;
    if (most_jobs == 1) {
      CHECK(a.part == dH);
    } else {
      CHECK(a.part_stride == T * d && inside(a.part, most_jobs * T * d * 4));
      const int64_t strip = a.g.Tc * a.g.Vc * eb;
      for (const void* x : {a.G, a.Gt}) CHECK((const char*)a.part >= (const char*)x + strip);
      CHECK((const char*)a.g.yt >= (const char*)a.part + most_jobs * T * d * 4);
    }
  }
  return true;
}

// What a forward launched: every token block meets every tile of every shard, in as many
// splits as the merge reads, and the partial states lie side by side inside the workspace.
// y: the target logits' place where it is not the workspace.
static bool check_fwd_args(const vp_problem& p, const vpce::FwdArgs& a, const char* ws, int64_t bytes, const float* y) {
  const vpce::FwdTile t = vpce::fwd_tile(p.dtype, a.kind);
  CHECK(a.kind >= 0 && a.kind < vpce::kFwdKinds && a.T == p.T && a.d == p.d);
  CHECK(a.n_tok_blocks == ceil_div(p.T, t.bn));
  CHECK(a.n_splits >= 1 && (a.kind == 0 || a.n_splits <= a.n_tiles));
  CHECK((int64_t)a.n_tok_blocks * a.n_splits < (1ll << 31) / 512);  // threads of the grid
  int64_t tiles = 0;
  for (int i = 0; i < a.st.P; ++i) {
    CHECK(a.st.tile0[i] == tiles);
    tiles += ceil_div(a.st.rows[i], t.bm);
  }
  CHECK(tiles == a.n_tiles && a.st.tile0[a.st.P] == tiles);
  const int64_t part = (int64_t)a.n_splits * p.T * 4;
  const char *m = (const char*)a.m_part, *s = (const char*)a.s_part, *e = (const char*)(y ? y : a.y_tgt);
  CHECK(m >= ws + kHeaderBytes && s >= m + part && s + part <= ws + bytes);
  CHECK(a.y_tgt == (const float*)e && (y || (e >= s + part && e + p.T * 4 <= ws + bytes)));
  return true;
}

static bool check_forward(const vp_problem& p) {
  fwds.clear();
  combs.clear();
  folds.clear();
  size_t bytes = 0;
  CHECK(vp_ce_workspace_size(&p, &bytes, nullptr) == VP_OK);
  char* ws = (char*)(1ll << 44);
  const char* H = (const char*)(2ll << 44);
  float *loss = (float*)(6ll << 44), *lse = (float*)(7ll << 44), *state = (float*)(8ll << 44);
  const int64_t* targets = (const int64_t*)64;
  std::vector<const void*> W(p.P);
  for (int q = 0; q < p.P; ++q) W[q] = (const void*)((4ll << 44) + ((int64_t)q << 38));
  // the least that was ever asked for: at most 32 splits, and one byte less is refused
  const size_t least = fwd_ws_min(&p);
  CHECK(least <= bytes && least <= kHeaderBytes + 2 * align256(32 * p.T * 4) + align256(p.T * 4));
  CHECK(vp_ce_forward(&p, H, W.data(), targets, loss, lse, ws, least - 1, nullptr) == VP_ERR_WORKSPACE && fwds.empty());
  for (size_t n : {least, (least + bytes) / 2, bytes, bytes + (1 << 20)}) {
    CHECK(vp_ce_forward(&p, H, W.data(), targets, loss, lse, ws, n, nullptr) == VP_OK);
    const vpce::FwdArgs& a = fwds.back();
    const vpce::CombArgs& c = combs.back();
    CHECK(check_fwd_args(p, a, ws, (int64_t)n, nullptr));
    CHECK(a.counter == (unsigned long long*)ws && c.bad_counter == a.counter);
    CHECK(c.m_part == a.m_part && c.s_part == a.s_part && c.y_tgt == a.y_tgt && c.n_splits == a.n_splits && c.T == p.T);
    if (n > bytes) CHECK(a.n_splits == fwds[fwds.size() - 2].n_splits);  // more room changes nothing
  }
  const vp_status st = vp_ce_forward_noalloc(&p, H, W.data(), targets, loss, lse, nullptr);
  CHECK(st == (least > vpce::kScratchBytes ? VP_ERR_WORKSPACE : VP_OK));
  if (st == VP_OK) CHECK(check_fwd_args(p, fwds.back(), kScratch, vpce::kScratchBytes, nullptr));
  int64_t off = 0;
  for (int q = 0; q < p.P; off += p.shard_rows[q++]) {
    vp_problem one = p;
    int64_t rows = p.shard_rows[q];
    one.P = 1;
    one.shard_rows = &rows;
    one.order = nullptr;
    CHECK(fwd_ws_min(&one) == least);
    for (size_t n : {least, bytes}) {
      const size_t before = fwds.size();
      CHECK(vp_ce_fold_shard(&one, off, H, W[q], targets, state, ws, n, nullptr) == VP_OK);
      CHECK(fwds.size() == before + (rows > 0) && folds.size() <= fwds.size());
      if (rows == 0) continue;
      const vpce::FwdArgs& a = fwds.back();
      const vpce::FoldArgs& f = folds.back();
      CHECK(check_fwd_args(one, a, ws, (int64_t)n, state + 2 * p.T));
      CHECK(!a.counter && a.st.off[0] == off && a.n_splits <= a.n_tiles);
      CHECK(f.m_part == a.m_part && f.s_part == a.s_part && f.n_splits == a.n_splits && f.T == p.T && f.state == state);
    }
  }
  return true;
}

// plan DTYPE T D STRIP ROWS...: the tiles that a problem runs on
static int print_plan(int argc, char** argv) {
  vp_problem p;
  memset(&p, 0, sizeof(p));
  p.dtype = atoi(argv[0]);
  p.T = atoll(argv[1]);
  p.d = atoll(argv[2]);
  p.strip_elems = atoll(argv[3]);
  std::vector<int64_t> rows;
  for (int i = 4; i < argc; ++i) rows.push_back(atoll(argv[i]));
  p.P = (int)rows.size();
  p.shard_rows = rows.data();
  if (validate(&p, nullptr) != VP_OK) return 1;
  BwdPlan f = plan_bwd(&p);
  cut_strips(&p, &f);
  size_t most = 0;
  for (const BwdStrip& st : f.strips) most = std::max(most, st.segs.size());
  const FwdPlan w = plan_fwd(&p, partial_slots(&p));
  printf("class %d Tc %lld Vc %lld strips %d segs %d jobs %d kind %d splits %d", f.cls, (long long)f.Tc, (long long)f.Vc,
         (int)f.strips.size(), (int)most, f.max_jobs, w.kind, w.splits);
  for (int64_t r : rows) {  // each shard folded by itself
    vp_problem one = p;
    one.P = 1;
    one.shard_rows = &r;
    printf(" fold %d", r > 0 ? plan_fwd(&one, partial_slots(&one)).kind : -1);
  }
  printf("\n");
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 6 && !strcmp(argv[1], "plan")) return print_plan(argc - 2, argv + 2);
  std::mt19937_64 r(argc > 1 ? atoi(argv[1]) : 1);
  auto log_int = [&](double lo, double hi) {
    return (int64_t)exp(std::uniform_real_distribution<double>(log(lo), log(hi))(r));
  };
  int classes[4] = {0, 0, 0, 0}, kinds[vpce::kFwdKinds] = {0}, jobs = 0, joined = 0, fewer = 0;
  for (int n = 0; n < 600; ++n) {
    vp_problem p;
    memset(&p, 0, sizeof(p));
    p.T = log_int(1, n % 50 == 0 ? 4e6 : 100000);
    p.d = std::max<int64_t>(8, log_int(8, n % 50 == 1 ? 100000 : 8192) / 8 * 8);
    p.P = 1 + (int)(r() % (n % 10 == 0 ? 64 : 9));
    p.dtype = (int)(r() % 2);
    p.strip_elems = r() % 3 ? 0 : log_int(n % 25 == 2 ? 1 : 1 << 18, 1 << 28);
    const bool large = n % 20 == 3;
    if (large) {
      p.T = log_int(20000, 60000);
      p.d = log_int(2048, 8192) / 8 * 8;
      p.strip_elems = 0;
    }
    std::vector<int64_t> rows(p.P);
    for (auto& x : rows) x = r() % 8 == 0 ? 0 : log_int(large ? 3000 : 1, 60000);
    rows[r() % p.P] = log_int(large ? 3000 : 1, 60000);
    std::vector<int32_t> order(p.P);
    for (int i = 0; i < p.P; ++i) order[i] = i;
    std::shuffle(order.begin(), order.end(), r);
    p.shard_rows = rows.data();
    p.order = order.data();
    p.ignore_index = -100;
    if (!check(p, r() % 2) || !check_forward(p)) {
      printf("T=%lld d=%lld P=%d dtype=%d strip=%lld class=%d rows:", (long long)p.T, (long long)p.d, p.P, p.dtype,
             (long long)p.strip_elems, last_cls);
      for (auto x : rows) printf(" %lld", (long long)x);
      printf("\n");
      return 1;
    }
    ++classes[last_cls];
    for (const auto& a : fwds) {
      ++kinds[a.kind];
      fewer += p.T > kFewTokens && a.st.P == p.P && a.n_splits < splits_for(&p);
    }
    for (const auto& a : launches) {
      jobs += a.n_job > 1;
      joined += a.n_cseg > 1;
    }
  }
  printf("classes %d %d %d %d, launches with several jobs %d, with joined shards %d; kinds %d %d %d, fewer splits %d\n",
         classes[0], classes[1], classes[2], classes[3], jobs, joined, kinds[0], kinds[1], kinds[2], fewer);
  return classes[0] && classes[1] && classes[2] && classes[3] && jobs && joined && kinds[0] && kinds[1] && kinds[2] && fewer
             ? 0
             : 1;
}
