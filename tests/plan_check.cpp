// Runs vp_ce_backward's host side on the CPU with the kernels replaced by recorders, on
// random problems, and checks what it would have launched: that the residual tiles cover
// every (vocabulary row, token) once, that the dW and dH contractions read each of them once,
// after it was written and before its buffer is written again, that partial sums start from
// beta = 0 and are all added up, and that every buffer lies inside the workspace.
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

namespace vpce {
TileShape tile_shape(int dtype) {
  return dtype == VP_BF16 ? TileShape{256, 256, 64} : TileShape{256, 256, 32};
}
FwdTile fwd_tile(int, int) { return FwdTile{256, 256, 1, 1.4, 1.8}; }
BwdTile bwd_tile(int dtype, int cls) {  // the sizes of the kernels' tiles; any times will do
  const bool b = dtype == VP_BF16;
  return cls == 1 ? BwdTile{128, 64, b ? 0.34 : 1.0} : cls == 2 ? BwdTile{128, 128, b ? 0.55 : 1.88}
                                                                  : BwdTile{256, 256, b ? 1.4 : 6.9};
}
int bwd_col_blocks(int cls, int d) {
  const int bm = cls == 1 || cls == 2 ? 128 : 256, rem = d % bm;
  return bm == 256 && d >= 256 && rem > 0 && rem <= 64 ? d / bm : (d + bm - 1) / bm;
}
bool scratch_base(void**) { return false; }
bool run_ws_init(unsigned long long*, hipStream_t) { return true; }
bool run_fill_zero(float*, int64_t, hipStream_t) { return true; }
bool run_fwd(int, const FwdArgs&, hipStream_t) { return true; }
bool run_comb(const CombArgs&, hipStream_t) { return true; }
bool run_state_init(float*, int64_t, hipStream_t) { return true; }
bool run_fold_merge(const FoldArgs&, hipStream_t) { return true; }
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

int main(int argc, char** argv) {
  std::mt19937_64 r(argc > 1 ? atoi(argv[1]) : 1);
  auto log_int = [&](double lo, double hi) {
    return (int64_t)exp(std::uniform_real_distribution<double>(log(lo), log(hi))(r));
  };
  int classes[4] = {0, 0, 0, 0}, jobs = 0, joined = 0;
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
    if (!check(p, r() % 2)) {
      printf("T=%lld d=%lld P=%d dtype=%d strip=%lld class=%d rows:", (long long)p.T, (long long)p.d, p.P, p.dtype,
             (long long)p.strip_elems, last_cls);
      for (auto x : rows) printf(" %lld", (long long)x);
      printf("\n");
      return 1;
    }
    ++classes[last_cls];
    for (const auto& a : launches) {
      jobs += a.n_job > 1;
      joined += a.n_cseg > 1;
    }
  }
  printf("classes %d %d %d %d, launches with several jobs %d, with joined shards %d\n", classes[0], classes[1],
         classes[2], classes[3], jobs, joined);
  return classes[0] && classes[1] && classes[2] && classes[3] && jobs && joined ? 0 : 1;
}
