// Host side of the C ABI declared in include/vpce.h: argument validation,
// workspace planning and launch sequencing.  Every argument, shape, alignment
// and workspace error is detected here before any HIP call is made, so these
// paths run (and are tested) on a machine without a GPU.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "vpce_internal.h"

namespace {

constexpr size_t kHeaderBytes = 256;       // error counter + reserved
constexpr int64_t kDefaultStrip = 100ll << 20;  // residual-strip budget in elements per layout
constexpr int64_t kCUs = 256;                      // compute units of one MI355X
constexpr int64_t kPanelCacheBudget = 160ll << 20;  // of the 256 MiB memory-side cache
constexpr int kMaxSplits = 32;

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
inline int64_t round_down(int64_t x, int64_t m) { return x / m * m; }
inline int64_t ceil_div(int64_t x, int64_t m) { return (x + m - 1) / m; }

size_t elem_bytes(int dtype) { return dtype == VP_BF16 ? 2 : 4; }

constexpr int64_t kMaxT = (1ll << 23) - 256;
constexpr int64_t kMaxD = 1ll << 22;

vp_status validate(const vp_problem* p, int64_t* V_out, bool allow_empty_vocab = false) {
  if (!p) return VP_ERR_NULL;
  if (p->dtype != VP_F32 && p->dtype != VP_BF16) return VP_ERR_DTYPE;
  // The bf16 GEMM tiles address a 256-row operand tile with 32-bit byte offsets
  // (256 rows x leading dimension x 2 bytes < 2^32): leading dimensions are d,
  // the padded token count and strip widths, so T and d are capped below 2^23.
  if (p->T < 0 || p->d < 8 || p->d % 8 != 0 || p->d > kMaxD) return VP_ERR_SHAPE;
  if (p->T > kMaxT) return VP_ERR_SHAPE;
  if (p->P < 1 || p->P > VP_MAX_SHARDS) return VP_ERR_SHAPE;
  if (!p->shard_rows) return VP_ERR_NULL;
  if (p->strip_elems < 0 || p->strip_elems > (1ll << 30)) return VP_ERR_SHAPE;
  int64_t V = 0;
  for (int i = 0; i < p->P; ++i) {
    if (p->shard_rows[i] < 0 || p->shard_rows[i] > (1ll << 30)) return VP_ERR_SHAPE;
    V += p->shard_rows[i];
  }
  if (V < (allow_empty_vocab ? 0 : 1) || V > (1ll << 31) - 1) return VP_ERR_SHAPE;
  if (p->order) {
    bool seen[VP_MAX_SHARDS] = {false};
    for (int i = 0; i < p->P; ++i) {
      const int q = p->order[i];
      if (q < 0 || q >= p->P || seen[q]) return VP_ERR_ORDER;
      seen[q] = true;
    }
  }
  if (V_out) *V_out = V;
  return VP_OK;
}

inline bool misaligned(const void* ptr) { return ((uintptr_t)ptr & 15u) != 0; }

// Vocabulary splits of the forward on 256 x 256 tiles: workgroup (token block, split)
// folds one token block over one contiguous range of the vocabulary tiles, and an XCD
// runs 32 consecutive workgroups at a time, i.e. 32 / S token blocks by S splits.  S
// is the smallest power of two (at most 32) that
// - fills the CUs (token blocks x S >= 256);
// - is at least 4, so that those 32 tiles share 12 operand panels in the XCD's L2
//   (8 x 4 or 4 x 8);
// - keeps the H panels of the 256 / S token blocks running at once within 160 MiB,
//   so that they stay in the memory-side cache while every vocabulary tile re-reads
//   them.
int splits_for(const vp_problem* p) {
  const vpce::TileShape ts = vpce::tile_shape(p->dtype);
  const int64_t tok_blocks = std::max<int64_t>(1, ceil_div(p->T, ts.bn));
  const int64_t panel = (int64_t)ts.bn * p->d * (int64_t)elem_bytes(p->dtype);
  const int64_t need = std::max<int64_t>(
      4, std::max(ceil_div(kCUs, tok_blocks), ceil_div(kCUs * panel, kPanelCacheBudget)));
  int s = 4;
  while (s < need && s < kMaxSplits) s *= 2;
  return s;
}

// Few tokens: at most kFewTokens = 256 CUs / 32 splits x 256 tokens, where 32 splits
// no longer give every CU a workgroup.  There the forward may take more splits and
// smaller tiles (plan_fwd); the partial states it may write per call (splits x T) are
// at least what 32 splits need, and otherwise the 64 Ki that 32 splits take at
// kFewTokens, but no more than a quarter of the bytes of H itself (8 bytes each) or
// 8 Ki, whichever is larger.  Up to kFewTokens the count never falls as T grows; above, it
// falls where splits_for halves (122880 states at T = 3840, d = 256, and 61456 at 3841).
constexpr int64_t kFewTokens = 2048;
int64_t partial_slots(const vp_problem* p) {
  const int64_t T = p->T, base = (int64_t)splits_for(p) * T;
  if (T == 0 || T > kFewTokens) return base;
  const int64_t quarter = T * p->d * (int64_t)elem_bytes(p->dtype) / 32;
  return std::max(base, std::min<int64_t>(32 * kFewTokens, std::max<int64_t>(8192, quarter)));
}
size_t fwd_bytes(int64_t slots, int64_t T) {
  return kHeaderBytes + 2 * align256((size_t)slots * 4) + align256((size_t)T * 4);
}

size_t fwd_ws_bytes(const vp_problem* p) { return fwd_bytes(partial_slots(p), p->T); }
// What the forward needs at least: the partial states of splits_for() splits.
size_t fwd_ws_min(const vp_problem* p) {
  return fwd_bytes((int64_t)splits_for(p) * p->T, p->T);
}

// Vocabulary tiles of `bm` rows over all shards.
int64_t count_tiles(const vp_problem* p, int bm) {
  int64_t n = 0;
  for (int q = 0; q < p->P; ++q) n += ceil_div(p->shard_rows[q], bm);
  return n;
}

// Tile kind and splits of a forward over the problem's shards with room for `slots`
// partial states.  Above kFewTokens tokens the 256 x 256 tile with at most splits_for()
// splits.
// Below, the kind whose launch is estimated shortest: every workgroup runs
// ceil(tiles / splits) tiles one after the other, the launch takes ceil(workgroups /
// places on the chip) such turns, and a tile takes d / slice depth times the measured
// time per slice of its kind (the same d for every kind, so it is left out).  Measured
// both ways (microseconds, kinds 0 / 1 / 2): d = 4096, V = 151936 in 16 shards, bf16:
// T = 40: 310 / 258 / 245, T = 100: 308 / 267 / 348, T = 256: 333 / 425 / 608, T = 1024:
// 1071 / 1470 / 2261; d = 1000, V = 32003 in 5: T = 40: 36 / 31 / 27, T = 300: 87 / 70 /
// 54; float32 d = 2880, V = 50000 in 4: T = 64: 668 / 399 / 248, T = 1024: 2612 / 2686 /
// 2900.  With at most 32 splits of 256 x 256 tiles the first of these took 1550.
struct FwdPlan {
  int kind, splits;
};
FwdPlan plan_fwd(const vp_problem* p, int64_t slots) {
  FwdPlan best{0, splits_for(p)};
  if (p->T > kFewTokens) {
    // Whole tiles on the 256 x 256 tile again: where splits_for's workgroups leave a last
    // round mostly empty, fewer splits are taken if they save more than 3% of the turns
    // (below the four that share panels, more than a fifth).  d = 2880, V = 201088, bf16:
    // T = 2304, 28 splits instead of 32: 3.60 -> 2.33 ms; T = 9000, 7 instead of 8: 13.5 ->
    // 8.0 ms; T = 12000, 5 instead of 8: 12.9 -> 10.9 ms.  The turns also outweigh the cache
    // budget of splits_for: at wide d fewer splits mean more H panels at once, and are still
    // the fastest (ms, panels in MiB): bf16 T = 38494, d = 6912, V = 142765, 8 splits 64.8
    // (108), 6 70.9 (145), 5 63.9 (176); bf16 T = 58208, d = 7104, V = 11195, 8 splits 8.1
    // (111), 4 7.9 (222); f32 T = 25549, d = 5696, V = 25891, 16 splits 63.6 (89), 5 59.1 (289).
    const vpce::FwdTile t = vpce::fwd_tile(p->dtype, 0);
    const int64_t blocks = ceil_div(p->T, t.bn), tiles = std::max<int64_t>(1, count_tiles(p, t.bm));
    auto turns = [&](int64_t S) { return ceil_div(tiles, S) * ceil_div(blocks * S, kCUs); };
    const int64_t base = turns(best.splits);
    int64_t least = base * 97 / 100;
    for (int S = best.splits - 1; S >= 2; --S) {
      if (S == 3) least = std::min(least, base * 80 / 100);
      if (turns(S) < least) {
        best.splits = S;
        least = turns(S);
      }
    }
    return best;
  }
  double best_time = 0;
  for (int kind = 0; kind < vpce::kFwdKinds; ++kind) {
    const vpce::FwdTile t = vpce::fwd_tile(p->dtype, kind);
    const int64_t blocks = ceil_div(p->T, t.bn), places = kCUs * t.per_cu;
    const int64_t tiles = std::max<int64_t>(1, count_tiles(p, t.bm));
    int64_t S = std::max<int64_t>(1, std::min(std::min(slots / p->T, places / blocks), tiles));
    const int64_t turn = ceil_div(tiles, S);
    S = ceil_div(tiles, turn);  // the same turns with the fewest splits
    const double time = (double)(turn * ceil_div(blocks * S, places)) *
                        std::max(t.shared, blocks == 1 ? t.stream : 0.0);
    if (kind == 0 || time < best_time) {
      best = FwdPlan{kind, (int)S};
      best_time = time;
    }
  }
  return best;
}

// The backward's workspace.  The softmax residual of a strip of Tc tokens by Vc
// vocabulary rows is staged in both layouts (G [Vc][Tc] and G^T [Tc][Vc]),
// twice: one launch writes the residual of strip c+1 while it contracts strip
// c into dH and dW.  Tc*Vc <= budget; tokens in balanced chunks no larger than
// the square root of the budget (the float32 read-modify-write traffic of dH
// across vocabulary chunks plus that of dW across token chunks is proportional
// to 1/Vc + 1/Tc).  The workspace also holds H^T [d][T_pad] (written once per
// call) and W^T [d][Vc] of the current vocabulary chunk; a backward that reads W and H
// as they are uses that room for longer strips and partial sums of dH (plan_bwd).
// Nothing here depends on V.
struct StripPlan {
  int64_t Tc, Vc, T_pad;
  size_t total;
};

StripPlan strip_plan(const vp_problem* p) {
  const vpce::TileShape ts = vpce::tile_shape(p->dtype);
  const int64_t budget = p->strip_elems > 0 ? p->strip_elems : kDefaultStrip;
  const int64_t T = std::max<int64_t>(p->T, 1);
  const int64_t side = std::max<int64_t>(ts.bn, round_down((int64_t)std::sqrt((double)budget), ts.bn));
  StripPlan s;
  s.Tc = std::min<int64_t>(round_up(T, ts.bn), round_up(ceil_div(T, ceil_div(T, side)), ts.bn));
  s.Vc = std::max<int64_t>(ts.bm, std::min<int64_t>(round_down(budget / s.Tc, ts.bm),
                                                        32768));
  s.T_pad = round_up(T, 256);
  const size_t eb = elem_bytes(p->dtype);
  s.total = kHeaderBytes + 4 * align256((size_t)s.Vc * s.Tc * eb) + align256((size_t)p->d * s.T_pad * eb) +
            align256((size_t)p->d * s.Vc * eb) + align256((size_t)T * 4);
  return s;
}

size_t bwd_ws_bytes(const vp_problem* p) { return strip_plan(p).total; }

void build_table(const vp_problem* p, const void* const* W_shards, int bm, vpce::ShardTable* st,
                 int32_t* n_tiles) {
  int64_t off[VP_MAX_SHARDS];
  int64_t acc = 0;
  for (int q = 0; q < p->P; ++q) {
    off[q] = acc;
    acc += p->shard_rows[q];
  }
  st->P = p->P;
  int32_t tiles = 0;
  for (int i = 0; i < p->P; ++i) {
    const int q = p->order ? p->order[i] : i;
    st->w[i] = W_shards[q];
    st->off[i] = off[q];
    st->rows[i] = (int32_t)p->shard_rows[q];
    st->tile0[i] = tiles;
    tiles += (int32_t)ceil_div(p->shard_rows[q], bm);
  }
  for (int i = p->P; i <= VP_MAX_SHARDS; ++i) st->tile0[i] = tiles;
  for (int i = p->P; i < VP_MAX_SHARDS; ++i) {
    st->w[i] = nullptr;
    st->off[i] = acc;
    st->rows[i] = 0;
  }
  *n_tiles = tiles;
}

vp_status check_shards(const vp_problem* p, const void* const* W_shards) {
  if (!W_shards) return VP_ERR_NULL;
  for (int q = 0; q < p->P; ++q) {
    if (p->shard_rows[q] > 0 && !W_shards[q]) return VP_ERR_NULL;
    if (p->shard_rows[q] > 0 && misaligned(W_shards[q])) return VP_ERR_ALIGN;
  }
  return VP_OK;
}

// How a backward is cut: tile class, token chunks of Tc, vocabulary strips of at most Vc
// padded rows, dH partial sums.  Everything is laid out in the workspace that strip_plan
// asks for.
struct BwdStrip {  // vocabulary side of the strips; each meets every token chunk
  struct Seg {
    int q;
    int64_t v0, rows, row0;
  };
  std::vector<Seg> segs;
  std::vector<vpce::StageJob> jobs;
  int64_t rows_pad = 0;
};
struct BwdPlan {
  int cls = 0, slots = 1;
  int64_t Tc = 0, Vc = 0;  // Vc: most padded rows a strip may have
  double time = -1;
  // filled in by cut_strips
  std::vector<BwdStrip> strips;
  int64_t Vr = 0;  // padded rows of the longest strip
  int max_jobs = 1;
  size_t off_g[2], off_gt[2], off_part, off_ht, off_wt, off_yt;
};

// Walks the strips of a plan's vocabulary side in visiting order: a shard above Vc is cut
// into balanced pieces, a strip each; smaller shards share a strip while they fit.  A
// shard of less than 256 rows keeps a strip of its own (beside others it would be padding
// for the most part).  seg(new_strip, q, v0, rows, padded rows) for every segment.
template <class F>
void walk_strips(const vp_problem* p, int64_t Vc, int bm, F&& seg) {
  int64_t used = 0, last_rows = 0;
  int n_seg = 0;
  for (int i = 0; i < p->P; ++i) {
    const int q = p->order ? p->order[i] : i;
    const int64_t Vq = p->shard_rows[q], pad = round_up(Vq, bm);
    if (Vq == 0) continue;
    if (pad <= Vc) {
      const bool join = n_seg > 0 && n_seg < vpce::kMaxSegs && used + pad <= Vc && Vq >= 256 && last_rows >= 256;
      seg(!join, q, (int64_t)0, Vq, pad);
      n_seg = join ? n_seg + 1 : 1;
      used = join ? used + pad : pad;
      last_rows = Vq;
      continue;
    }
    const int64_t vc = round_up(ceil_div(Vq, ceil_div(Vq, Vc)), bm);
    for (int64_t v0 = 0; v0 < Vq; v0 += vc) {
      const int64_t rows = std::min(vc, Vq - v0);
      seg(true, q, v0, rows, round_up(rows, bm));
    }
    n_seg = 0;  // nothing joins a piece
  }
}

// Slices that a strip's dH sum has, and the most that one job should take: half of what
// its launch gives a CU to do, no less than eight, and as many as the slots ask for.
int64_t job_slices(int64_t ks, int64_t launch_work, int slots) {
  return std::max(std::max<int64_t>(8, launch_work / kCUs / 2), ceil_div(ks, slots));
}

// Estimated time (us) of a plan's launches.  A launch takes its slices (with two more per
// tile for its ends) spread over the CUs and half of its longest tile for the last round,
// or that tile alone; about 8 us of launch and fill; and 0.3 of the time its bytes take at
// 5 TB/s, the part that does not hide behind the rest.  Fitted to backwards of T = 40 to
// 2048 tokens, d = 256 to 4096, V = 2048 to 201088.  On 64 random problems (T = 40 to 65536,
// d = 256 to 7168, every class timed) the class it picks took 1.4% longer than the fastest
// one on average up to 2048 tokens (15% at worst) and 2.5% above (19%).
double plan_time(const vp_problem* p, const BwdPlan& f) {
  constexpr int64_t kEnds = 2;
  const vpce::BwdTile ft = vpce::bwd_tile(p->dtype, f.cls);
  const int64_t KB = vpce::tile_shape(p->dtype).kblock, kd = ceil_div(p->d, KB), d = p->d;
  const int64_t eb = (int64_t)elem_bytes(p->dtype), n_nb = vpce::bwd_col_blocks(f.cls, (int)d);
  const int64_t n_tc = ceil_div(p->T, f.Tc), N = std::min(f.Tc, p->T);
  const int64_t n_tb = ceil_div(N, ft.bn), kt = ceil_div(N, KB);
  auto launch = [&](int64_t work, int64_t longest, int64_t bytes) {
    const double mm = std::max((double)work / kCUs + 0.5 * longest, (double)longest);
    return ft.us * mm + 0.3 * (double)bytes / 5e6 + 8.0;
  };
  double total = 0;
  int64_t slices = 0, pads = 0;         // of the strip being walked
  int64_t c_work = 0, c_long = 0, c_bytes = 0;  // contractions left to the next launch
  auto close = [&]() {
    if (pads == 0) return;
    const int64_t res = pads / ft.bm * n_tb * (kd + kEnds);
    const int64_t dw = ceil_div(pads, ft.bn) * n_nb * (kt + kEnds);
    const int64_t per = std::min(slices, job_slices(slices, res + dw + n_tb * n_nb * slices, f.slots));
    const int64_t jobs = ceil_div(slices, per), dh = n_tb * n_nb * (slices + jobs * kEnds);
    const int64_t strip = 2 * pads * N * eb;
    total += launch(res + c_work, std::max(kd + kEnds, c_long), pads * d * eb + strip + c_bytes);
    c_work = dw + dh;
    c_long = std::max(per, kt) + kEnds;
    c_bytes = pads * d * (eb + 4) + strip + 2 * jobs * N * d * 4;
    total += (double)(n_tc - 1) * launch(res + c_work, std::max(kd + kEnds, c_long), pads * d * eb + strip + c_bytes);
    if (jobs > 1) total += (double)(jobs * p->T * d * 4) / 5e6;
  };
  walk_strips(p, f.Vc, ft.bm, [&](bool fresh, int, int64_t, int64_t rows, int64_t pad) {
    if (fresh) {
      close();
      slices = pads = 0;
    }
    slices += ceil_div(rows, KB);
    pads += pad;
  });
  close();
  total += launch(c_work, c_long, c_bytes);
  if (f.cls == 3) {  // the transposed copies, at 5 TB/s
    int64_t V = 0;
    for (int q = 0; q < p->P; ++q) V += p->shard_rows[q];
    total += 2.0 * (double)(V + p->T) * d * eb / 5e6;
  }
  return total;
}

// The plan with the shortest estimated time, of the tile classes, one or many dH partial
// sums, and two ways to cut the tokens: the strip plan's balanced chunks of at most the
// root of the budget, or, in float32, longer ones where the whole vocabulary is shorter than
// that.  bfloat16 dW tiles sum a token chunk in one chain (float32 ones in two levels), which
// longer chunks would make less exact: H of mean 8 and deviation 1, T = 10^6, d = 64, V = 64,
// dW off float64 by 1.8e-6 in chains of 10240 tokens and by 6.5e-6 in chains of 500032.
BwdPlan plan_bwd(const vp_problem* p) {
  const StripPlan s = strip_plan(p);
  const int64_t eb = (int64_t)elem_bytes(p->dtype);
  const int64_t budget = p->strip_elems > 0 ? p->strip_elems : kDefaultStrip;
  const int64_t avail = (int64_t)s.total - (int64_t)kHeaderBytes - (int64_t)align256((size_t)p->T * 4) - 5 * 256;
  const int64_t slot = p->T * p->d * 4;
  BwdPlan best;
  auto consider = [&](int cls, int slots, int64_t Tc, int64_t Vc) {
    BwdPlan f;
    f.cls = cls;
    f.slots = slots;
    f.Tc = Tc;
    f.Vc = Vc;
    f.time = plan_time(p, f);
    if (best.time < 0 || f.time < best.time) best = std::move(f);
  };
  consider(3, 1, s.Tc, s.Vc);
  for (int cls = p->dtype == VP_BF16 ? 0 : 1; cls < 3; ++cls) {
    const vpce::BwdTile ft = vpce::bwd_tile(p->dtype, cls);
    int64_t rows = 0;
    for (int q = 0; q < p->P; ++q) rows += round_up(p->shard_rows[q], ft.bm);
    int64_t tcs[2] = {std::min(s.Tc, round_up(p->T, ft.bn)), 0};
    const int64_t most = round_down(std::min(budget / rows, avail / (4 * eb * rows)), ft.bn);
    if (p->dtype == VP_F32 && most > tcs[0] && tcs[0] < p->T)
      tcs[1] = std::min(most, round_up(ceil_div(p->T, ceil_div(p->T, most)), ft.bn));
    for (int64_t Tc : tcs) {
      if (Tc <= 0) continue;
      for (int slots = 1; slots <= vpce::kMaxJobs; slots *= 2) {
        const int64_t room = avail - (slots > 1 ? slots * slot : 0);
        int64_t Vc = round_down(std::min(budget / Tc, room / (4 * Tc * eb)), ft.bm);
        if (Vc < ft.bm && slots == 1) Vc = ft.bm;  // strip_plan has room for it
        if (room <= 0 || Vc < ft.bm) break;
        consider(cls, slots, Tc, Vc);
      }
    }
  }
  return best;
}

// The strips, dH jobs and workspace layout of a plan.
void cut_strips(const vp_problem* p, BwdPlan* f) {
  const vpce::BwdTile ft = vpce::bwd_tile(p->dtype, f->cls);
  const int64_t KB = vpce::tile_shape(p->dtype).kblock, eb = (int64_t)elem_bytes(p->dtype);
  walk_strips(p, f->Vc, ft.bm, [&](bool fresh, int q, int64_t v0, int64_t rows, int64_t pad) {
    if (fresh) f->strips.emplace_back();
    BwdStrip& st = f->strips.back();
    st.segs.push_back({q, v0, rows, st.rows_pad});
    st.rows_pad += pad;
  });
  const int64_t N = std::min(f->Tc, p->T), n_tb = ceil_div(N, ft.bn);
  const int64_t n_nb = vpce::bwd_col_blocks(f->cls, (int)p->d);
  bool used[vpce::kMaxJobs] = {false};
  for (BwdStrip& st : f->strips) {
    f->Vr = std::max(f->Vr, st.rows_pad);
    int64_t ks = 0;
    for (const BwdStrip::Seg& sg : st.segs) ks += ceil_div(sg.rows, KB);
    const int64_t work = st.rows_pad / ft.bm * n_tb * ceil_div(p->d, KB) +
                         ceil_div(st.rows_pad, ft.bn) * n_nb * ceil_div(N, KB) + n_tb * n_nb * ks;
    int64_t per = job_slices(ks, work, f->slots);
    auto add = [&](int seg, int n_seg, int64_t k0, int64_t rows) {
      const size_t j = st.jobs.size();
      st.jobs.push_back({seg, n_seg, (int32_t)k0, (int32_t)rows, used[j] ? 1 : 0});
      used[j] = true;
    };
    // whole segments gather in a job up to `per` slices; a longer segment is cut
    for (;; per += ceil_div(per, 4)) {
      int n = 0;
      int64_t have = 0;
      for (const BwdStrip::Seg& sg : st.segs) {
        const int64_t b = ceil_div(sg.rows, KB);
        if (have > 0 && have + b <= per) {
          have += b;
          continue;
        }
        n += (int)ceil_div(b, per);
        have = b <= per ? b : per;  // nothing gathers behind a cut segment
      }
      if (n <= f->slots || f->slots == 1) break;
    }
    if (f->slots == 1) {
      add(0, (int)st.segs.size(), 0, st.segs.size() == 1 ? st.segs[0].rows : 0);
    } else {
      int64_t have = 0;
      for (size_t i = 0; i < st.segs.size(); ++i) {
        const int64_t b = ceil_div(st.segs[i].rows, KB);
        if (have > 0 && have + b <= per) {
          ++st.jobs.back().n_seg;
          have += b;
          continue;
        }
        const int64_t step = ceil_div(b, ceil_div(b, per));
        for (int64_t k = 0; k < b; k += step)
          add((int)i, 1, k * KB, std::min(st.segs[i].rows, (k + step) * KB) - k * KB);
        have = b <= per ? b : per;
      }
    }
    f->max_jobs = std::max(f->max_jobs, (int)st.jobs.size());
  }
  const size_t strip = align256((size_t)(f->Vr * f->Tc * eb));
  size_t off = kHeaderBytes;
  for (int b = 0; b < 2; ++b) {
    f->off_g[b] = off;
    f->off_gt[b] = off + strip;
    off += 2 * strip;
  }
  f->off_part = off;
  if (f->max_jobs > 1) off += align256((size_t)(f->max_jobs * p->T * p->d * 4));
  f->off_ht = f->off_wt = off;
  if (f->cls == 3) {
    f->off_wt = f->off_ht + align256((size_t)(p->d * round_up(p->T, 256) * eb));
    off = f->off_wt + align256((size_t)(p->d * f->Vr * eb));
  }
  f->off_yt = off;
}

}  // namespace

extern "C" {

int vp_abi_version(void) { return VPCE_ABI_VERSION; }

const char* vp_status_str(vp_status s) {
  switch (s) {
    case VP_OK: return "ok";
    case VP_ERR_NULL: return "a required pointer is NULL";
    case VP_ERR_SHAPE: return "invalid shape (T, d, P or shard rows)";
    case VP_ERR_DTYPE: return "unsupported dtype";
    case VP_ERR_ORDER: return "order is not a permutation of the shards";
    case VP_ERR_ALIGN: return "a device pointer is not 16-byte aligned";
    case VP_ERR_WORKSPACE: return "workspace missing or too small";
    case VP_ERR_TARGET: return "a target is outside [0, V) and not ignore_index";
    case VP_ERR_HIP: return "HIP runtime or kernel launch failure";
    case VP_ERR_UNSUPPORTED: return "unsupported request";
  }
  return "unknown status";
}

vp_status vp_ce_workspace_size(const vp_problem* prob, size_t* fwd_bytes, size_t* bwd_bytes) {
  const vp_status st = validate(prob, nullptr);
  if (st != VP_OK) return st;
  if (fwd_bytes) *fwd_bytes = fwd_ws_bytes(prob);
  if (bwd_bytes) *bwd_bytes = bwd_ws_bytes(prob);
  return VP_OK;
}

}  // extern "C"

namespace {

// Argument checks of the forward shared by vp_ce_forward and vp_ce_forward_noalloc
// (everything except the workspace).
vp_status check_forward(const vp_problem* prob, const void* H, const void* const* W_shards,
                        const int64_t* targets, float* loss, float* lse, int64_t* V) {
  vp_status st = validate(prob, V);
  if (st != VP_OK) return st;
  if ((st = check_shards(prob, W_shards)) != VP_OK) return st;
  if (prob->T > 0) {
    if (!H || !targets || !loss || !lse) return VP_ERR_NULL;
    if (misaligned(H)) return VP_ERR_ALIGN;
  }
  return VP_OK;
}

// Partial states a workspace of ws_bytes >= fwd_ws_min(p) is used for: a caller that
// sized it with vp_ce_workspace_size gets all of partial_slots, whatever it has beyond.
int64_t slots_in(const vp_problem* p, size_t ws_bytes) {
  return ws_bytes >= fwd_ws_bytes(p) ? partial_slots(p) : (int64_t)splits_for(p) * p->T;
}

// The forward on a checked problem, with a workspace of at least fwd_ws_min(prob) bytes.
vp_status forward_impl(const vp_problem* prob, int64_t V, const void* H,
                       const void* const* W_shards, const int64_t* targets, float* loss,
                       float* lse, void* ws, size_t ws_bytes, hipStream_t s) {
  const int64_t T = prob->T;
  unsigned long long* counter = (unsigned long long*)ws;
  if (T == 0) return vpce::run_ws_init(counter, s) ? VP_OK : VP_ERR_HIP;

  const FwdPlan plan = plan_fwd(prob, slots_in(prob, ws_bytes));
  const vpce::FwdTile ft = vpce::fwd_tile(prob->dtype, plan.kind);
  const int S = plan.splits;
  char* base = (char*)ws + kHeaderBytes;
  vpce::FwdArgs a;
  memset(&a, 0, sizeof(a));
  build_table(prob, W_shards, ft.bm, &a.st, &a.n_tiles);
  a.H = H;
  a.targets = targets;
  a.T = T;
  a.d = (int32_t)prob->d;
  a.n_tok_blocks = (int32_t)ceil_div(T, ft.bn);
  a.n_splits = S;
  a.kind = plan.kind;
  a.counter = counter;
  a.m_part = (float*)base;
  a.s_part = (float*)(base + align256((size_t)S * T * 4));
  a.y_tgt = (float*)(base + 2 * align256((size_t)S * T * 4));
  if (!vpce::run_fwd(prob->dtype, a, s)) return VP_ERR_HIP;

  vpce::CombArgs c;
  c.m_part = a.m_part;
  c.s_part = a.s_part;
  c.y_tgt = a.y_tgt;
  c.targets = targets;
  c.T = T;
  c.V = V;
  c.ignore_index = prob->ignore_index;
  c.n_splits = S;
  c.loss = loss;
  c.lse = lse;
  c.bad_counter = counter;
  if (!vpce::run_comb(c, s)) return VP_ERR_HIP;
  return VP_OK;
}

}  // namespace

extern "C" {

vp_status vp_ce_forward(const vp_problem* prob, const void* H, const void* const* W_shards,
                        const int64_t* targets, float* loss, float* lse, void* ws,
                        size_t ws_bytes, void* stream) {
  int64_t V = 0;
  vp_status st = validate(prob, &V);
  if (st != VP_OK) return st;
  if ((st = check_shards(prob, W_shards)) != VP_OK) return st;
  if (!ws) return VP_ERR_WORKSPACE;
  if (ws_bytes < fwd_ws_min(prob)) return VP_ERR_WORKSPACE;
  if (misaligned(ws)) return VP_ERR_ALIGN;
  if ((st = check_forward(prob, H, W_shards, targets, loss, lse, &V)) != VP_OK) return st;
  return forward_impl(prob, V, H, W_shards, targets, loss, lse, ws, ws_bytes,
                      (hipStream_t)stream);
}

vp_status vp_ce_forward_noalloc(const vp_problem* prob, const void* H,
                                const void* const* W_shards, const int64_t* targets,
                                float* loss, float* lse, void* stream) {
  int64_t V = 0;
  const vp_status st = check_forward(prob, H, W_shards, targets, loss, lse, &V);
  if (st != VP_OK) return st;
  if (fwd_ws_min(prob) > vpce::kScratchBytes) return VP_ERR_WORKSPACE;
  void* ws = nullptr;
  if (!vpce::scratch_base(&ws)) return VP_ERR_HIP;
  return forward_impl(prob, V, H, W_shards, targets, loss, lse, ws, vpce::kScratchBytes,
                      (hipStream_t)stream);
}

vp_status vp_ce_state_init(float* state, int64_t T, void* stream) {
  if (T < 0 || T > kMaxT) return VP_ERR_SHAPE;
  if (T == 0) return VP_OK;
  if (!state) return VP_ERR_NULL;
  if (((uintptr_t)state & 3u) != 0) return VP_ERR_ALIGN;
  return vpce::run_state_init(state, T, (hipStream_t)stream) ? VP_OK : VP_ERR_HIP;
}

vp_status vp_ce_fold_shard(const vp_problem* shard, int64_t id_offset, const void* H,
                           const void* W_shard, const int64_t* targets, float* state, void* ws,
                           size_t ws_bytes, void* stream) {
  int64_t Vq = 0;
  vp_status st = validate(shard, &Vq, /*allow_empty_vocab=*/true);
  if (st != VP_OK) return st;
  if (shard->P != 1) return VP_ERR_SHAPE;
  if (id_offset < 0 || id_offset > (1ll << 31) - 1 - Vq) return VP_ERR_SHAPE;
  const int64_t T = shard->T;
  // an empty strip leaves the state unchanged: nothing is launched, nothing is read
  if (T == 0 || Vq == 0) return VP_OK;
  if (!ws) return VP_ERR_WORKSPACE;
  if (ws_bytes < fwd_ws_min(shard)) return VP_ERR_WORKSPACE;
  if (misaligned(ws)) return VP_ERR_ALIGN;
  if (!H || !W_shard || !targets || !state) return VP_ERR_NULL;
  if (misaligned(H) || misaligned(W_shard)) return VP_ERR_ALIGN;
  if (((uintptr_t)state & 3u) != 0) return VP_ERR_ALIGN;
  hipStream_t s = (hipStream_t)stream;

  const FwdPlan plan = plan_fwd(shard, slots_in(shard, ws_bytes));
  const vpce::FwdTile ft = vpce::fwd_tile(shard->dtype, plan.kind);
  const int32_t tiles = (int32_t)ceil_div(Vq, ft.bm);
  const int S = std::min(plan.splits, (int)tiles);
  char* base = (char*)ws + kHeaderBytes;
  vpce::FwdArgs a;
  memset(&a, 0, sizeof(a));
  a.st.P = 1;
  a.st.w[0] = W_shard;
  a.st.off[0] = id_offset;
  a.st.rows[0] = (int32_t)Vq;
  a.st.tile0[0] = 0;
  for (int i = 1; i <= VP_MAX_SHARDS; ++i) a.st.tile0[i] = tiles;
  for (int i = 1; i < VP_MAX_SHARDS; ++i) a.st.off[i] = id_offset + Vq;
  a.n_tiles = tiles;
  a.H = H;
  a.targets = targets;
  a.T = T;
  a.d = (int32_t)shard->d;
  a.n_tok_blocks = (int32_t)ceil_div(T, ft.bn);
  a.n_splits = S;
  a.kind = plan.kind;
  a.m_part = (float*)base;
  a.s_part = (float*)(base + align256((size_t)S * T * 4));
  a.y_tgt = state + 2 * T;  // written only for targets this shard owns
  if (!vpce::run_fwd(shard->dtype, a, s)) return VP_ERR_HIP;

  vpce::FoldArgs f;
  f.m_part = a.m_part;
  f.s_part = a.s_part;
  f.T = T;
  f.n_splits = S;
  f.state = state;
  return vpce::run_fold_merge(f, s) ? VP_OK : VP_ERR_HIP;
}

vp_status vp_ce_fold_finalize(const vp_problem* prob, const int64_t* targets, const float* state,
                              float* loss, float* lse, void* ws, size_t ws_bytes, void* stream) {
  int64_t V = 0;
  vp_status st = validate(prob, &V);
  if (st != VP_OK) return st;
  if (!ws) return VP_ERR_WORKSPACE;
  if (ws_bytes < kHeaderBytes) return VP_ERR_WORKSPACE;
  if (misaligned(ws)) return VP_ERR_ALIGN;
  const int64_t T = prob->T;
  if (T > 0) {
    if (!targets || !state || !loss || !lse) return VP_ERR_NULL;
    if (((uintptr_t)state & 3u) != 0) return VP_ERR_ALIGN;
  }
  hipStream_t s = (hipStream_t)stream;
  unsigned long long* counter = (unsigned long long*)ws;
  if (!vpce::run_ws_init(counter, s)) return VP_ERR_HIP;
  vpce::FinArgs f;
  f.state = state;
  f.targets = targets;
  f.T = T;
  f.V = V;
  f.ignore_index = prob->ignore_index;
  f.loss = loss;
  f.lse = lse;
  f.bad_counter = counter;
  return vpce::run_fold_finalize(f, s) ? VP_OK : VP_ERR_HIP;
}

vp_status vp_ce_plan_info(const vp_problem* prob, vp_plan_info* info) {
  const vp_status st = validate(prob, nullptr);
  if (st != VP_OK) return st;
  if (!info) return VP_ERR_NULL;
  vp_problem p = *prob;
  p.T = std::max<int64_t>(p.T, 1);
  const BwdPlan plan = plan_bwd(&p);
  int64_t n = 0;
  walk_strips(&p, plan.Vc, vpce::bwd_tile(p.dtype, plan.cls).bm,
              [&](bool fresh, int, int64_t, int64_t, int64_t) { n += fresh; });
  if (prob->T == 0) n = 0;
  info->Tc = plan.Tc;
  info->Vc = plan.Vc;
  info->strips = n * ceil_div(p.T, plan.Tc);
  info->stage_launches = info->strips > 0 ? info->strips + 1 : 0;
  return VP_OK;
}

vp_status vp_ce_backward(const vp_problem* prob, const void* H, const void* const* W_shards,
                         const int64_t* targets, const float* lse, const float* grad_loss,
                         float* dH, float* const* dW_shards, void* ws, size_t ws_bytes,
                         void* stream) {
  int64_t V = 0;
  vp_status st = validate(prob, &V);
  if (st != VP_OK) return st;
  if ((st = check_shards(prob, W_shards)) != VP_OK) return st;
  if (!dW_shards) return VP_ERR_NULL;
  for (int q = 0; q < prob->P; ++q) {
    if (prob->shard_rows[q] > 0 && !dW_shards[q]) return VP_ERR_NULL;
    if (prob->shard_rows[q] > 0 && misaligned(dW_shards[q])) return VP_ERR_ALIGN;
  }
  if (!ws) return VP_ERR_WORKSPACE;
  if (ws_bytes < bwd_ws_bytes(prob)) return VP_ERR_WORKSPACE;
  if (misaligned(ws)) return VP_ERR_ALIGN;
  const int64_t T = prob->T;
  if (T > 0) {
    if (!H || !targets || !lse || !grad_loss || !dH) return VP_ERR_NULL;
    if (misaligned(H) || misaligned(dH)) return VP_ERR_ALIGN;
  }
  hipStream_t s = (hipStream_t)stream;
  unsigned long long* counter = (unsigned long long*)ws;
  const bool accumulate = (prob->flags & VP_ACCUMULATE_DW) != 0;
  const int64_t d = prob->d;

  if (T == 0) {  // G is empty: dW = 0 (or unchanged when accumulating); dH has no rows
    if (!vpce::run_ws_init(counter, s)) return VP_ERR_HIP;
    if (!accumulate)
      for (int q = 0; q < prob->P; ++q)
        if (!vpce::run_fill_zero(dW_shards[q], prob->shard_rows[q] * d, s)) return VP_ERR_HIP;
    return VP_OK;
  }
  BwdPlan f = plan_bwd(prob);
  cut_strips(prob, &f);
  if (f.off_yt + align256((size_t)T * 4) > ws_bytes) return VP_ERR_WORKSPACE;
  const vpce::BwdTile ft = vpce::bwd_tile(prob->dtype, f.cls);
  const size_t eb = elem_bytes(prob->dtype);
  const int64_t KB = vpce::tile_shape(prob->dtype).kblock;
  char* wsb = (char*)ws;
  float* yt = (float*)(wsb + f.off_yt);
  float* part = f.max_jobs > 1 ? (float*)(wsb + f.off_part) : dH;
  {  // the target logit of every token, read by the residual tiles for the one-hot term
    vpce::TgtArgs ta;
    memset(&ta, 0, sizeof(ta));
    int32_t n_tiles = 0;
    build_table(prob, W_shards, ft.bm, &ta.st, &n_tiles);
    ta.H = H;
    ta.targets = targets;
    ta.T = T;
    ta.V = V;
    ta.d = (int32_t)d;
    ta.yt = yt;
    ta.ignore_index = prob->ignore_index;
    if (T <= kFewTokens) {
      ta.count = counter;
    } else if (!vpce::run_ws_init(counter, s) ||
               !vpce::run_count_bad(targets, T, V, prob->ignore_index, counter, s)) {
      return VP_ERR_HIP;
    }
    if (!vpce::run_target_logits(prob->dtype, ta, s)) return VP_ERR_HIP;
  }
  auto copy_transposed = [&](const void* in, int64_t rows, void* out, int64_t rows_pad) {
    vpce::TransposeArgs tr;
    tr.in = in;
    tr.ld_in = d;
    tr.out = out;
    tr.R = (int32_t)rows;
    tr.C = (int32_t)d;
    tr.R_pad = (int32_t)rows_pad;
    return vpce::run_transpose(prob->dtype, tr, s);
  };
  if (f.cls == 3 && !copy_transposed(H, T, wsb + f.off_ht, round_up(T, 256))) return VP_ERR_HIP;
  int64_t off[VP_MAX_SHARDS];
  int64_t acc = 0;
  for (int q = 0; q < prob->P; ++q) {
    off[q] = acc;
    acc += prob->shard_rows[q];
  }
  auto segments = [&](const BwdStrip& st, vpce::StageSeg* out) {
    for (size_t i = 0; i < st.segs.size(); ++i) {
      const BwdStrip::Seg& sg = st.segs[i];
      out[i].w = (const char*)W_shards[sg.q] + (size_t)(sg.v0 * d) * eb;
      out[i].dw = dW_shards[sg.q] + sg.v0 * d;
      out[i].gid0 = off[sg.q] + sg.v0;
      out[i].rows = (int32_t)sg.rows;
      out[i].row0 = (int32_t)sg.row0;
    }
    return (int32_t)st.segs.size();
  };
  // Launch k writes the residual of strip k (into buffer k % 2) and contracts strip
  // k - 1 (from the other one).  Stream order gives every dependency: strip k - 1 was
  // written by launch k - 1; buffer k % 2 was last read by launch k - 1; dH rows and dW
  // chunks are only updated by consecutive launches.
  const int64_t n_tc = ceil_div(T, f.Tc), n = (int64_t)f.strips.size() * n_tc;
  for (int64_t k = 0; k <= n; ++k) {
    vpce::StageArgs a;
    memset(&a, 0, sizeof(a));
    a.g.H = H;
    a.g.targets = targets;
    a.g.lse = lse;
    a.g.grad = grad_loss;
    a.g.strip = wsb + f.off_g[k % 2];
    a.g.strip_t = wsb + f.off_gt[k % 2];
    a.g.Tc = f.Tc;
    a.g.Vc = f.Vr;
    a.g.V = V;
    a.g.ignore_index = prob->ignore_index;
    a.g.yt = yt;
    a.g.d = (int32_t)d;
    if (k < n) {
      const BwdStrip& st = f.strips[k / n_tc];
      a.g.t0 = k % n_tc * f.Tc;
      a.g.N = (int32_t)std::min(f.Tc, T - a.g.t0);
      a.n_gseg = segments(st, a.gseg);
      a.g.n_vt = (int32_t)(st.rows_pad / ft.bm);
    }
    int64_t longest = 0;
    if (k >= 1) {
      const BwdStrip& st = f.strips[(k - 1) / n_tc];
      a.c_t0 = (k - 1) % n_tc * f.Tc;
      a.c_N = (int32_t)std::min(f.Tc, T - a.c_t0);
      a.n_cseg = segments(st, a.cseg);
      if (f.cls == 3) {
        a.Ht = wsb + f.off_ht;
        a.Wt = wsb + f.off_wt;
        if (a.c_t0 == 0)  // the first strip of this vocabulary chunk
          for (int i = 0; i < a.n_cseg; ++i)
            if (!copy_transposed(a.cseg[i].w, a.cseg[i].rows,
                                 wsb + f.off_wt + (size_t)(a.cseg[i].row0 * d) * eb,
                                 round_up(a.cseg[i].rows, KB)))
              return VP_ERR_HIP;
      }
      a.n_job = (int32_t)st.jobs.size();
      for (size_t j = 0; j < st.jobs.size(); ++j) {
        a.job[j] = st.jobs[j];
        int64_t len = ceil_div(st.jobs[j].rows, KB);
        if (st.jobs[j].n_seg > 1) {
          len = 0;
          for (int i = 0; i < st.jobs[j].n_seg; ++i) len += ceil_div(st.segs[st.jobs[j].seg + i].rows, KB);
        }
        longest = std::max(longest, len);
      }
      a.w_tiles = (int32_t)ceil_div(st.rows_pad, ft.bn);
      a.G = wsb + f.off_g[(k - 1) % 2];
      a.Gt = wsb + f.off_gt[(k - 1) % 2];
      a.part = part;
      a.part_stride = T * d;
      a.beta_w = (a.c_t0 > 0 || accumulate) ? 1 : 0;
    }
    // the kinds with the longest sums first, so that the last round of tiles is short
    const int64_t slices[3] = {longest, ceil_div(std::min(f.Tc, T), KB), ceil_div(d, KB)};
    for (int i = 0; i < 3; ++i) a.order[i] = i;
    std::sort(a.order, a.order + 3, [&](int x, int y) { return slices[x] > slices[y]; });
    if (!vpce::run_stage(prob->dtype, f.cls, a, s)) return VP_ERR_HIP;
  }
  if (f.max_jobs > 1 && !vpce::run_sum_parts(part, f.max_jobs, T * d, dH, s)) return VP_ERR_HIP;
  return VP_OK;
}

vp_status vp_ce_check(const void* ws, void* stream, int64_t* bad_targets) {
  if (!ws) return VP_ERR_NULL;
  unsigned long long count = 0;
  hipStream_t s = (hipStream_t)stream;
  if (hipMemcpyAsync(&count, ws, sizeof(count), hipMemcpyDeviceToHost, s) != hipSuccess)
    return VP_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return VP_ERR_HIP;
  if (bad_targets) *bad_targets = (int64_t)count;
  return count ? VP_ERR_TARGET : VP_OK;
}

}  // extern "C"
