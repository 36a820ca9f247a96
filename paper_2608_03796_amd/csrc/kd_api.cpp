// C ABI of the fused chunked top-K KL loss: argument checks, workspace plan
// and the chunk schedule of Algorithm 1 (§3.2.3). Plain C++: every device
// operation goes through the launchers of kd_kernels.hip.
#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <numeric>

#include "../../include/kdtopk.h"
#include "kd_launch.h"

static_assert(KD_SCRATCH_BYTES == kd_scratch_bytes_max - kd_scratch_slack,
              "scratch size in the header");

namespace {

constexpr int64_t kTile = 256;
constexpr int64_t kMaxN = (int64_t)1 << 31;     // N < 2^31
constexpr int64_t kMaxV = (int64_t)1 << 20;     // keeps 32-bit buffer offsets in range
constexpr int64_t kMaxD = 65536;
constexpr int64_t kMaxChunk = (int64_t)1 << 20; // rows per chunk actually used
// teacher entries per token: a 256-token tile's 256 K entries are numbered in
// 20 bits by the bucket pass, and k is packed in 16
constexpr int64_t kMaxK = 4096;

// the first bytes of every workspace: scalars, among them the index check's flag
constexpr size_t kMiscBytes = 256;
// no limit to the partial tiles of dH (see kd_dh_rounds): two rounds of 256 x 256
constexpr int kPartSpaceMax = 512 * 256 * 256 / 64;

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t rup(int64_t a, int64_t b) { return cdiv(a, b) * b; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Plan {
  int64_t N, D, V, K;
  int eb;              // element bytes of hidden / W / dZ
  int64_t c;           // rows per chunk
  int64_t cp;          // c rounded up to the 256-row tile
  int64_t Vp;          // V rounded up to the 256-column tile
  int64_t nVT;         // 256-column vocabulary tiles
  int64_t nP;          // (reference, sum) partials per token: vocabulary tiles of the projection
  int64_t nchunks;
  int64_t nblk;        // loss partials of a full chunk (one per kLossRows rows)
  int64_t G;           // chunks whose dZ rows are gathered before one dH and one dW GEMM
  int64_t merged;      // caller's chunks per chunk of the plan (1 or the group size)
  int64_t ngroups;
  bool dh_per_group;   // dH once per group (a chunk alone has too few tiles) or per chunk
  bool prep_per_group; // rows prepared once per group (chunks of whole 256-token tiles)
  int64_t ng;          // rows of the per-row arrays: the group's, or one chunk's (padded)
  int64_t ksteps;      // K steps of dH (the vocabulary)
  int64_t dh_rows[2];  // the row counts dH runs on: of the full and the last chunk or group
  size_t dh_bytes, dw_bytes;  // partial tiles of their split last rounds it holds
  size_t off_misc, off_p, off_tidx, off_rows, off_pm, off_ps, off_hits, off_hitp, off_hoff, off_zhit,
      off_lossp, off_dz, off_fac, off_ht, off_rowmap, off_parts, total;
};

kd_status check_problem(const kd_problem* p) {
  if (p == nullptr) return KD_ERR_NULL_PTR;
  if ((p->flags & ~(KD_FLAG_TEACHER_LOGPROBS | KD_FLAG_GRAD_HIDDEN_F32)) != 0) return KD_ERR_BAD_ARG;
  if (p->dtype != KD_F32 && p->dtype != KD_BF16) return KD_ERR_UNSUPPORTED;
  if (p->N < 0 || p->N >= kMaxN) return KD_ERR_BAD_SHAPE;
  if (p->D < 64 || p->D > kMaxD) return KD_ERR_BAD_SHAPE;
  if (p->V < 1 || p->V > kMaxV) return KD_ERR_BAD_SHAPE;
  if (p->K < 1 || (int64_t)p->K > p->V || p->K > kMaxK) return KD_ERR_BAD_SHAPE;
  if (p->chunk < 1) return KD_ERR_BAD_ARG;
  if (!(isfinite(p->temperature) && p->temperature > 0.0f)) return KD_ERR_BAD_ARG;
  if (p->D % 64 != 0) return KD_ERR_UNSUPPORTED;
  return KD_OK;
}

// Tile edge of each contraction over n token rows: fp32 runs 128x128 tiles; bf16
// 256x256 tiles, whose main loop is 10 to 25% faster, unless these are so few
// that most of the chip would idle. The lines are where whole calls crossed
// (256 and 128 tiles, us; t = 256x256 tiles of the launch):
//  * projection, t <= 128: 400 x 1024 x 8192 (t = 64) 90.3, 80.6; 600 x 3072 x
//    10000 (120) 179, 172; 1000 x 512 x 16000 (252) 104, 110;
//  * dH, t <= 8: 256 x 256 x 8192 (1) 69, 63; 512 x 1024 x 32000 (8) 154, 148;
//    128 x 4096 x 32000 (16) 322, 326; 1024 x 1024 x 32000 (16) 233, 239;
//  * dW, t <= 128: 2000 x 512 x 4096 (32) 110, 90; 1000 x 512 x 16000 (126) 104,
//    97; 2000 x 4096 x 4096 (256) 226, 238. Also up to two K steps (128 tokens)
//    in up to two rounds, where a tile is all epilogue: 77 x 768 x 32003
//    (t = 375) 109, 86. Past two rounds 90 calls of 16 to 128 tokens, D = 64 to
//    4096, took 0.90 to 1.04 of the time in 128x128 tiles up to t = 1400 (0.95 in the
//    middle) and 0.98 to 1.13 from 1530 on (128 x 1024 x 100003, t = 1564: 265, 285):
//    the line could lie at about 1400.
int64_t tiles256(int64_t m, int64_t n) { return cdiv(m, 256) * cdiv(n, 256); }
int proj_tile(const Plan& pl, int64_t n) {
  return pl.eb == 4 || tiles256(pl.V, n) <= 128 ? 128 : 256;
}
// The projection's 256x256 tiles over n rows that run whole; the others run as
// 128x128 tiles in a launch of their own: up to 64 tiles behind full rounds,
// which would occupy a quarter of the chip for a round's time (512 x 2048 x
// 37000, 290 tiles: 350 and 336 us; forward only 3000 x 2048 x 33000, 1548
// tiles: 390 and 378 us; 2000 x 2048 x 50021, 1568 tiles: 1163 and 1158 us).
// With 128 of them it no longer paid (768 x 2048 x 32768: 360 and 364 us).
int64_t proj_large(const Plan& pl, int64_t n) {
  if (proj_tile(pl, n) == 128) return 0;
  const int64_t t = tiles256(pl.V, n), rem = t % 256;
  if (t < 256 || rem == 0 || rem > 64) return t;
  return t - rem;
}
int dh_tile(const Plan& pl, int64_t n) {
  return pl.eb == 4 || tiles256(pl.D, n) <= 8 ? 128 : 256;
}
int dw_tile(const Plan& pl, int64_t n) {
  const int64_t t = tiles256(pl.D, pl.V);
  return pl.eb == 4 || t <= 128 || (n <= 128 && t <= 512) ? 128 : 256;
}

// Tiles of dH over n rows, and how they run with all the partial tiles they like.
int dh_tiles(const Plan& pl, int64_t n) {
  const int ts = dh_tile(pl, n);
  return (int)(cdiv(n, ts) * cdiv(pl.D, ts));
}
KdRounds dh_split(const Plan& pl, int64_t n, int ts) {
  return kd_dh_rounds((int)n, (int)pl.D, ts, (int)pl.ksteps, pl.eb == 4, kPartSpaceMax);
}
KdRounds dh_split(const Plan& pl, int64_t n) { return dh_split(pl, n, dh_tile(pl, n)); }
// The most bytes of partial tiles dH over 1..n rows in the tiles of n rows needs
// (fewer rows hold tokens when ignored ones are left out).
size_t dh_part_bytes(const Plan& pl, int64_t n) {
  const int ts = dh_tile(pl, n), units = kd_units(ts);
  const int64_t tm_max = cdiv(n, ts), td = cdiv(pl.D, ts);
  // the tiles left over for the last round repeat with this many tile rows, and
  // take the most space in the last repetition
  const int64_t period = units / std::gcd(td, (int64_t)units);
  size_t bytes = 0;
  for (int64_t tm = tm_max; tm > std::max<int64_t>(0, tm_max - period); --tm) {
    const int64_t rows = std::min(tm * ts, n);
    const KdRounds s = dh_split(pl, rows, ts);
    const int64_t part = s.dp == 0 ? rows * pl.D : (int64_t)s.rem * ts * ts;  // of a range
    if (s.split > 1) bytes = std::max(bytes, (size_t)4 * s.split * part);
  }
  return bytes;
}
// The partial tiles dW over n tokens needs.
int dw_parts(const Plan& pl, int64_t n) {
  const int ts = dw_tile(pl, n);
  const KdRounds s =
      kd_split_rounds((int)(cdiv(pl.D, ts) * cdiv(pl.V, ts)), (int)(rup(n, 64) * pl.eb / 128),
                      kd_units(ts), kd_part_cost(ts, pl.eb == 4), 1 << 20);
  return s.split > 1 ? s.rem * s.split : 0;
}

// The plan without the partial tiles of split last rounds; g_max > 0 caps the
// chunks per dW group (see plan_within).
Plan base_plan(const kd_problem* p, int64_t g_max = 0) {
  Plan pl{};
  pl.N = p->N;
  pl.D = p->D;
  pl.V = p->V;
  pl.K = p->K;
  pl.eb = p->dtype == KD_BF16 ? 2 : 4;
  pl.c = std::min<int64_t>(std::min<int64_t>(p->chunk, std::max<int64_t>(p->N, 1)), kMaxChunk);
  pl.cp = rup(pl.c, kTile);
  pl.Vp = rup(pl.V, kTile);
  pl.nVT = pl.Vp / kTile;
  pl.ksteps = pl.Vp * pl.eb / 128;
  pl.nchunks = cdiv(pl.N, pl.c);
  pl.nblk = cdiv(pl.c, kLossRows);
  // dW is accumulated in fp32 in place: each dW GEMM reads and writes all of
  // grad_W once, so gather the dZ rows of up to ~16384 tokens (and at most
  // 4 GiB of dZ) per GEMM
  pl.G = std::max<int64_t>(1, std::min<int64_t>(16384 / pl.c, std::max<int64_t>(pl.nchunks, 1)));
  pl.G = std::max<int64_t>(
      1, std::min<int64_t>(pl.G, ((int64_t)4 << 30) / std::max<int64_t>(pl.c * pl.Vp * pl.eb, 1)));
  if (g_max > 0) pl.G = std::min<int64_t>(pl.G, g_max);
  // The chunks of a dW group are processed as one chunk of the group's rows
  // when that saves work: the same transient (the group's dZ rows), the same
  // arithmetic per token and per grad_W contraction.
  //  * A chunk of few tiles (dH does not fill the compute units with it and
  //    runs per group anyway): one projection per group instead of one per
  //    chunk, unless the chunk's projection fills whole rounds of the 256
  //    compute units with 2048 rows or more. Measured at D = 4096,
  //    V = 131072 (whole rounds), unmerged and merged: chunk 256, 4096 tokens
  //    10.80 and 9.55 ms; 512, 8192 tokens 19.26 and 18.59 ms; 1024, 16384
  //    tokens 37.99 and 37.88 ms; 2048, 16384 tokens 37.61 and 37.84 ms. fp32,
  //    256 tokens in chunks of 64 (fp32 MFMAs in 256x256 tiles): 488 and 250 us.
  //    Other heads of whole rounds (D = 512 to 8192, V = 32768 to 131072, 8192 and
  //    16384 tokens), merged over unmerged: chunk 256 0.87 to 0.91, 512 0.95 to
  //    0.99, 1024 0.96 to 1.03 (above 1 at D = 512, V = 65536 only), 2048 0.97 to
  //    1.02, 4096 0.97 to 1.02: no clear winner from 2048 on.
  //  * A chunk whose tiles fill the chip is merged only when padding its last
  //    256-token tile costs more than merging (above 5% of its rows): each
  //    chunk's dH right after its own projection is faster than one dH over
  //    the group (chunk 4000, 2.4% padding: 36.72 unmerged, 37.42 ms merged).
  pl.merged = 1;
  const bool dh_grouped = dh_tiles(pl, pl.c) < kd_units(dh_tile(pl, pl.c)) || dh_split(pl, pl.c).split > 1;
  const int pts = proj_tile(pl, pl.c);
  const bool full_rounds = pl.c % kTile == 0 &&
                           cdiv(pl.c, pts) * (pl.Vp / pts) % kd_units(pts) == 0 && pl.c >= 2048;
  const bool padded = (rup(pl.c, kTile) - pl.c) * 20 > pl.c;
  if (pl.G > 1 && (padded || (dh_grouped && !full_rounds))) {
    pl.merged = pl.G;
    pl.c = std::min<int64_t>(pl.c * pl.G, pl.N);
    pl.cp = rup(pl.c, kTile);
    pl.nchunks = cdiv(pl.N, pl.c);
    pl.nblk = cdiv(pl.c, kLossRows);
    pl.G = 1;
  }
  // dH runs per chunk when a chunk's tiles fill the chip, else once per group
  // of G chunks (G times the tiles, dW's grouping); its vocabulary range is
  // split only when the rows it covers still have too few tiles
  pl.ngroups = cdiv(pl.nchunks, pl.G);
  // the teacher prologue, bucketing and reference logits run once per group
  // when every chunk starts on a 256-token tile of the group (the buckets are
  // per tile), else once per chunk
  pl.prep_per_group = pl.G > 1 && pl.c % kTile == 0;
  pl.ng = pl.prep_per_group ? pl.G * pl.c : pl.cp;
  pl.dh_per_group = dh_split(pl, pl.c).split > 1;
  if (pl.dh_per_group) {
    pl.dh_rows[0] = std::min<int64_t>(pl.G * pl.c, pl.N);
    pl.dh_rows[1] = pl.N - (pl.ngroups - 1) * pl.G * pl.c;
  } else {
    pl.dh_rows[0] = pl.c;
    pl.dh_rows[1] = pl.N - (pl.nchunks - 1) * pl.c;
  }
  // rows of the last chunk, whose tiles may differ from the others'
  const int64_t c_last = pl.N - (std::max<int64_t>(pl.nchunks, 1) - 1) * pl.c;
  const bool small = proj_large(pl, pl.c) < tiles256(pl.V, pl.c) ||
                     proj_large(pl, c_last) < tiles256(pl.V, c_last);
  pl.nP = small ? 2 * pl.nVT : pl.nVT;
  size_t t = 0;
  auto take = [&](size_t bytes) {
    const size_t o = align256(t);
    t = o + bytes;
    return o;
  };
  pl.off_misc = take(kMiscBytes);
  pl.off_p = take((size_t)pl.ng * pl.K * 4);
  pl.off_tidx = take((size_t)pl.ng * pl.K * 4);
  pl.off_rows = take((size_t)7 * pl.ng * 4);
  pl.off_pm = take((size_t)pl.cp * pl.nP * 4);
  pl.off_ps = take((size_t)pl.cp * pl.nP * 4);
  pl.off_hits = take((size_t)pl.ng * pl.K * 4);
  pl.off_hitp = take((size_t)pl.ng * pl.K * 4);
  pl.off_hoff = take((size_t)(pl.ng / kTile) * (pl.nVT + 1) * 4);
  pl.off_zhit = take((size_t)pl.ng * pl.K * 4);
  pl.off_lossp = take((size_t)std::max<int64_t>(pl.nchunks, 1) * pl.nblk * 4);
  pl.off_dz = take((size_t)pl.G * pl.c * pl.Vp * pl.eb);
  // factor of each dZ row of the group in the single-projection schedule
  pl.off_fac = take((size_t)pl.G * pl.c * 4);
  // the hidden rows of one dW group, transposed (tokens padded to 64); until
  // the group's dW it holds the group's tokens that are not ignored, as rows
  pl.off_ht = take((size_t)pl.D * rup(pl.G * pl.c, 64) * pl.eb);
  // the token of each of those rows
  pl.off_rowmap = take((size_t)pl.G * pl.c * 4);
  pl.total = align256(t);
  return pl;
}

// Adds the partial tiles of dH's and dW's split last rounds, at most `room`
// bytes of them: where these are fewer than the model would like, it splits into
// fewer ranges (its max_parts). Both have the same place: a group's tail has
// added up dH's parts before its dW starts.
void add_parts(Plan* pl, size_t room = (size_t)1 << 40) {
  size_t dh = 0, dw = 0;
  for (int i = 0; i < 2; ++i) {
    const int64_t r = pl->dh_rows[i];
    if (r <= 0 || (i == 1 && r == pl->dh_rows[0])) continue;
    dh = std::max(dh, dh_part_bytes(*pl, r));
  }
  const int64_t g_full = std::min<int64_t>(pl->G * pl->c, pl->N);
  const int64_t g_last = pl->N - (std::max<int64_t>(pl->ngroups, 1) - 1) * pl->G * pl->c;
  for (int64_t r : {g_full, g_last}) {
    if (r <= 0) continue;
    const int ts = dw_tile(*pl, r);
    dw = std::max(dw, (size_t)dw_parts(*pl, r) * ts * ts * 4);
  }
  pl->dh_bytes = std::min(dh, room);
  pl->dw_bytes = std::min(dw, room);
  pl->off_parts = pl->total;
  pl->total = align256(pl->off_parts + std::max(pl->dh_bytes, pl->dw_bytes));
}

Plan make_plan(const kd_problem* p, int64_t g_max = 0) {
  Plan pl = base_plan(p, g_max);
  add_parts(&pl);
  return pl;
}

// The plan of make_plan when it fits the static scratch; else with fewer chunks
// per dW group; at last one chunk per group with the partial tiles that fit (a
// dH without any leaves most of the chip idle: 1888 x 2048 x 24507 in fp32 has
// 240 tiles for 512 workgroups). False if one chunk without partial tiles
// exceeds `cap` bytes. The partials of 128-column vocabulary tiles above those
// of 256-column ones are not counted against the cap: kd_scratch_slack holds
// them, and where there are none, more partial tiles.
// The group is found by bisection, first of the plan without its partial tiles
// (a microsecond a step), then of the whole plan (2 to 15): the size grows with
// the group except for the partial tiles, of which some group sizes need none,
// so now and then a group is a few percent below the largest that fits. One by
// one from the whole group down, 20000 tokens of D = 256, V = 131072 in chunks
// of 64 took 2.9 ms before the first launch, now 21 us; N = 16384, D = 64 in
// chunks of one 187 ms, now 0.1 ms.
bool plan_within(const kd_problem* p, size_t cap, Plan* out) {
  // without its partial tiles; with them
  auto base_fits = [&](const Plan& q) {
    return q.total - (size_t)q.cp * (q.nP - q.nVT) * 8 <= cap;
  };
  auto fits = [](const Plan& q) { return q.total <= kd_scratch_bytes_max; };
  // the most chunks per group, up to g, that pass (1 is not tried)
  auto largest = [](int64_t g, auto ok) {
    int64_t lo = 1;
    while (lo < g) {
      const int64_t mid = lo + (g - lo + 1) / 2;
      if (ok(mid)) lo = mid;
      else g = mid - 1;
    }
    return lo;
  };
  Plan pl = base_plan(p);
  int64_t g = pl.G * pl.merged;  // the caller's chunks per dW group
  if (!base_fits(pl)) {
    g = largest(g - 1, [&](int64_t k) { return base_fits(base_plan(p, k)); });
    pl = base_plan(p, g);
    if (!base_fits(pl)) return false;
  }
  if (!fits(pl)) return false;
  add_parts(&pl);
  if (!fits(pl) && g > 1)
    pl = make_plan(p, largest(g - 1, [&](int64_t k) { return fits(make_plan(p, k)); }));
  if (!fits(pl)) {
    pl = base_plan(p, 1);
    add_parts(&pl, kd_scratch_bytes_max - pl.total);
  }
  *out = pl;
  return true;
}

inline bool aligned16(const void* q) { return ((uintptr_t)q & 15u) == 0; }

// KD_DEBUG_CHECK=1: every entry point validates the teacher indices first.
bool debug_index_check() {
  const char* e = getenv("KD_DEBUG_CHECK");
  return e != nullptr && e[0] == '1' && e[1] == '\0';
}

}  // namespace

extern "C" {

int kd_abi_version(void) { return KDTOPK_ABI_VERSION; }

const char* kd_status_string(int s) {
  switch (s) {
    case KD_OK: return "KD_OK: success";
    case KD_ERR_NULL_PTR: return "KD_ERR_NULL_PTR: a required pointer is NULL";
    case KD_ERR_BAD_SHAPE: return "KD_ERR_BAD_SHAPE: invalid N, D, V or K, or a size limit";
    case KD_ERR_BAD_ARG: return "KD_ERR_BAD_ARG: invalid chunk, temperature, flags or mode";
    case KD_ERR_UNSUPPORTED: return "KD_ERR_UNSUPPORTED: dtype, D % 64 != 0 or misaligned pointer";
    case KD_ERR_WORKSPACE_TOO_SMALL: return "KD_ERR_WORKSPACE_TOO_SMALL: workspace below the required size";
    case KD_ERR_BAD_INDEX: return "KD_ERR_BAD_INDEX: teacher index outside [0, V) or repeated in a row";
    case KD_ERR_DEVICE: return "KD_ERR_DEVICE: HIP launch or runtime error";
    default: return "unknown kd_status";
  }
}

kd_status kd_topk_kl_workspace_size(const kd_problem* p, size_t* bytes) {
  if (p == nullptr || bytes == nullptr) return KD_ERR_NULL_PTR;
  const kd_status st = check_problem(p);
  if (st != KD_OK) return st;
  *bytes = make_plan(p).total;
  return KD_OK;
}

}  // extern "C"

namespace {

// Arguments shared by the three entry points once they are validated.
struct Call {
  int mode;
  const void* hidden;
  const void* W;
  const int32_t* idx;
  const float* tlogit;
  const uint8_t* ignore;
  float* loss;              // forward modes
  float* lpt;
  float* logz_out;          // forward only
  const float* logz_in;     // backward only
  const float* gscale;
  const float* gtok;
  void* grad_hidden;        // backward modes
  float* grad_W;
  int accumulate;
  void* ws;
  size_t ws_bytes;
  void* stream;
};

// Common checks: problem, pointers every mode needs, alignment, workspace
// (unless the workspace is the library's own scratch).
kd_status validate(const kd_problem* p, const Call& c, const Plan& pl, bool own_ws = false) {
  if (!own_ws && c.ws == nullptr) return KD_ERR_NULL_PTR;
  if (p->N > 0 && (c.hidden == nullptr || c.W == nullptr || c.idx == nullptr ||
                   c.tlogit == nullptr))
    return KD_ERR_NULL_PTR;
  if (c.accumulate != 0 && c.accumulate != 1) return KD_ERR_BAD_ARG;
  if (!aligned16(c.hidden) || !aligned16(c.W) || !aligned16(c.grad_hidden) ||
      !aligned16(c.grad_W) || !aligned16(c.ws))
    return KD_ERR_UNSUPPORTED;
  if (!own_ws && c.ws_bytes < pl.total) return KD_ERR_WORKSPACE_TOO_SMALL;
  return KD_OK;
}

// Enqueues Algorithm 1 for one call: the host chunk schedule (§3.2.3).
kd_status enqueue(const kd_problem* p, const Plan& pl, const Call& c) {
  const bool fwd = c.mode != KD_MODE_BWD, bwd = c.mode != KD_MODE_FWD;
  char* ws = static_cast<char*>(c.ws);
  // 1/N_valid: counted on the device with a mask, known here without
  const bool compact = c.ignore != nullptr && pl.N > 0;
  float* inv_nvalid = compact ? reinterpret_cast<float*>(ws + pl.off_misc + 4) : nullptr;
  const float inv_n = pl.N > 0 ? 1.0f / (float)pl.N : 0.0f;
  float* lossp = reinterpret_cast<float*>(ws + pl.off_lossp);
  const bool want_dh = bwd && c.grad_hidden != nullptr && pl.N > 0;
  const bool want_dw = bwd && c.grad_W != nullptr && pl.N > 0;

  if (bwd && c.grad_W != nullptr && pl.N == 0 && !c.accumulate &&
      kd_launch_fill(c.grad_W, pl.V * pl.D, c.stream) != 0)
    return KD_ERR_DEVICE;

  float* rows = reinterpret_cast<float*>(ws + pl.off_rows);
  float* fac = reinterpret_cast<float*>(ws + pl.off_fac);
  // the single-projection schedule stores dZ up to a factor per row, which
  // dH applies to its rows and dW to the hidden rows
  const bool scaled = fwd && bwd && (want_dh || want_dw);
  // With a mask, every entry point leaves the ignored tokens out (their loss
  // and gradient rows are 0): each dW group's other tokens are gathered
  // first, and the group's rows are those tokens in order, then rows without
  // a token, whose tiles the contractions skip (their count is on the
  // device).
  int* rowmap = reinterpret_cast<int*>(ws + pl.off_rowmap);
  int* gnrow = reinterpret_cast<int*>(ws + pl.off_misc + 16);
  char* hcomp = ws + pl.off_ht;
  int64_t n_partials = 0;
  int64_t group_tokens = 0;
  bool dw_done = false;
  // the per-row arrays from row `o` of the prepared rows; `g` = the row of
  // the chunk within its dW group
  auto chunk_args = [&](int64_t row0, int rcount, int64_t o, int64_t g, int stages) {
    KdChunkArgs a{};
    a.dtype = p->dtype;
    a.large_tiles = (int)proj_large(pl, rcount);
    a.nP = (int)pl.nP;
    a.mode = c.mode;
    a.stages = stages;
    a.one_projection = scaled ? 1 : 0;
    a.teacher_logprobs = (p->flags & KD_FLAG_TEACHER_LOGPROBS) ? 1 : 0;
    a.gscale = c.gscale;
    a.gtok = c.gtok;
    a.logz_in = c.logz_in;
    a.logz_out = c.logz_out ? (compact ? c.logz_out : c.logz_out + row0) : nullptr;
    a.D = pl.D;
    a.V = pl.V;
    a.K = (int)pl.K;
    a.row0 = row0;
    a.rows = rcount;
    a.inv_tau = 1.0f / p->temperature;
    a.W = c.W;
    a.Hc = compact ? hcomp + g * pl.D * pl.eb
                   : static_cast<const char*>(c.hidden) + row0 * pl.D * pl.eb;
    a.hidden = c.hidden;
    a.tidx_in = c.idx;
    a.tidx = reinterpret_cast<int32_t*>(ws + pl.off_tidx) + o * pl.K;
    a.tlogit = c.tlogit;
    a.ignore = c.ignore;
    a.inv_nvalid = inv_nvalid;
    a.inv_n = inv_n;
    a.grad_hidden = want_dh ? c.grad_hidden : nullptr;
    a.gh_f32 = (p->flags & KD_FLAG_GRAD_HIDDEN_F32) ? 1 : 0;
    a.lpt_full = c.lpt;
    a.rowmap = compact ? rowmap + g : nullptr;
    a.nrow = compact ? gnrow : nullptr;
    a.nrow_base = (int)g;
    a.p = reinterpret_cast<float*>(ws + pl.off_p) + o * pl.K;
    a.rowM = rows + o;
    a.rowH = rows + pl.ng + o;
    a.rowCoef = rows + 2 * pl.ng + o;
    a.rowCoefM = rows + 3 * pl.ng + o;
    a.rowL2 = rows + 4 * pl.ng + o;
    a.rowR = rows + 5 * pl.ng + o;
    a.rowFlag = reinterpret_cast<int*>(rows + 6 * pl.ng) + o;
    a.part_m = reinterpret_cast<float*>(ws + pl.off_pm);
    a.part_s = reinterpret_cast<float*>(ws + pl.off_ps);
    a.hits = reinterpret_cast<uint32_t*>(ws + pl.off_hits) + o * pl.K;
    a.hitp = reinterpret_cast<float*>(ws + pl.off_hitp) + o * pl.K;
    a.hoff = reinterpret_cast<int*>(ws + pl.off_hoff) + (o / kTile) * (pl.nVT + 1);
    a.zhit = reinterpret_cast<float*>(ws + pl.off_zhit) + o * pl.K;
    a.nVT = (int)pl.nVT;
    return a;
  };
  for (int64_t ci = 0; ci < pl.nchunks; ++ci) {
    const int64_t row0 = ci * pl.c;
    const int rcount = (int)std::min<int64_t>(pl.c, pl.N - row0);
    const int64_t slot = ci % pl.G;
    if (compact && slot == 0) {
      KdCompactArgs k{};
      k.ignore = c.ignore;
      k.N = pl.N;
      k.row0 = row0;
      k.rows = (int)std::min<int64_t>(pl.G * pl.c, pl.N - row0);
      k.rowmap = rowmap;
      k.nrow = gnrow;
      k.inv_nvalid = ci == 0 ? inv_nvalid : nullptr;
      if (kd_launch_compact(&k, c.stream) != 0) return KD_ERR_DEVICE;
    }
    if (pl.prep_per_group && slot == 0) {
      const int grows = (int)std::min<int64_t>(pl.G * pl.c, pl.N - row0);
      KdChunkArgs g = chunk_args(row0, grows, 0, 0, KD_STAGE_PREP);
      if (kd_launch_chunk(&g, c.stream) != 0) return KD_ERR_DEVICE;
    }
    KdChunkArgs a = chunk_args(row0, rcount, pl.prep_per_group ? slot * pl.c : 0, slot * pl.c,
                               pl.prep_per_group ? KD_STAGE_CHUNK
                                                 : (KD_STAGE_PREP | KD_STAGE_CHUNK));
    a.rowFactor = fac + slot * pl.c;
    a.dZ = (want_dh || want_dw) ? ws + pl.off_dz + slot * pl.c * pl.Vp * pl.eb : nullptr;
    a.ldz = pl.Vp;
    a.loss_per_token = c.lpt ? (compact ? c.lpt : c.lpt + row0) : nullptr;
    a.block_partial = lossp + n_partials;
    if (kd_launch_chunk(&a, c.stream) != 0) return KD_ERR_DEVICE;
    n_partials += cdiv(rcount, kLossRows);
    group_tokens += rcount;
    const bool last = ci == pl.nchunks - 1, group_end = last || slot == pl.G - 1;
    KdTailArgs tail{};
    tail.dtype = p->dtype;
    tail.D = pl.D;
    // dH over rows [r0, r0 + n) of the dZ buffer (from its row `zrow`)
    // (the parts of a split dH are added up by the group's tail: only the last
    // launch of a group is split)
    KdDhArgs h{};
    auto dh = [&](int64_t r0, int64_t n, int64_t zrow) -> bool {
      h.dtype = p->dtype;
      h.D = pl.D;
      h.V = pl.V;
      h.dZ = ws + pl.off_dz + zrow * pl.Vp * pl.eb;
      h.ldz = pl.Vp;
      h.W = c.W;
      h.tokens = n;
      h.tile = dh_tile(pl, n);
      h.part_space = group_end ? (int)(pl.dh_bytes / 256) : 0;
      h.partial = h.part_space > 0 ? reinterpret_cast<float*>(ws + pl.off_parts) : nullptr;
      h.gh_f32 = (p->flags & KD_FLAG_GRAD_HIDDEN_F32) ? 1 : 0;
      h.gH = compact ? c.grad_hidden
                     : static_cast<char*>(c.grad_hidden) + r0 * pl.D * (h.gh_f32 ? 4 : pl.eb);
      h.rowscale = scaled ? fac + zrow : nullptr;
      h.rowmap = compact ? rowmap + zrow : nullptr;
      h.nrow = compact ? gnrow : nullptr;
      h.nrow_base = (int)zrow;
      tail.dh = &h;
      return kd_launch_dh(&h, c.stream) == 0;
    };
    if (want_dh && !pl.dh_per_group && !dh(row0, rcount, slot * pl.c)) return KD_ERR_DEVICE;
    if (last && fwd) {
      tail.block_partial = lossp;
      tail.n_partials = (int)n_partials;
      tail.inv_nvalid = inv_nvalid;
      tail.inv_n = inv_n;
      tail.loss = c.loss;
    }
    if (!last && (!(want_dh || want_dw) || !group_end)) continue;
    // the group's dH (when it runs per group) and dW over the G chunks' dZ rows
    const int64_t row_first = row0 + rcount - group_tokens;
    if (want_dh && pl.dh_per_group && !dh(row_first, group_tokens, 0)) return KD_ERR_DEVICE;
    if (want_dw) {
      tail.Hg = compact ? c.hidden : static_cast<const char*>(c.hidden) + row_first * pl.D * pl.eb;
      tail.tokens = group_tokens;
      tail.Ht = ws + pl.off_ht;
      tail.rowscale = scaled ? fac : nullptr;
      tail.rowmap = compact ? rowmap : nullptr;
    }
    if (kd_launch_tail(&tail, c.stream) != 0) return KD_ERR_DEVICE;
    if (want_dw) {
      KdDwArgs d{};
      d.dtype = p->dtype;
      d.tile = dw_tile(pl, group_tokens);
      d.D = pl.D;
      d.V = pl.V;
      d.dZ = ws + pl.off_dz;
      d.ldz = pl.Vp;
      d.tokens = group_tokens;
      d.Ht = ws + pl.off_ht;
      d.beta = (dw_done || c.accumulate) ? 1 : 0;
      d.gW = c.grad_W;
      d.max_parts = (int)(pl.dw_bytes / ((size_t)d.tile * d.tile * 4));
      d.partial = d.max_parts > 0 ? reinterpret_cast<float*>(ws + pl.off_parts) : nullptr;
      d.nrow = compact ? gnrow : nullptr;
      if (kd_launch_dw(&d, c.stream) != 0) return KD_ERR_DEVICE;
      dw_done = true;
    }
    group_tokens = 0;
  }
  if (fwd && pl.nchunks == 0) {
    KdTailArgs tail{};
    tail.dtype = p->dtype;
    tail.loss = c.loss;
    if (kd_launch_tail(&tail, c.stream) != 0) return KD_ERR_DEVICE;
  }
  return KD_OK;
}

}  // namespace

extern "C" {

kd_status kd_topk_kl_fwd_bwd(const kd_problem* p, const void* hidden, const void* W,
                             const int32_t* teacher_idx, const float* teacher_logit,
                             const uint8_t* ignore, float* loss, float* loss_per_token,
                             void* grad_hidden, float* grad_W, int accumulate_grad_W,
                             void* workspace, size_t workspace_bytes, void* hip_stream) {
  kd_status st = check_problem(p);
  if (st != KD_OK) return st;
  if (loss == nullptr) return KD_ERR_NULL_PTR;
  const Call c{KD_MODE_FWD_BWD, hidden, W, teacher_idx, teacher_logit, ignore, loss,
               loss_per_token, nullptr, nullptr, nullptr, nullptr, grad_hidden, grad_W,
               accumulate_grad_W, workspace, workspace_bytes, hip_stream};
  const Plan pl = make_plan(p);
  st = validate(p, c, pl);
  if (st != KD_OK) return st;
  if (debug_index_check() && p->N > 0) {
    st = kd_topk_kl_check_indices(p, teacher_idx, workspace, workspace_bytes, hip_stream);
    if (st != KD_OK) return st;
  }
  return enqueue(p, pl, c);
}

kd_status kd_topk_kl_fwd(const kd_problem* p, const void* hidden, const void* W,
                         const int32_t* teacher_idx, const float* teacher_logit,
                         const uint8_t* ignore, float* loss, float* loss_per_token,
                         float* saved_logz, void* workspace, size_t workspace_bytes,
                         void* hip_stream) {
  kd_status st = check_problem(p);
  if (st != KD_OK) return st;
  if (loss == nullptr || (p->N > 0 && saved_logz == nullptr)) return KD_ERR_NULL_PTR;
  const Call c{KD_MODE_FWD, hidden, W, teacher_idx, teacher_logit, ignore, loss,
               loss_per_token, saved_logz, nullptr, nullptr, nullptr, nullptr, nullptr, 0,
               workspace, workspace_bytes, hip_stream};
  const Plan pl = make_plan(p);
  st = validate(p, c, pl);
  if (st != KD_OK) return st;
  if (debug_index_check() && p->N > 0) {
    st = kd_topk_kl_check_indices(p, teacher_idx, workspace, workspace_bytes, hip_stream);
    if (st != KD_OK) return st;
  }
  return enqueue(p, pl, c);
}

kd_status kd_topk_kl_bwd(const kd_problem* p, const void* hidden, const void* W,
                         const int32_t* teacher_idx, const float* teacher_logit,
                         const uint8_t* ignore, const float* saved_logz,
                         const float* grad_loss, const float* grad_loss_per_token,
                         void* grad_hidden, float* grad_W, int accumulate_grad_W,
                         void* workspace, size_t workspace_bytes, void* hip_stream) {
  kd_status st = check_problem(p);
  if (st != KD_OK) return st;
  if (p->N > 0 && saved_logz == nullptr) return KD_ERR_NULL_PTR;
  const Call c{KD_MODE_BWD, hidden, W, teacher_idx, teacher_logit, ignore, nullptr, nullptr,
               nullptr, saved_logz, grad_loss, grad_loss_per_token, grad_hidden, grad_W,
               accumulate_grad_W, workspace, workspace_bytes, hip_stream};
  const Plan pl = make_plan(p);
  st = validate(p, c, pl);
  if (st != KD_OK) return st;
  if (debug_index_check() && p->N > 0) {
    st = kd_topk_kl_check_indices(p, teacher_idx, workspace, workspace_bytes, hip_stream);
    if (st != KD_OK) return st;
  }
  return enqueue(p, pl, c);
}

kd_status kd_topk_kl_check_indices(const kd_problem* p, const int32_t* teacher_idx,
                                   void* workspace, size_t workspace_bytes, void* hip_stream) {
  kd_status st = check_problem(p);
  if (st != KD_OK) return st;
  if (workspace == nullptr || (p->N > 0 && teacher_idx == nullptr)) return KD_ERR_NULL_PTR;
  if (!aligned16(workspace)) return KD_ERR_UNSUPPORTED;
  if (workspace_bytes < kMiscBytes) return KD_ERR_WORKSPACE_TOO_SMALL;
  int* flag = reinterpret_cast<int*>(static_cast<char*>(workspace) + 8);
  int host_flag = 0;
  if (kd_launch_check_indices(teacher_idx, p->N, p->K, p->V, flag, &host_flag, hip_stream) != 0)
    return KD_ERR_DEVICE;
  return host_flag ? KD_ERR_BAD_INDEX : KD_OK;
}

static bool overlap(const void* a, int64_t an, const void* b, int64_t bn) {
  return (uintptr_t)a < (uintptr_t)b + (uintptr_t)bn && (uintptr_t)b < (uintptr_t)a + (uintptr_t)an;
}

// Checks one gradient of kd_scale_grads: in [n] fp32 -> out [n] dtype.
static kd_status check_scale(const float* in, int32_t dtype, const void* out, int64_t n) {
  if ((in == nullptr) != (out == nullptr)) return KD_ERR_NULL_PTR;
  if (n < 0) return KD_ERR_BAD_SHAPE;
  if (in == nullptr || n == 0) return KD_OK;
  if (dtype != KD_F32 && dtype != KD_BF16) return KD_ERR_UNSUPPORTED;
  if (!aligned16(in) || !aligned16(out)) return KD_ERR_UNSUPPORTED;
  // fp32 output: in place or disjoint; bf16 output: disjoint from the input
  if (overlap(in, n * 4, out, n * (dtype == KD_F32 ? 4 : 2)) && !(dtype == KD_F32 && in == out))
    return KD_ERR_BAD_ARG;
  return KD_OK;
}

kd_status kd_scale_grads(const float* grad_loss, const float* grad_hidden_f32,
                         int32_t hidden_dtype, void* grad_hidden_out, int64_t n_hidden,
                         const float* grad_W_f32, int32_t w_dtype, void* grad_W_out, int64_t n_W,
                         void* hip_stream) {
  if (grad_loss == nullptr) return KD_ERR_NULL_PTR;
  kd_status st = check_scale(grad_hidden_f32, hidden_dtype, grad_hidden_out, n_hidden);
  if (st != KD_OK) return st;
  st = check_scale(grad_W_f32, w_dtype, grad_W_out, n_W);
  if (st != KD_OK) return st;
  const KdScaleArg none{nullptr, nullptr, 0, 0};
  const KdScaleArg h{grad_hidden_f32, grad_hidden_out, grad_hidden_f32 != nullptr ? n_hidden : 0,
                     hidden_dtype == KD_BF16};
  const KdScaleArg w{grad_W_f32, grad_W_out, grad_W_f32 != nullptr ? n_W : 0, w_dtype == KD_BF16};
  // one launch, or one after the other where a gradient reads or writes what the
  // other one writes
  const int64_t hb = h.n * (h.out_bf16 ? 2 : 4), wb = w.n * (w.out_bf16 ? 2 : 4);
  const bool ordered = h.n > 0 && w.n > 0 &&
                       (overlap(h.y, hb, w.x, w.n * 4) || overlap(h.y, hb, w.y, wb) ||
                        overlap(h.x, h.n * 4, w.y, wb));
  if (kd_launch_scale(&h, ordered ? &none : &w, grad_loss, hip_stream) != 0 ||
      (ordered && kd_launch_scale(&w, &none, grad_loss, hip_stream) != 0))
    return KD_ERR_DEVICE;
  return KD_OK;
}

kd_status kd_topk_kl_fwd_bwd_noalloc(const kd_problem* p, const void* hidden, const void* W,
                                     const int32_t* teacher_idx, const float* teacher_logit,
                                     const uint8_t* ignore, float* loss, float* loss_per_token,
                                     void* grad_hidden, float* grad_W, int accumulate_grad_W,
                                     void* hip_stream) {
  kd_status st = check_problem(p);
  if (st != KD_OK) return st;
  if (loss == nullptr) return KD_ERR_NULL_PTR;
  Call c{KD_MODE_FWD_BWD, hidden, W, teacher_idx, teacher_logit, ignore, loss,
         loss_per_token, nullptr, nullptr, nullptr, nullptr, grad_hidden, grad_W,
         accumulate_grad_W, nullptr, 0, hip_stream};
  Plan pl;
  if (!plan_within(p, KD_SCRATCH_BYTES, &pl)) return KD_ERR_WORKSPACE_TOO_SMALL;
  st = validate(p, c, pl, true);
  if (st != KD_OK) return st;
  // the device's scratch array (its address is looked up once per device)
  void* ws = nullptr;
  if (kd_scratch_get(&ws) != 0 || ws == nullptr) return KD_ERR_DEVICE;
  c.ws = ws;
  c.ws_bytes = kd_scratch_bytes_max;
  if (debug_index_check() && p->N > 0) {
    int* flag = reinterpret_cast<int*>(static_cast<char*>(ws) + pl.off_misc + 8);
    int host_flag = 0;
    if (kd_launch_check_indices(teacher_idx, p->N, p->K, p->V, flag, &host_flag, hip_stream) != 0)
      return KD_ERR_DEVICE;
    if (host_flag) return KD_ERR_BAD_INDEX;
  }
  kd_launch_suppress_profiling(1);
  st = enqueue(p, pl, c);
  kd_launch_suppress_profiling(0);
  return st;
}

}  // extern "C"
