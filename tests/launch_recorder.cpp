// The launchers of kd_launch.h without a device: they record what the host
// schedule (kd_api.cpp, compiled next to this file) would launch. Pointers are
// never dereferenced.
#include <vector>

#include "../paper_2608_03796_amd/csrc/kd_launch.h"

namespace {
// kind 3: a launch of kd_scale_grads, its two element counts
// one launch of dH (kind 1) or dW (kind 2): its token rows, tile edge, whole
// tiles, tiles and parts of the split last round, K steps, the bytes its partial
// tiles may take, and the scratch bytes up to the end of these
struct Rec {
  int64_t kind, tokens, tile, dp, rem, split, ksteps, part_bytes, part_end;
};
std::vector<Rec> recs;
char* const kScratch = reinterpret_cast<char*>((uintptr_t)1 << 40);

void record(int64_t kind, int64_t tokens, int64_t tile, const KdRounds& r, int64_t ksteps,
            int64_t part_bytes, const float* partial) {
  const int64_t at = part_bytes > 0 ? reinterpret_cast<const char*>(partial) - kScratch : 0;
  recs.push_back({kind, tokens, tile, r.dp, r.rem, r.split, ksteps, part_bytes, at + part_bytes});
}
}  // namespace

extern "C" {
int rec_count() { return (int)recs.size(); }
void rec_clear() { recs.clear(); }
void rec_get(int i, int64_t* out) {
  const Rec& r = recs[i];
  const int64_t v[9] = {r.kind, r.tokens, r.tile, r.dp, r.rem, r.split, r.ksteps, r.part_bytes,
                        r.part_end};
  for (int k = 0; k < 9; ++k) out[k] = v[k];
}
// the bytes of partial tiles that dH over n rows takes of the `part_bytes` it has
int64_t rec_dh_bytes(int n, int D, int tile, int ksteps, int f32, int64_t part_bytes) {
  const KdRounds r = kd_dh_rounds(n, D, tile, ksteps, f32 != 0, (int)(part_bytes / 256));
  if (r.split < 2) return 0;
  return 4 * (int64_t)r.split * (r.dp == 0 ? (int64_t)n * D : (int64_t)r.rem * tile * tile);
}

// dH over 0..tokens rows: 0 if every count's workgroups and partial tiles stay
// within the launch's and the model's choice is the least of all numbers of
// ranges (as a wave takes it on the device), else a count for which one fails, + 1
int rec_dh_counts(int tokens, int D, int tile, int ksteps, int f32, int space) {
  const int blocks = kd_dh_blocks(tokens, D, tile, ksteps, f32 != 0, space);
  const int units = kd_units(tile), cost = kd_part_cost(tile, f32 != 0);
  for (int n = 0; n <= tokens; ++n) {
    const KdRounds r = kd_dh_rounds(n, D, tile, ksteps, f32 != 0, space);
    if (r.dp + r.rem * r.split > blocks) return n + 1;
    const int64_t bytes =
        4 * (int64_t)r.split * (r.dp == 0 ? (int64_t)n * D : (int64_t)r.rem * tile * tile);
    if (r.split > 1 && bytes > (int64_t)space * 256) return n + 1;
    const int tiles = r.dp + r.rem, parts = kd_dh_max_parts(tiles, n, D, tile, space);
    int best = 1;
    for (int s = 2; s <= kSplitMax; ++s)
      if (kd_split_time(s, r.rem, ksteps, units, cost, parts) <
          kd_split_time(best, r.rem, ksteps, units, cost, parts))
        best = s;
    if (r.rem > 0 && best != r.split) return n + 1;
  }
  return 0;
}

int kd_launch_fill(float*, int64_t, void*) { return 0; }
int kd_launch_chunk(const KdChunkArgs*, void*) { return 0; }
int kd_launch_compact(const KdCompactArgs*, void*) { return 0; }
int kd_launch_tail(const KdTailArgs*, void*) { return 0; }
int kd_launch_scale(const KdScaleArg* a, const KdScaleArg* b, const float*, void*) {
  recs.push_back({3, a->n, b->n, 0, 0, 0, 0, 0, 0});
  return 0;
}
int kd_launch_dh(const KdDhArgs* a, void*) {
  const int eb = a->dtype == 1 ? 2 : 4, ksteps = (int)(a->ldz * eb / 128);
  record(1, a->tokens, a->tile,
         kd_dh_rounds((int)a->tokens, (int)a->D, a->tile, ksteps, eb == 4, a->part_space), ksteps,
         (int64_t)a->part_space * 256, a->partial);
  return 0;
}
int kd_launch_dw(const KdDwArgs* a, void*) {
  const int eb = a->dtype == 1 ? 2 : 4, ts = a->tile;
  const int ksteps = (int)((a->tokens + 63) / 64 * 64 * eb / 128);
  const int tiles = (int)((a->D + ts - 1) / ts * ((a->V + ts - 1) / ts));
  record(2, a->tokens, ts,
         kd_split_rounds(tiles, ksteps, kd_units(ts), kd_part_cost(ts, eb == 4), a->max_parts),
         ksteps, (int64_t)a->max_parts * ts * ts * 4, a->partial);
  return 0;
}
int kd_scratch_get(void** ptr) {
  *ptr = kScratch;
  return 0;
}
void kd_launch_suppress_profiling(int) {}
int kd_launch_check_indices(const int32_t*, int64_t, int, int64_t, int*, int* host_flag, void*) {
  *host_flag = 0;
  return 0;
}
}
