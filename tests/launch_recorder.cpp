// The launchers of kd_launch.h without a device: they record what the host
// schedule (kd_api.cpp, compiled next to this file) would launch. Pointers are
// never dereferenced.
#include <vector>

#include "../paper_2608_03796_amd/csrc/kd_launch.h"

namespace {
// one launch of dH (kind 1) or dW (kind 2): its token rows, tile edge, whole
// tiles, tiles and parts of the split last round, K steps, the most partial
// tiles it may use, and the scratch bytes up to the end of these
struct Rec {
  int64_t kind, tokens, tile, dp, rem, split, ksteps, max_parts, part_end;
};
std::vector<Rec> recs;
char* const kScratch = reinterpret_cast<char*>((uintptr_t)1 << 40);

int64_t tiles(int64_t a, int64_t b, int64_t ts) { return (a + ts - 1) / ts * ((b + ts - 1) / ts); }
void record(int64_t kind, int64_t tokens, int64_t tile, int64_t n_tiles, int64_t ksteps, bool f32,
            int max_parts, const float* partial) {
  const KdRounds r = kd_split_rounds((int)n_tiles, (int)ksteps, kd_units(tile),
                                     kd_part_cost((int)tile, f32), max_parts);
  const int64_t end =
      max_parts > 0
          ? (int64_t)(reinterpret_cast<const char*>(partial) - kScratch) + max_parts * tile * tile * 4
          : 0;
  recs.push_back({kind, tokens, tile, r.dp, r.rem, r.split, ksteps, max_parts, end});
}
}  // namespace

extern "C" {
int rec_count() { return (int)recs.size(); }
void rec_clear() { recs.clear(); }
void rec_get(int i, int64_t* out) {
  const Rec& r = recs[i];
  const int64_t v[9] = {r.kind, r.tokens, r.tile, r.dp, r.rem, r.split, r.ksteps, r.max_parts,
                        r.part_end};
  for (int k = 0; k < 9; ++k) out[k] = v[k];
}
// the most partial tiles the device may use for any count of token rows
int64_t rec_model_parts(int64_t n_tiles, int64_t ksteps, int64_t tile, int f32, int max_parts) {
  const KdRounds r = kd_split_rounds((int)n_tiles, (int)ksteps, kd_units(tile),
                                     kd_part_cost((int)tile, f32 != 0), max_parts);
  return r.split > 1 ? r.rem * r.split : 0;
}

int kd_launch_fill(float*, int64_t, void*) { return 0; }
int kd_launch_chunk(const KdChunkArgs*, void*) { return 0; }
int kd_launch_compact(const KdCompactArgs*, void*) { return 0; }
int kd_launch_tail(const KdTailArgs*, void*) { return 0; }
int kd_launch_scale(const KdScaleArg*, const KdScaleArg*, const float*, void*) { return 0; }
int kd_launch_dh(const KdDhArgs* a, void*) {
  const int eb = a->dtype == 1 ? 2 : 4;
  record(1, a->tokens, a->tile, tiles(a->tokens, a->D, a->tile), a->ldz * eb / 128, eb == 4,
         a->max_parts, a->partial);
  return 0;
}
int kd_launch_dw(const KdDwArgs* a, void*) {
  const int eb = a->dtype == 1 ? 2 : 4;
  record(2, a->tokens, a->tile, tiles(a->D, a->V, a->tile), (a->tokens + 63) / 64 * 64 * eb / 128,
         eb == 4, a->max_parts, a->partial);
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
