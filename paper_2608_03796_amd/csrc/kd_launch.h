// Internal interface between the host scheduler (kd_api.cpp, plain C++) and
// the HIP launchers (kd_kernels.hip). No HIP types: streams travel as void*.
#pragma once

#include <stddef.h>
#include <stdint.h>

enum { KD_MODE_FWD_BWD = 0, KD_MODE_FWD = 1, KD_MODE_BWD = 2 };

// bytes of the allocation-free entry point's static per-device scratch: the
// 256 MiB a plan without its partial tiles may count, and a slack for the
// projection's partials of 128-column vocabulary tiles above those of 256-column
// ones: 8 bytes per row (padded to 256) and 256 columns, at most 8 MiB (256 rows
// at V = 2^20; more rows only with fewer columns). Partial tiles take what is left.
constexpr size_t kd_scratch_slack = (size_t)8 << 20;
constexpr size_t kd_scratch_bytes_max = ((size_t)256 << 20) + kd_scratch_slack;

// tokens per loss partial (one block of the row-loss kernels, a wave per token)
constexpr int kLossRows = 4;

// Stages of kd_launch_chunk: preparing rows (prologue, bucketing) and the
// chunk's projection and what follows it. The host prepares the rows of a whole dW
// group at once when chunks align with 256-token tiles, else each chunk.
enum { KD_STAGE_PREP = 1, KD_STAGE_CHUNK = 2 };

struct KdChunkArgs {
  int dtype;
  int large_tiles;          // bf16: the projection's tiles that run as 256x256 (the first
                            // of the tile order; the rest as 128x128)
  int mode;                 // KD_MODE_*: which half of Algorithm 1 runs
  int stages;               // KD_STAGE_* bits
  int one_projection;       // loss and gradients together (k_logits_dz schedule)
  int teacher_logprobs;     // cached log-probabilities (partial mass) instead of logits
  const float* gscale;      // upstream gradient of the mean (device scalar) or null = 1
  const float* gtok;        // full [N] upstream per-token gradients or null
  const float* logz_in;     // full [N] saved log Z (backward only) or null
  float* logz_out;          // this chunk's rows of the saved log Z (forward; full [N]
                            // with a rowmap) or null
  int64_t D, V;
  int K;
  int64_t row0;             // first token of the chunk (of the prepared rows)
  int rows;                 // tokens in the chunk (prepared rows)
  float inv_tau;
  const void* W;            // [V, D]
  const void* Hc;           // the projection's token rows (hidden + row0 * D, or the
                            // workspace's copy of the rows' hidden rows with a rowmap)
  const void* hidden;       // full [N, D] (the reference logits read rows by token)
  const int32_t* tidx_in;   // full [N, K] (the caller's)
  int32_t* tidx;            // [rows, K] the prologue's copy (repeats -1), read by the rest
  const float* tlogit;      // full [N, K] (prologue indexes with row0)
  const uint8_t* ignore;    // full [N] or null
  const float* inv_nvalid;  // device 1/N_valid, or null: inv_n
  float inv_n;
  // ignored tokens left out (one-projection schedule): row r of the prepared
  // rows is token rowmap[r] (-1: no token; such rows come after every token),
  // and *nrow - nrow_base of the rows hold tokens. Null: row r is token row0 + r.
  const int* rowmap;
  const int* nrow;
  int nrow_base;
  // with a rowmap the prologue copies the rows' hidden rows to Hc and sets the
  // ignored tokens' outputs to 0: grad_hidden (full, or null), the full
  // loss_per_token (or null) and logz_out
  void* grad_hidden;
  int gh_f32;
  float* lpt_full;
  // per-chunk workspace
  float* p;                 // [rows, K]
  float *rowM, *rowH, *rowCoef, *rowCoefM, *rowL2;   // [rows]
  float* rowR;              // [rows] reference logit of the single projection
  int* rowFlag;             // [rows] a tile fell back to its own max
  float* rowFactor;         // [rows] factor of the row's stored gradient (this
                            // chunk's rows of the group's factor array)
  float *part_m, *part_s;   // [rows, nP]
  int nP;                   // partials per token: nVT, or 2 nVT with 128x128 tiles
  int nVT;
  uint32_t* hits;           // [cdiv(rows, 256) * 256 * K] teacher entries by vocab tile
  float* hitp;              // their p
  int* hoff;                // [cdiv(rows, 256), nVT + 1] bucket offsets
  float* zhit;              // [rows, K] student logit at each teacher entry
  void* dZ;                 // this chunk's rows of the group's dZ [rows, ldz]
  int64_t ldz;              // = padded vocabulary (columns V..ldz: finite, z = 0 there)
  // outputs
  float* loss_per_token;    // + row0 (full [N] with a rowmap), or null
  float* block_partial;     // this chunk's cdiv(rows, kLossRows) partial sums
};

// dH GEMM over the chunks of one group: grad_hidden[rows] = dZ[rows] W (the
// parts of a split launch are added up by the tail)
struct KdDhArgs {
  int dtype;
  int tile;                 // tile edge of the contraction (256 or 128; fp32: 128)
  int64_t D, V;
  const void* dZ;           // the group's dZ rows [tokens, ldz]
  int64_t ldz;
  const void* W;            // [V, D]
  int64_t tokens;           // tokens in the group
  float* partial;           // partial tiles of the split last round
  int part_space;           // their space in units of 256 bytes (0: no split)
  void* gH;                 // grad_hidden + the group's first row * D (full with a rowmap)
  int gh_f32;               // grad_hidden is fp32 (else the operands' dtype)
  const float* rowscale;    // [tokens] factor of each dZ row, or null (= 1)
  const int* rowmap;        // [tokens] grad_hidden row of each dZ row (-1: none), or null
  const int* nrow;          // with rowmap: *nrow - nrow_base dZ rows hold tokens
  int nrow_base;
};

// The contractions run in square tiles of 256 (bf16; one workgroup per compute
// unit) or 128 (fp32, and bf16 launches of few tiles; two workgroups per
// compute unit): the workgroups the chip runs at once.
constexpr int kd_units(int64_t tile) { return tile == 256 ? 256 : 512; }

// How the tiles of dH and dW run: those of the full rounds whole (`dp` of them),
// the `rem` tiles left over for the last round each split into `split` ranges
// of their K (the vocabulary or the tokens), whose fp32 partial tiles are added
// up afterwards (dH's by the tail launch, dW's by k_dw_fixup). The split is the
// one with the least time by a model in K steps of a tile: a round costs its
// longest range plus kSplitRound steps (pipeline fill and epilogue), a partial
// tile its write and read, and adding the parts up kSplitRound more. Splitting
// only the last round keeps the partial traffic small. Whole calls, against
// splitting every dH tile to fill the rounds: 6001 tokens, D = 2560, V = 40001
// (240 tiles) 3.26 and 2.90 ms; 77 tokens, D = 768, V = 32003 (3 tiles) 126 and
// 109 us; dW of few tiles unsplit: 4000 tokens, D = 256, V = 4096 105 and 91
// us. Evaluated on the device where the number of rows is only known there
// (ignored tokens left out). At most max_parts partial tiles, and at most two
// rounds of them (their traffic).
// The model is in integers (1024ths of a K step), so that host and device choose
// alike.
#ifdef __HIP__
#define KD_HOST_DEVICE __host__ __device__
#else
#define KD_HOST_DEVICE
#endif
constexpr int kSplitRound = 4 * 1024;
constexpr int kSplitMax = 64;
struct KdRounds {
  int dp, rem, split;
};
// the model's time of `rem` tiles in s ranges each, INT_MAX if s is too many
KD_HOST_DEVICE inline int kd_split_time(int s, int rem, int ksteps, int units, int part_cost,
                                        int max_parts) {
  if (s == 1) return ksteps * 1024 + kSplitRound;
  const int parts = rem * s;
  if (parts > max_parts || parts > 2 * units || ksteps < 4 * s) return 0x7fffffff;
  return (parts > units ? 2 : 1) * ((ksteps + s - 1) / s * 1024 + kSplitRound) + parts * part_cost +
         kSplitRound;
}
inline KdRounds kd_split_rounds(int tiles, int ksteps, int units, int part_cost, int max_parts) {
  KdRounds r;
  r.dp = tiles / units * units;
  r.rem = tiles - r.dp;
  r.split = 1;
  if (r.rem == 0) return r;
  int best = kd_split_time(1, r.rem, ksteps, units, part_cost, max_parts);
  for (int s = 2; s <= kSplitMax; ++s) {
    const int t = kd_split_time(s, r.rem, ksteps, units, part_cost, max_parts);
    if (t == 0x7fffffff) break;  // and so for more ranges
    if (t < best) {
      best = t;
      r.split = s;
    }
  }
  return r;
}
// 1024ths of a tile's K step that one partial tile's write and read cost (a 256
// KB partial tile against 1.44 us, a 64 KB one against 2 us (fp32) or 0.65 us)
constexpr int kd_part_cost(int tile, bool f32) { return tile == 256 ? 82 : f32 ? 15 : 46; }

// The most partial tiles of dH over n token rows, D features, in `space` units of
// 256 bytes. Where all tiles are split (no full rounds), a range's partial
// tiles are stored as one [n, D] array, without the padding of the tiles; else
// each is TS x TS on its own.
KD_HOST_DEVICE inline int kd_dh_max_parts(int tiles, int n, int D, int tile, int space) {
  if (tiles >= kd_units(tile)) return space / (tile * tile / 64);
  const int fit = n > 0 ? space / (n * (D / 64)) : 0;  // ranges
  return tiles * (fit < kSplitMax ? fit : kSplitMax);
}
inline KdRounds kd_dh_rounds(int n, int D, int tile, int ksteps, bool f32, int space) {
  const int tiles = (n + tile - 1) / tile * ((D + tile - 1) / tile);
  return kd_split_rounds(tiles, ksteps, kd_units(tile), kd_part_cost(tile, f32),
                         kd_dh_max_parts(tiles, n, D, tile, space));
}

// Workgroups of a dH launch over `tokens` rows of which the device may find any
// number to hold tokens: the most any count needs (the fewest rows of a tile row
// leave room for the most ranges).
inline int kd_dh_blocks(int tokens, int D, int tile, int ksteps, bool f32, int space) {
  const int units = kd_units(tile), td = (D + tile - 1) / tile;
  int blocks = 0;
  for (int tm = (tokens + tile - 1) / tile; tm > 0; --tm) {
    // (full rounds and at most two of parts: no fewer rows need more)
    if (tm * td / units * units + 2 * units <= blocks) break;
    const KdRounds r = kd_dh_rounds((tm - 1) * tile + 1, D, tile, ksteps, f32, space);
    if (r.dp + r.rem * r.split > blocks) blocks = r.dp + r.rem * r.split;
  }
  return blocks;
}

// the most parts of a split dW tile that k_dw_fixup has in flight at a time
constexpr int kDwMaxSplit = 4;

// dW GEMM over the chunks of one group: grad_W (+)= dZ[:tokens]^T H[:tokens]
struct KdDwArgs {
  int dtype;
  int tile;                 // tile edge of the contraction (256 or 128; fp32: 128)
  int64_t D, V;
  const void* dZ;           // the group's dZ rows [tokens, ldz]
  int64_t ldz;
  int64_t tokens;           // tokens in the group
  const void* Ht;           // the tail's transposed hidden rows: [D, tokens rounded up to 64]
  int beta;                 // 0 overwrite, 1 accumulate
  float* gW;
  float* partial;           // partial tiles of the split last round
  int max_parts;            // their number (0: no split)
  const int* nrow;          // ignored tokens left out: the dZ rows [0, *nrow) hold tokens;
                            // or null
};

// Between a group's dH and dW: hidden rows transposed (Ht not null), the parts
// of a split dH added up (dh not null), the loss (loss not null)
struct KdTailArgs {
  int dtype;
  int64_t D;
  const void* Hg;           // the group's hidden rows [tokens, D] (full with a rowmap)
  int64_t tokens;
  void* Ht;                 // [D, tokens rounded up to 64], or null
  const float* rowscale;    // [tokens] factor of each dZ row (applied to the
                            // hidden rows), or null (= 1)
  const int* rowmap;        // [tokens] hidden row of each dZ row (-1: none), or null
  const KdDhArgs* dh;       // the dH launch whose parts are to be added up, or null
  const float* block_partial;
  int n_partials;
  const float* inv_nvalid;  // device 1/N_valid, or null: inv_n
  float inv_n;
  float* loss;
};

// Ignored tokens of one dW group [row0, row0 + rows) left out: rowmap[j] =
// the j-th token not ignored (then -1), *nrow = their count; with inv_nvalid
// also 1/N_valid of the whole mask.
struct KdCompactArgs {
  const uint8_t* ignore;    // full [N]
  int64_t N;
  int64_t row0;
  int rows;
  int* rowmap;
  int* nrow;
  float* inv_nvalid;        // or null
};

// out = g x for one gradient: x fp32, out fp32 or bf16, n elements (0: nothing)
struct KdScaleArg {
  const float* x;
  void* y;
  int64_t n;
  int out_bf16;
};

extern "C" {
int kd_launch_fill(float* p, int64_t n, void* stream);  // n zeros
int kd_launch_chunk(const KdChunkArgs* a, void* stream);
int kd_launch_dh(const KdDhArgs* a, void* stream);
int kd_launch_dw(const KdDwArgs* a, void* stream);
int kd_launch_compact(const KdCompactArgs* a, void* stream);
int kd_launch_tail(const KdTailArgs* a, void* stream);
int kd_launch_scale(const KdScaleArg* a, const KdScaleArg* b, const float* g, void* stream);
// the current device's scratch address (hipGetSymbolAddress on first use)
int kd_scratch_get(void** ptr);
// nonzero: the calling thread's launches record no profiling events
void kd_launch_suppress_profiling(int on);
int kd_launch_check_indices(const int32_t* idx, int64_t N, int K, int64_t V, int* flag,
                            int* host_flag, void* stream);
}
