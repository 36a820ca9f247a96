// HIP kernels (gfx950) of the fused chunked top-K KL loss and their launchers.
//
// Per group of chunks, with a mask:
//              compact_scan      -> the group's tokens that are not ignored (row map,
//                                   count); the kernels below skip the rows past
//                                   them. The first one also counts N_valid.
// Per chunk:   prep              -> per row p, M, H, g/tau          (§3.2, Eq. 2 terms),
//                                   its hidden row copied next to the others'
//                                   (with a mask), the reference logit R; teacher
//                                   entries grouped by vocabulary tile (in launches
//                                   of their own, prologue and bucket, for K > 128
//                                   and for the separate backward)
//   loss and gradients together (one projection per chunk):
//              logits_dz         -> (reference, sum-exp) partials per (token, vocab
//                                   tile), z at the teacher entries, dZ'' = 2^(y - R)
//              row_finish        -> log Z, the row factor (g/tau) M 2^(R - log2 Z),
//                                   fallback rows, teacher cells (Eq. 3) / factor,
//                                   l_t = H - C/tau + M log Z       (Eq. 2)
//   forward only:  logits_lse (with z at the teacher entries), lse_merge, row_loss
//   backward only: dz            -> recomputed logits, dZ = g/tau (M q - p)
//              dh                -> dH = dZ W (per chunk or per group; rows scaled
//                                   by the factor in the one-projection schedule)
// Per group of chunks: tail      -> dH's split parts added up, the hidden rows
//                                   transposed, the loss (mean over non-ignored
//                                   tokens) after the last chunk
//              dw                -> grad_W (+)= dZ^T H (fp32 accumulate)
//
// A kernel of a few microseconds of work occupies the stream for about 4.7 us,
// so the small passes share launches where nothing orders them: a step of one
// group is 6 launches, which were 11, and one more each with a mask, for K > 128
// (prologue and buckets apart), where the projection's last tiles run as small ones
// and where dW's last round is split (fixup).
#include "kd_device.h"
#include "kd_f32.h"
#include <type_traits>
#include "kd_launch.h"

#include <string.h>

namespace kd {

// ------------------------------------------------------------------ small --
__global__ void k_fill_f32(float* p, int64_t n, float v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// Prepares each row, one wave per row.
//
// Teacher distribution over the K cached entries (§3.2):
// p = softmax(teacher_logit / tau), or p = exp(value) as given for cached
// log-probabilities (partial mass); M = sum p, H = sum p log p (0 log 0 = 0).
// Row weight coef = g/tau, g = 1/N_valid times the upstream gradient of the
// mean (gscale, default 1), or the upstream gradient of the token's own loss
// (gtok); 0 for ignored rows. With a saved log-normaliser (backward only) the
// row's log2 Z is set from it. With a rowmap, row r is token rowmap[r], whose
// hidden row is copied to hcomp's row r; a row without a token (-1) gets
// p = 0, index -1 and weight 0; and if token row0 + r is ignored, its
// grad_hidden row, per-token loss and saved log Z are set to 0 (the rest of
// the call never writes them).
//
// The support is a set; a row that repeats an index is read as the dense
// teacher row that sums the repeated entries (scatter-add): the first
// occurrence carries the sum of their probabilities (in entry order), H takes
// P log P of that sum, and the later occurrences get p = 0 and the index -1 in
// tidx_out, the row's copy of its indices that every later kernel reads (an
// index outside [0, V) is skipped everywhere). Rows without repeats are
// unchanged. Repeats are found with a hash set of the row's indices in LDS
// (an insertion that meets its own index); only a wave in which some row
// repeats an index compares the row's entries pairwise, in entry order.
//
// With rowR (one-projection schedule), the row's reference logit for
// k_logits_dz: R = z log2(e)/tau at the teacher entry with the largest
// teacher logit (a valid index), plus kRefShift; -inf when the row has no
// valid index. The logit part never exceeds the row's max y beyond rounding,
// so 2^(y - R) keeps every term that matters; a tile whose sum of 2^(y - R)
// exceeds 2^kRefGap falls back to its own max. The row's fallback flag is
// cleared.
//
// LDS hash set of the row's valid indices (power-of-two slots, at least K):
// size in ints for K entries
__host__ __device__ constexpr int prologue_hash_slots(int K) {
  int t = 64;
  while (t < 2 * K && t < 4096) t *= 2;
  return t;
}

// largest exponent (base 2) of the sum of a tile row's stored provisional
// gradients 2^(y - R), and so of each of them
constexpr float kRefGap = 40.f;
constexpr float kRefGapScale = 1099511627776.f;  // 2^kRefGap
// R is the reference logit plus this many (base 2): stored values are then
// smaller, which the dH and dW contractions run about 1% faster on (MFMA power
// depends on the operands); terms below 2^-126 relative to R + kRefShift,
// i.e. 2^-102 below the reference logit, flush to zero
constexpr float kRefShift = 24.f;

constexpr int prologue_lds(int K) { return 4 * prologue_hash_slots(K) + 8 * K; }

struct PrologueArgs {
  const int32_t* tidx;
  int32_t* tidx_out;
  const float* tlogit;
  const uint8_t* ignore;
  int64_t row0;
  const int* rowmap;
  int rows, K, V, D;
  float inv_tau;
  int logprobs;
  const float* inv_nvalid;  // device 1/N_valid, or null: inv_n
  float inv_n;
  const float *gscale, *gtok, *logz_in;
  float *p_out, *rowM, *rowH, *rowCoef, *rowCoefM, *rowL2;
  // one-projection schedule (rowR not null)
  const void *hidden, *W;
  float k2;
  float* rowR;
  int* rowFlag;
  // with a rowmap
  char* hcomp;
  char* gH;
  int64_t gh_row_bytes;
  float *lpt, *logz_out;
};

// LDS accesses of one wave stay in order: only the compiler is held back
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// row r by the calling wave, with prologue_lds(K) bytes of LDS of its own
template <typename T>
__device__ __forceinline__ void prologue_row(const PrologueArgs& a, int r, char* lds) {
  const int K = a.K, V = a.V;
  const int S = prologue_hash_slots(K);
  int* hset = reinterpret_cast<int*>(lds);
  int* sidx = hset + S;
  float* sp = reinterpret_cast<float*>(sidx + K);
  const int lane = threadIdx.x & 63;
  if (r >= a.rows) return;
  int64_t t = a.row0 + r;
  if (a.rowmap != nullptr) {
    if (a.ignore[t] != 0) {
      if (a.gH != nullptr) {
        u32x4_t* z = reinterpret_cast<u32x4_t*>(a.gH + t * a.gh_row_bytes);
        for (int64_t q = lane; q < a.gh_row_bytes / 16; q += 64) z[q] = u32x4_t{0u, 0u, 0u, 0u};
      }
      if (lane == 0) {
        if (a.lpt != nullptr) a.lpt[t] = 0.f;
        if (a.logz_out != nullptr) a.logz_out[t] = 0.f;
      }
    }
    t = a.rowmap[r];
  }
  float* p_out = a.p_out + (int64_t)r * K;
  int32_t* tidx_out = a.tidx_out + (int64_t)r * K;
  if (t < 0) {
    for (int k = lane; k < K; k += 64) {
      p_out[k] = 0.f;
      tidx_out[k] = -1;
    }
    if (lane == 0) {
      a.rowM[r] = 0.f;
      a.rowH[r] = 0.f;
      a.rowCoef[r] = 0.f;
      a.rowCoefM[r] = 0.f;
      if (a.logz_in != nullptr) a.rowL2[r] = 0.f;
      if (a.rowR != nullptr) {
        a.rowR[r] = -INFINITY;
        a.rowFlag[r] = 0;
      }
    }
    return;
  }
  constexpr int VPT = 16 / (int)sizeof(T);  // elements per 16-byte piece
  const T* hrow = static_cast<const T*>(a.hidden) + t * a.D;
  if (a.rowmap != nullptr) {
    const u32x4_t* src = reinterpret_cast<const u32x4_t*>(hrow);
    u32x4_t* dst = reinterpret_cast<u32x4_t*>(a.hcomp + (int64_t)r * a.D * sizeof(T));
#pragma unroll 4
    for (int q = lane; q < a.D / VPT; q += 64) dst[q] = src[q];
  }
  const float* u = a.tlogit + t * (int64_t)K;
  const int32_t* ix = a.tidx + t * (int64_t)K;
  for (int i = lane; i < S; i += 64) hset[i] = -1;
  float mx = 0.f, logs = 0.f, scale = 1.f;
  if (!a.logprobs) {
    mx = -INFINITY;
    for (int k = lane; k < K; k += 64) mx = fmaxf(mx, u[k] * a.inv_tau);
    mx = wave_max(mx);
    float s = 0.f;
    for (int k = lane; k < K; k += 64) s += expf(u[k] * a.inv_tau - mx);
    s = wave_sum(s);
    logs = logf(s);
    scale = a.inv_tau;
  }
  wave_lds_sync();  // the cleared hash set
  // p, and the row's indices into the hash set: an insertion that finds its
  // own index already there has seen a repeat (invalid indices are skipped
  // by every kernel and take no part)
  float m = 0.f;
  bool seen = false;
  for (int k = lane; k < K; k += 64) {
    const float pk = expf(u[k] * scale - mx - logs);
    const int v = ix[k];
    sidx[k] = v;
    sp[k] = pk;
    m += pk;
    if ((unsigned)v < (unsigned)V) {
      uint32_t h = ((uint32_t)v * 2654435761u) >> 7;
      for (int probe = 0; probe < S; ++probe, ++h) {
        const int prev = atomicCAS(&hset[h & (S - 1)], -1, v);
        if (prev == -1) break;
        if (prev == v) {
          seen = true;
          break;
        }
      }
    }
  }
  const bool any_repeat = __builtin_amdgcn_ballot_w64(seen) != 0ull;
  wave_lds_sync();  // sidx and sp of the whole row
  float h = 0.f;
  float best = -INFINITY;  // the valid entry with the largest teacher logit, the first of equals
  int bk = K;
  for (int k = lane; k < K; k += 64) {
    const int v = sidx[k];
    const float pk = sp[k];
    bool dup = false;
    float acc = pk;
    if (any_repeat) {
      // rare: an entry repeats an earlier index (p = 0, index -1) or is the
      // first of repeats (their probabilities summed in entry order)
      if ((unsigned)v < (unsigned)V) {
        for (int j = 0; j < K; ++j) {
          if (j != k && sidx[j] == v) {
            if (j < k) dup = true;
            else acc += sp[j];
          }
        }
      }
    }
    const float uk = u[k];
    const float lp = uk * scale - mx - logs;
    float pe = pk, term = pk > 0.f ? pk * lp : 0.f;
    if (dup) {
      pe = 0.f;
      term = 0.f;
    } else if (acc != pk) {
      pe = acc;
      term = acc > 0.f ? acc * logf(acc) : 0.f;
    }
    p_out[k] = pe;
    tidx_out[k] = dup ? -1 : v;
    h += term;
    if (!dup && (unsigned)v < (unsigned)V && (uk > best || (uk == best && k < bk))) {
      best = uk;
      bk = k;
    }
  }
  m = wave_sum(m);
  h = wave_sum(h);
  if (lane == 0) {
    const bool valid = a.ignore == nullptr || a.ignore[t] == 0;
    const float inv_n = a.inv_nvalid != nullptr ? a.inv_nvalid[0] : a.inv_n;
    const float g =
        a.gtok != nullptr ? a.gtok[t] : inv_n * (a.gscale != nullptr ? a.gscale[0] : 1.f);
    const float coef = valid ? a.inv_tau * g : 0.f;
    a.rowM[r] = m;
    a.rowH[r] = h;
    a.rowCoef[r] = coef;
    a.rowCoefM[r] = coef * m;
    if (a.logz_in != nullptr) a.rowL2[r] = a.logz_in[t] * kLog2e;
  }
  if (a.rowR == nullptr) return;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float ob = __shfl_xor(best, o);
    const int ok = __shfl_xor(bk, o);
    if (ob > best || (ob == best && ok < bk)) {
      best = ob;
      bk = ok;
    }
  }
  float z = 0.f;
  if (bk < K) {
    // 16-byte pieces of both rows (D is a multiple of 64, rows 16-byte aligned)
    const T* w = static_cast<const T*>(a.W) + (int64_t)sidx[bk] * a.D;
#pragma unroll 4
    for (int d = lane * VPT; d < a.D; d += 64 * VPT) {
      const u32x4_t hv = *reinterpret_cast<const u32x4_t*>(hrow + d);
      const u32x4_t wv = *reinterpret_cast<const u32x4_t*>(w + d);
      T he[VPT], we[VPT];
      __builtin_memcpy(he, &hv, 16);
      __builtin_memcpy(we, &wv, 16);
#pragma unroll
      for (int x = 0; x < VPT; ++x) z += (float)he[x] * (float)we[x];
    }
    z = wave_sum(z);
  }
  if (lane == 0) {
    a.rowR[r] = bk < K ? z * a.k2 + kRefShift : -INFINITY;
    a.rowFlag[r] = 0;
  }
}

// ------------------------------------------------------- contraction core --
// One TS x TS tile of the contraction: bf16 operands in 256x256 tiles
// (gemm_tile) or, for launches of few tiles, in 128x128 tiles (gemm_small);
// fp32 operands in 128x128 tiles of split bf16 (gemm_f32). LDS bytes: gemm_lds.
template <typename T, int TS, bool SPREAD, typename OA, typename OB>
__device__ __forceinline__ void gemm(const OA& a, const OB& b, int kb, int ke, char* lds,
                                     AccTile<TS>& acc) {
  if constexpr (TS == 256) gemm_tile<OA, OB, SPREAD>(a, b, kb, ke, lds, acc);
  else if constexpr (sizeof(T) == 2) gemm_small<OA, OB>(a, b, kb, ke, lds, acc);
  else gemm_f32<OA, OB>(a, b, kb, ke, lds, acc);
}
template <typename T, int TS>
constexpr int gemm_lds = TS == 256 ? kLdsA3 : sizeof(T) == 2 ? kLdsSmall : kLdsF32;

// The tiles of a projection launch: part [first, first + count) of the order of
// the projection's TM x TN tiles of 256x256, whole (TS = 256) or as four
// 128x128 tiles each. Every token has nP (reference, sum) partials, one per
// 256 or per 128 vocabulary columns.
struct ProjTiles {
  int TM, TN, first, count, nP;
};
template <int TS>
__device__ __forceinline__ void proj_tile(const ProjTiles& p, int& m0, int& n0) {
  int mt, nt;
  if constexpr (TS == 256) {
    tile_at(p.first + tile_order_xcd(blockIdx.x, p.count), p.TM, p.TN, 4, mt, nt);
    m0 = mt * 256;
    n0 = nt * 256;
  } else {
    const int q = tile_order_xcd(blockIdx.x, 4 * p.count);
    tile_at(p.first + (q >> 2), p.TM, p.TN, 4, mt, nt);
    m0 = mt * 256 + 128 * (q & 1);
    n0 = nt * 256 + 128 * ((q >> 1) & 1);
  }
}
// token t's partial of the tile at column m0; `none` completes a 256-column
// tile's two 128-column partials
template <int TS>
__device__ __forceinline__ void put_partial(const ProjTiles& p, float* pm, float* ps, int64_t t,
                                            int m0, float ref, float sum, float none) {
  const bool fine = p.nP != p.TM;
  const int64_t o = t * p.nP + (m0 >> (fine ? 7 : 8));
  pm[o] = ref;
  ps[o] = sum;
  if (TS == 256 && fine) {
    pm[o + 1] = none;
    ps[o + 1] = 0.f;
  }
}

// Epilogues of the projection kernels stage the fp32 tile in LDS half of its
// tokens at a time, as [token][vocab] rows of TS floats with a 16-byte-slot
// swizzle.
template <int TS>
constexpr int stage_bytes = TS / 2 * TS * 4;  // 128 KiB or 32 KiB
__device__ __forceinline__ int hsw16(int n) { return (n ^ (n >> 3)) & 15; }
template <int TS>
__device__ __forceinline__ float* stage_cell(float* st, int n, int v) {
  return st + n * TS + ((((v >> 2) ^ hsw16(n)) << 2) | (v & 3));
}
// the waves holding half h's tokens write it
template <int TS>
__device__ __forceinline__ void stage_half(float* st, const AccTile<TS>& acc, int h, int wm, int wn,
                                           int lane) {
  typedef Geo<TS> G;
  if (wn / (G::NW / 4) != h) return;
#pragma unroll
  for (int i = 0; i < G::NI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = G::acc_n(wn, j, lane) & (TS / 2 - 1);  // token row of the half
      const int vl = G::acc_m(wm, i, lane, 0);             // 4 consecutive vocab
      *reinterpret_cast<f32x4_t*>(stage_cell<TS>(st, n, vl)) = acc.v[i][j];
    }
}
// The teacher entries of a tile: the bucket of the 256x256 tile that holds it.
// An entry's token and column within the TS x TS tile at (m0, n0); false when
// it lies in another part of the 256x256 tile.
template <int TS>
__device__ __forceinline__ bool entry_cell(uint32_t e, int m0, int n0, int& tl, int& v) {
  tl = (int)(e & 255u) - (n0 & 255);
  v = (int)((e >> 8) & 255u) - (m0 & 255);
  return TS == 256 || ((unsigned)tl < (unsigned)TS && (unsigned)v < (unsigned)TS);
}

// f(entry, p) for the entries of a tile's bucket past the first one of each thread
// (p null: 0). Each is a load and what depends on it, one latency after the
// other: a small tile, whose bucket is that of four tiles, loads four at a time.
// Where the entries crowd few vocabulary tiles (190 x 128 x 351, K = 351) the
// projection took 94 us one by one, now 54 (eight at a time 43, but their code cost
// every other small launch 0.5 to 1 us).
template <int TS, typename F>
__device__ __forceinline__ void rest_entries(int tid, int cnt, const uint32_t* __restrict__ hits,
                                             const float* __restrict__ hitp, F f) {
  constexpr int U = TS == 128 ? 4 : 1, TH = Geo<TS>::kThreads;
  if (__builtin_expect(cnt <= TH, 1)) return;
  for (int q = TH + tid; q < cnt; q += U * TH) {
    uint32_t e[U];
    float p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(q + u * TH, cnt - 1);
      e[u] = hits[i];
      p[u] = hitp != nullptr ? hitp[i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (q + u * TH < cnt) f(e[u], p[u]);
  }
}

// ------------------------------------------------- logits + online LSE -----
// Tile of z^T = W H_c^T (M = vocabulary, N = chunk tokens). Each lane holds 32
// vocabulary values of 4 tokens; the per-token max and sum of 2^(y - max) of
// y = z log2(e)/tau are reduced in registers, across the four lane groups of
// the wave, and across the two waves sharing the tokens through LDS. Output per (token,
// vocabulary tile): (max, sum) in base-2 units.
//
// With zhit set (forward-only calls, which have no logit recompute), the tile
// also records z at its teacher entries for C = sum_k p z (Eq. 2), in O(1)
// per entry: the entries of the tile's bucket mark a 256 x 256 bit map of
// cells (token, column) in LDS; an exclusive prefix sum of the words' bit
// counts numbers the marked cells; the lane holding a marked cell stores its
// z at that number in an LDS array; then every entry reads the z of its cell.
// A tile with more marked cells than the array holds (a teacher whose
// entries crowd one vocabulary tile) has the holders of the excess cells
// search the bucket for their entries instead.
constexpr int kZhBits = 0;                      // LDS: 256 tokens x 8 words
constexpr int kZhPre = 8192;                    // exclusive prefix per word
constexpr int kZhWs = 16384;                    // per-wave totals of the scan
constexpr int kZhVal = 16384 + 64;              // z of the marked cells
constexpr int kZhCap = (kLdsA3 - 32768 - kZhVal) / 4; // 28656 cells

template <typename T, int TS>
__global__ __launch_bounds__(Geo<TS>::kThreads, TS == 256 ? 1 : 2) void k_logits_lse(const T* __restrict__ W,
                                                            const T* __restrict__ Hc, int D,
                                                            int V, int rows, ProjTiles tiles,
                                                            float k2, float* part_m,
                                                            float* part_s, int nVT,
                                                            const uint32_t* __restrict__ hits,
                                                            const int* __restrict__ hoff, int K,
                                                            float* zhit,
                                                            const int* __restrict__ nrow,
                                                            int nrow_base) {
  typedef Geo<TS> G;
  __shared__ __attribute__((aligned(16))) char lds[gemm_lds<T, TS>];
  int m0, n0;
  proj_tile<TS>(tiles, m0, n0);
  const int eb = Elt<T>::bytes;
  const int ld = D * eb;
  // with ignored tokens left out only the first *nrow - nrow_base rows hold
  // tokens (as in k_logits_dz)
  int trows = rows;
  if (nrow != nullptr) trows = min(rows, __builtin_amdgcn_readfirstlane(*nrow) - nrow_base);
  if (n0 >= trows) return;
  const int mrows = max(0, min(TS, V - m0)), nrows = min(TS, trows - n0);
  AccTile<TS> acc;
  gemm<T, TS, false>(
      KcOp{reinterpret_cast<const char*>(W + (int64_t)m0 * D), (uint32_t)(mrows * ld), ld},
      KcOp{reinterpret_cast<const char*>(Hc + (int64_t)n0 * D), (uint32_t)(nrows * ld), ld}, 0,
      ld / kRowB, lds, acc);

  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);
  const bool full = m0 + TS <= V;
  const int tid = threadIdx.x;
  const int nt256 = n0 / kTile;
  const int64_t seg = (int64_t)nt256 * kTile * K;
  const int* ho = hoff + (int64_t)nt256 * (nVT + 1) + m0 / kTile;
  const int hb = ho[0], cnt = ho[1] - hb;
  const uint32_t* hl = hits + seg + hb;
  if constexpr (TS == 128) {
    // a small tile: staged in LDS, each entry reads its cell
    float* st = reinterpret_cast<float*>(lds);
    for (int h = 0; h < 2; ++h) {
      stage_half<TS>(st, acc, h, wm, wn, lane);
      __syncthreads();
      auto rec = [&](uint32_t e, float) {
        int tl, v;
        if (entry_cell<TS>(e, m0, n0, tl, v) && tl / (TS / 2) == h)
          zhit[(int64_t)(n0 + tl) * K + (e >> 16)] = *stage_cell<TS>(st, tl & (TS / 2 - 1), v);
      };
      if (tid < cnt) rec(hl[tid], 0.f);
      rest_entries<TS>(tid, cnt, hl, nullptr, rec);
      __syncthreads();
    }
  } else {
    constexpr int kThreads = G::kThreads;
    uint32_t* bits = reinterpret_cast<uint32_t*>(lds + kZhBits);
    int* pre = reinterpret_cast<int*>(lds + kZhPre);
    int* wsum = reinterpret_cast<int*>(lds + kZhWs);
    float* zval = reinterpret_cast<float*>(lds + kZhVal);
    *reinterpret_cast<u32x4_t*>(bits + 4 * tid) = u32x4_t{0u, 0u, 0u, 0u};
    __syncthreads();
    for (int q = tid; q < cnt; q += kThreads) {
      const uint32_t e = hl[q];
      const int tl = (int)(e & 255u), vl = (int)((e >> 8) & 255u);
      atomicOr(&bits[tl * 8 + (vl >> 5)], 1u << (vl & 31));
    }
    __syncthreads();
    // exclusive prefix of the 2048 word counts: thread tid owns words 4 tid .. 4 tid + 3
    {
      const u32x4_t wd = *reinterpret_cast<const u32x4_t*>(bits + 4 * tid);
      const int c0 = __builtin_popcount(wd[0]), c1 = __builtin_popcount(wd[1]);
      const int c2 = __builtin_popcount(wd[2]), c3 = __builtin_popcount(wd[3]);
      const int run = c0 + c1 + c2 + c3;
      const int incl = wave_incl_scan(run);
      if (lane == 63) wsum[wave] = incl;
      __syncthreads();
      int base = incl - run;
      for (int w = 0; w < wave; ++w) base += wsum[w];
      *reinterpret_cast<i32x4_t*>(pre + 4 * tid) =
          i32x4_t{base, base + c0, base + c0 + c1, base + c0 + c1 + c2};
    }
    __syncthreads();
    const int g = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = G::acc_n(wn, j, lane);  // token in the tile
      const u32x4_t wd = *reinterpret_cast<const u32x4_t*>(bits + n * 8 + wm * 4);
      const i32x4_t wp = *reinterpret_cast<const i32x4_t*>(pre + n * 8 + wm * 4);
#pragma unroll
      for (int i = 0; i < G::NI; ++i) {
        const int sh = 16 * (i & 1) + 4 * g;  // bit of the cell's first column in its word
        const uint32_t nib = (wd[i >> 1] >> sh) & 15u;
        if (nib == 0u) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (((nib >> r) & 1u) == 0u) continue;
          const int rank = wp[i >> 1] + __builtin_popcount(wd[i >> 1] & ((1u << (sh + r)) - 1u));
          if (rank < kZhCap) {
            zval[rank] = acc.v[i][j][r];
          } else {
            const uint32_t cell = (uint32_t)n | ((uint32_t)G::acc_m(wm, i, lane, r) << 8);
            for (int q = 0; q < cnt; ++q) {
              const uint32_t e = hl[q];
              if ((e & 0xffffu) == cell) zhit[(int64_t)(n0 + n) * K + (e >> 16)] = acc.v[i][j][r];
            }
          }
        }
      }
    }
    __syncthreads();
    for (int q = tid; q < cnt; q += kThreads) {
      const uint32_t e = hl[q];
      const int tl = (int)(e & 255u), vl = (int)((e >> 8) & 255u);
      const int w = tl * 8 + (vl >> 5);
      const int rank = pre[w] + __builtin_popcount(bits[w] & ((1u << (vl & 31)) - 1u));
      if (rank < kZhCap) zhit[(int64_t)(n0 + tl) * K + (e >> 16)] = zval[rank];
    }
    __syncthreads();
  }
  float* xch = reinterpret_cast<float*>(lds);  // [wn][j][16 lanes][max, sum]
  float rm[4], rs[4];
  // Per token: the max is taken over z itself (k2 > 0), then sum 2^(z k2 - max)
  // (one fma, one exp2 and one add per element). Only the last vocabulary
  // tile of a V that is not a multiple of 256 tests its columns.
  auto lse = [&](auto full_tile) {
    constexpr bool kFull = decltype(full_tile)::value;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float za = -INFINITY;
#pragma unroll
      for (int i = 0; i < G::NI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kFull || m0 + G::acc_m(wm, i, lane, r) < V) za = fmaxf(za, acc.v[i][j][r]);
      // the four lane groups (lane>>4) hold the other rows of the same token
      za = fmaxf(za, __shfl_xor(za, 16));
      za = fmaxf(za, __shfl_xor(za, 32));
      const float mx = za * k2;
      float s = 0.f;
      if (mx != -INFINITY) {
#pragma unroll
        for (int i = 0; i < G::NI; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float e = fast_exp2(acc.v[i][j][r] * k2 - mx);
            if (kFull || m0 + G::acc_m(wm, i, lane, r) < V) s += e;
          }
      }
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      rm[j] = mx;
      rs[j] = s;
      if (wm == 1 && lane < 16) {
        xch[((wn * 4 + j) * 16 + lane) * 2 + 0] = mx;
        xch[((wn * 4 + j) * 16 + lane) * 2 + 1] = s;
      }
    }
  };
  if (full)
    lse(std::integral_constant<bool, true>());
  else
    lse(std::integral_constant<bool, false>());
  __syncthreads();
  if (wm == 0 && lane < 16) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = n0 + G::acc_n(wn, j, lane);
      const float m1 = rm[j], s1 = rs[j];
      const float m2 = xch[((wn * 4 + j) * 16 + lane) * 2 + 0];
      const float s2 = xch[((wn * 4 + j) * 16 + lane) * 2 + 1];
      const float mm = fmaxf(m1, m2);
      float ss = 0.f;
      if (mm != -INFINITY) ss = s1 * fast_exp2(m1 - mm) + s2 * fast_exp2(m2 - mm);
      if (t < rows) {
        put_partial<TS>(tiles, part_m, part_s, t, m0, mm, ss, -INFINITY);
      }
    }
  }
}

// log2 of the normaliser per token from the vocabulary-tile partials (fixed
// order, one wave per token). L2 = log2 sum_v 2^(z_v log2(e)/tau); a partial
// is the tile max and the sum of 2^(y - max) over the tile's columns.
__global__ void k_lse_merge(const float* part_m, const float* part_s, int rows, int nVT,
                            float* rowL2, const int* __restrict__ rowmap) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + wave_id();
  if (r >= rows) return;
  if (rowmap != nullptr && rowmap[r] < 0) {
    // a row without a token: its partials were never written
    if (lane == 0) rowL2[r] = 0.f;
    return;
  }
  const float* pm = part_m + (int64_t)r * nVT;
  const float* ps = part_s + (int64_t)r * nVT;
  float mx = -INFINITY;
  for (int j = lane; j < nVT; j += 64) mx = fmaxf(mx, pm[j]);
  mx = wave_max(mx);
  float s = 0.f;
  for (int j = lane; j < nVT; j += 64) {
    const float m = pm[j];
    if (m != -INFINITY) s += ps[j] * fast_exp2(m - mx);
  }
  s = wave_sum(s);
  if (lane == 0) rowL2[r] = mx + log2f(s);
}

// ------------------------------------------------ teacher entry buckets ----
// The K cached entries of each token are folded into the dZ tile that holds
// their vocabulary column (§3.2). One workgroup per 256-token tile groups the
// tile's entries by vocabulary tile with a counting sort in LDS: segment nt of
// `hits` (capacity 256 K) lists, for vocabulary tile b, the entries
// [hoff[nt][b], hoff[nt][b+1]) as (token in tile | column in tile << 8 | k << 16)
// with their teacher probability in `hitp` (when asked for: only the separate
// backward reads it). An index outside [0, V) gets no slot and a zero z (it
// contributes nothing to C or dZ).
//
// Latency-bound (one workgroup per 256 tokens). Up to kBucketRegs entries per
// thread (K <= 128, or fewer tokens) stay in registers: all of a thread's loads
// are in flight together, and the atomic that counts an entry also returns its
// place among the entries of its vocabulary tile, so each entry is read once and
// takes one atomic (512 tokens, K = 64, V = 32000: 22.5 us, now 12.2 us). More
// entries are read twice, counted and then placed: a kernel of its own, in which
// the registers of the first form would cost it a quarter (574 tokens, K = 2932,
// both passes of a split call: 860 us alone, 1080 beside it).
constexpr int kBucketThreads = 1024;
constexpr int kBucketRegs = 32;
constexpr int kBucketBatch = 8;  // entries per thread whose loads are in flight together
constexpr int kMaxVT = 4096;     // vocabulary tiles (V <= 2^20)

struct BucketArgs {
  const int32_t* tidx;  // [rows, K], or with rowmap the full [N, K] indexed by its tokens
  const int* rowmap;    // or null
  const float* p;
  int rows, K, V, nVT;
  uint32_t* hits;
  float* hitp;
  int* hoff;
  float* zhit;
};

struct BucketLds {
  int cnt[kMaxVT], cur[kMaxVT], wsum[kBucketThreads / 64];
};

// ONE: at most kBucketRegs entries per thread. PREP: rowmap may be set, no hitp
template <bool ONE, bool PREP>
__device__ __forceinline__ void bucket_tile(const BucketArgs& a, int block, BucketLds& l) {
  const int rows = a.rows, K = a.K, V = a.V, nVT = a.nVT;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int t0 = block * kTile;
  const int total = min(kTile, rows - t0) * K;
  const int64_t seg = (int64_t)block * kTile * K;
  uint32_t* hits = a.hits + seg;
  float* hitp = PREP || a.hitp == nullptr ? nullptr : a.hitp + seg;
  // entry e of the tile is element t0 K + e of the row-major [rows, K] arrays
  const int32_t* __restrict__ ti = a.tidx + (PREP && a.rowmap != nullptr ? 0 : (int64_t)t0 * K);
  const float* __restrict__ pt = a.p + (int64_t)t0 * K;
  float* zt = a.zhit + (int64_t)t0 * K;
  const float invK = 1.0f / (float)K;
  // token = e / K (exact: e < 2^20, and (e + 0.5) / K stays >= 1/(2K)
  // away from an integer while the float product errs by < 2^-12)
  auto token = [&](int e) { return (int)(((float)e + 0.5f) * invK); };
  auto index = [&](int e) -> int {
    if (!PREP || a.rowmap == nullptr) return ti[(uint32_t)e];
    const int tl = token(e), tok = a.rowmap[t0 + tl];
    return tok < 0 ? -1 : ti[(int64_t)tok * K + (e - tl * K)];
  };
  auto put = [&](int e, int v, int pos, float pk) {
    const int tl = token(e);
    const int k = e - tl * K;
    hits[(uint32_t)pos] = (uint32_t)tl | ((uint32_t)(v & 255) << 8) | ((uint32_t)k << 16);
    if (hitp != nullptr) hitp[(uint32_t)pos] = pk;
  };
  constexpr int NR = ONE ? kBucketRegs : 1;
  int v[NR], rank[NR];
  // p a batch ahead of its use (all of it in registers would spill)
  float pv[2][kBucketBatch];
  auto load_p = [&](int u0) {
    if (hitp == nullptr || u0 >= kBucketRegs) return;
#pragma unroll
    for (int u = 0; u < kBucketBatch; ++u) {
      const int e = (u0 + u) * kBucketThreads + tid;
      pv[u0 / kBucketBatch & 1][u] = e < total ? pt[(uint32_t)e] : 0.f;
    }
  };
  if constexpr (ONE) {
#pragma unroll
    for (int u = 0; u < kBucketRegs; ++u) {
      const int e = u * kBucketThreads + tid;
      v[u] = e < total ? index(e) : -1;
    }
  }
  for (int b = tid; b < nVT; b += kBucketThreads) l.cnt[b] = 0;
  __syncthreads();
  if constexpr (ONE) {
#pragma unroll
    for (int u = 0; u < kBucketRegs; ++u) {
      const int e = u * kBucketThreads + tid;
      if (u * kBucketThreads >= total) break;
      rank[u] = 0;
      if ((unsigned)v[u] < (unsigned)V)
        rank[u] = atomicAdd(&l.cnt[v[u] >> 8], 1);
      else if (e < total)
        zt[(uint32_t)e] = 0.f;
    }
    load_p(0);
  } else {
    for (int base = 0; base < total; base += kBucketThreads * kBucketBatch) {
      int w[kBucketBatch];
#pragma unroll
      for (int u = 0; u < kBucketBatch; ++u) {
        const int e = base + u * kBucketThreads + tid;
        w[u] = e < total ? index(e) : 0;
      }
#pragma unroll
      for (int u = 0; u < kBucketBatch; ++u) {
        const int e = base + u * kBucketThreads + tid;
        if (e >= total) continue;
        if ((unsigned)w[u] < (unsigned)V)
          atomicAdd(&l.cnt[w[u] >> 8], 1);
        else
          zt[(uint32_t)e] = 0.f;
      }
    }
  }
  __syncthreads();
  // exclusive scan: thread tid owns bins [tid R, tid R + R)
  const int R = (nVT + kBucketThreads - 1) / kBucketThreads;
  int run = 0;
  for (int q = 0; q < R; ++q) {
    const int b = tid * R + q;
    if (b < nVT) run += l.cnt[b];
  }
  const int incl = wave_incl_scan(run);
  if (lane == 63) l.wsum[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int x = lane < kBucketThreads / 64 ? l.wsum[lane] : 0;
    const int y = wave_incl_scan(x);
    if (lane < kBucketThreads / 64) l.wsum[lane] = y - x;
  }
  __syncthreads();
  int off = l.wsum[wave] + incl - run;
  int* ho = a.hoff + (int64_t)block * (nVT + 1);
  for (int q = 0; q < R; ++q) {
    const int b = tid * R + q;
    if (b < nVT) {
      l.cur[b] = off;
      ho[b] = off;
      off += l.cnt[b];
    }
  }
  if (tid == kBucketThreads - 1) ho[nVT] = off;
  __syncthreads();
  if constexpr (ONE) {
#pragma unroll
    for (int u0 = 0; u0 < kBucketRegs; u0 += kBucketBatch) {
      if (u0 * kBucketThreads >= total) break;
      load_p(u0 + kBucketBatch);
#pragma unroll
      for (int u = u0; u < u0 + kBucketBatch; ++u)
        if ((unsigned)v[u] < (unsigned)V)
          put(u * kBucketThreads + tid, v[u], l.cur[v[u] >> 8] + rank[u],
              pv[u / kBucketBatch & 1][u % kBucketBatch]);
    }
    return;
  }
  for (int base = 0; base < total; base += kBucketThreads * kBucketBatch) {
    int w[kBucketBatch];
    float pw[kBucketBatch];
#pragma unroll
    for (int u = 0; u < kBucketBatch; ++u) {
      const int e = base + u * kBucketThreads + tid;
      w[u] = e < total ? index(e) : -1;
      pw[u] = hitp != nullptr && e < total ? pt[(uint32_t)e] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kBucketBatch; ++u) {
      const int e = base + u * kBucketThreads + tid;
      if (e >= total || (unsigned)w[u] >= (unsigned)V) continue;
      put(e, w[u], atomicAdd(&l.cur[w[u] >> 8], 1), pw[u]);
    }
  }
}

// after the prologue, from its copy of the indices (no rowmap); ONE as above
template <bool ONE>
__global__ __launch_bounds__(kBucketThreads) void k_bucket(BucketArgs a) {
  __shared__ BucketLds l;
  bucket_tile<ONE, false>(a, blockIdx.x, l);
}

// The prologue of a row per wave and, in the first `nb` workgroups (K <=
// kPrepMaxK), the buckets: they run on a few compute units for as long as the
// prologue does on the others. The buckets then read the caller's indices, so
// a repeated index of a row gets an entry per repeat: harmless where entries
// only record z (the later ones have p = 0), but not for the separate
// backward, whose entries patch their cells: it runs k_bucket after the
// prologue. 512 tokens, K = 64: 20.2 us for both, now 13.1 us.
constexpr int kPrepMaxK = 128;
template <typename T>
__global__ __launch_bounds__(kBucketThreads) void k_prep(PrologueArgs a, BucketArgs b, int nb) {
  constexpr int kRowLds = prologue_lds(kPrepMaxK), NWV = kBucketThreads / 64;
  __shared__ __attribute__((aligned(16))) char lds[NWV * kRowLds];
  __shared__ BucketLds l;
  static_assert(kPrepMaxK * kTile <= kBucketThreads * kBucketRegs, "entries in registers");
  if ((int)blockIdx.x < nb) {
    bucket_tile<true, true>(b, blockIdx.x, l);
    return;
  }
  const int wave = wave_id();
  prologue_row<T>(a, ((int)blockIdx.x - nb) * NWV + wave, lds + wave * kRowLds);
}
template <typename T>
__global__ __launch_bounds__(64) void k_prologue(PrologueArgs a) {
  extern __shared__ __attribute__((aligned(16))) char psm[];
  prologue_row<T>(a, blockIdx.x, psm);
}

// --------------------------------------- logit recompute + dZ epilogue -----
// Same tile as k_logits_lse (bitwise identical z). Before the main loop the
// tile's per-token scalars (g/tau M, g/tau, log2 Z) and its teacher entries
// (one per thread) are loaded into registers, so the epilogue issues no
// global loads (a load waited for after a store would also wait for that
// store); after the loop the scalars go to LDS beside the staging area.
// The fp32 tile is staged half its tokens at a time as [token][vocab] with a
// 16-byte-slot swizzle; each teacher entry of the half is patched in place to
// its final value (g/tau)(M q - p), and a bitmap marks it; then one wave per token
// row forms G = (g/tau) M 2^(y - L2) elsewhere and stores the row of dZ[rows, Vp]
// (columns V..Vp: finite values of z = 0).
// epilogue LDS (the main loop's stages are free by then), after the staging area
template <int TS>
constexpr int kDzBits = stage_bytes<TS>;                // TS/2 x TS-bit hit map of one half
template <int TS>
constexpr int kDzRows = kDzBits<TS> + TS / 2 * TS / 8;  // 3 x TS floats: g/tau M, g/tau, log2 Z
static_assert(kDzRows<256> + 3 * 1024 <= kLdsA3, "dZ epilogue LDS");
static_assert(kDzRows<128> + 3 * 512 <= kLdsF32, "dZ epilogue LDS");

template <typename T, int TS>
__global__ __launch_bounds__(Geo<TS>::kThreads, TS == 256 ? 1 : 2) void k_dz(
    const T* __restrict__ W, const T* __restrict__ Hc, int D, int V, int rows, ProjTiles tiles,
    float k2, const float* __restrict__ rowL2, const float* __restrict__ rowCoef,
    const float* __restrict__ rowCoefM, const uint32_t* __restrict__ hits,
    const float* __restrict__ hitp, const int* __restrict__ hoff, int K, int nVT, T* dZ,
    int64_t ldz, const int* __restrict__ nrow, int nrow_base) {
  typedef Geo<TS> G;
  constexpr int kThreads = G::kThreads, HT = TS / 2;  // HT: tokens staged at a time
  __shared__ __attribute__((aligned(16))) char lds[gemm_lds<T, TS>];
  int m0, n0;
  proj_tile<TS>(tiles, m0, n0);
  const int eb = Elt<T>::bytes;
  const int ld = D * eb;
  // with ignored tokens left out only the first *nrow - nrow_base rows hold
  // tokens (as in k_logits_dz; the rows past them have weight 0)
  int trows = rows;
  if (nrow != nullptr) trows = min(rows, __builtin_amdgcn_readfirstlane(*nrow) - nrow_base);
  if (n0 >= trows) return;
  const int mrows = max(0, min(TS, V - m0)), nrows = min(TS, trows - n0);
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);

  // this tile's bucket of teacher entries
  const int64_t seg = (int64_t)(n0 / kTile) * kTile * K;
  const int* ho = hoff + (int64_t)(n0 / kTile) * (nVT + 1) + m0 / kTile;
  const int hb = ho[0], cnt = ho[1] - hb;
  // wave w holds the scalars of tokens [32 w, 32 w + 32): lane l has token
  // 32 w + (l & 31), g/tau M and g/tau (l < 32) or log2 Z (l >= 32, in rv0)
  float rv0, rv1 = 0.f;
  {
    const int t = n0 + 32 * wave + (lane & 31);
    const bool ok = t < rows;
    rv0 = ok ? (lane < 32 ? rowCoefM[t] : rowL2[t]) : 0.f;
    if (lane < 32) rv1 = ok ? rowCoef[t] : 0.f;
  }
  uint32_t fe = 0u;  // this thread's teacher entry (entry tid of the bucket) and its p
  float fpk = 0.f;
  if (tid < cnt) {
    fe = hits[seg + hb + tid];
    fpk = hitp[seg + hb + tid];
  }

  AccTile<TS> acc;
  gemm<T, TS, false>(
      KcOp{reinterpret_cast<const char*>(W + (int64_t)m0 * D), (uint32_t)(mrows * ld), ld},
      KcOp{reinterpret_cast<const char*>(Hc + (int64_t)n0 * D), (uint32_t)(nrows * ld), ld}, 0,
      ld / kRowB, lds, acc);
  {
    float* rs = reinterpret_cast<float*>(lds + kDzRows<TS>);
    const int t = 32 * wave + (lane & 31);
    if (lane < 32) {
      rs[t] = rv0;
      rs[TS + t] = rv1;
    } else {
      rs[2 * TS + t] = rv0;
    }
  }

  float* st = reinterpret_cast<float*>(lds);
  const float* rs_cm = reinterpret_cast<const float*>(lds + kDzRows<TS>);
  const float* rs_cf = rs_cm + TS;
  const float* rs_l2 = rs_cm + 2 * TS;
  uint32_t* hbits = reinterpret_cast<uint32_t*>(lds + kDzBits<TS>);
  // row pass: 4 vocabulary columns per lane, RPI token rows per wave and
  // iteration (the whole wave on one row of 256 columns, half of it on 128)
  constexpr int LPR = TS / 4, RPI = 64 / LPR;
  const int vl0 = 4 * (lane % LPR);

  // unrolled: a loop header here would make the compiler wait for the first
  // half's dZ stores before staging the second half
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    stage_half<TS>(st, acc, h, wm, wn, lane);
    for (int q = tid; q < HT * TS / 32; q += kThreads) hbits[q] = 0u;
    __syncthreads();

    // Teacher entries of this half: dZ = (g/tau) M q - (g/tau) p in place.
    // Thread tid has entry tid of the bucket in registers; a skewed teacher with
    // more entries in one tile than threads reads the rest from memory.
    auto fold = [&](uint32_t e, float pk) {
      int tl, v;
      if (!entry_cell<TS>(e, m0, n0, tl, v) || tl / HT != h) return;
      const int n = tl & (HT - 1);
      float* cell = stage_cell<TS>(st, n, v);
      const float z = *cell;
      *cell = rs_cm[tl] * fast_exp2(z * k2 - rs_l2[tl]) - rs_cf[tl] * pk;
      atomicOr(&hbits[n * (TS / 32) + (v >> 5)], 1u << (v & 31));
    };
    if (tid < cnt) fold(fe, fpk);
    // a bucket with more entries than threads: the rest from memory
    rest_entries<TS>(tid, cnt, hits + seg + hb, hitp + seg + hb, fold);
    __syncthreads();

    if (dZ != nullptr) {
      // The wave's 16 rows go in two batches of 8 whose LDS reads are all
      // issued before their arithmetic. The row pass is VALU-bound (every
      // element costs an exp2), so it carries no per-element selects: a row's
      // teacher cells (about one row in five has any) are substituted behind
      // a wave-uniform test, and columns past V get no mask (their z is
      // exactly 0, as W's rows past V read as zeros, so they hold finite
      // values that only ever meet those zero rows).
      const int rb = wave * 16 + lane / LPR;                        // first row in the half
      const int nrow = max(0, min(16, rows - (n0 + HT * h + wave * 16)));  // rows that exist
#pragma unroll
      for (int b8 = 0; b8 < 16 / RPI; b8 += 8) {
        f32x4_t zr[8];
        uint32_t mk[8];
#pragma unroll
        for (int rr = 0; rr < 8; ++rr) {
          const int n = rb + (b8 + rr) * RPI;
          zr[rr] = *reinterpret_cast<const f32x4_t*>(stage_cell<TS>(st, n, vl0));
          mk[rr] = (hbits[n * (TS / 32) + (vl0 >> 5)] >> (vl0 & 31)) & 15u;
        }
        float cmv[8], l2v[8];  // the rows' g/tau M and log2 Z
        if constexpr (RPI == 1) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {  // the same for the wave: 16-byte aligned runs
            const f32x4_t c4 = *reinterpret_cast<const f32x4_t*>(rs_cm + HT * h + rb + b8 + 4 * u);
            const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(rs_l2 + HT * h + rb + b8 + 4 * u);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              cmv[4 * u + e] = c4[e];
              l2v[4 * u + e] = l4[e];
            }
          }
        } else {
#pragma unroll
          for (int rr = 0; rr < 8; ++rr) {
            cmv[rr] = rs_cm[HT * h + rb + (b8 + rr) * RPI];
            l2v[rr] = rs_l2[HT * h + rb + (b8 + rr) * RPI];
          }
        }
#pragma unroll
        for (int rr = 0; rr < 8; ++rr) {
          const float cm = cmv[rr], L2 = l2v[rr];
          f32x4_t g;
#pragma unroll
          for (int e = 0; e < 4; ++e) g[e] = cm * fast_exp2(zr[rr][e] * k2 - L2);
          if (__builtin_amdgcn_ballot_w64(mk[rr] != 0u) != 0ull) {
            // teacher cells hold their final value (patched by the fold)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if ((mk[rr] >> e) & 1u) g[e] = zr[rr][e];
          }
          const int nr = (b8 + rr) * RPI + lane / LPR;
          if (nr < nrow) {
            T* dst = dZ + (int64_t)(n0 + HT * h + wave * 16 + nr) * ldz + m0 + vl0;
            if constexpr (sizeof(T) == 2) {
              u32x2_t pk2 = {pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3])};
              *reinterpret_cast<u32x2_t*>(dst) = pk2;
            } else {
              *reinterpret_cast<f32x4_t*>(dst) = g;
            }
          }
        }
      }
    }
    __syncthreads();
  }
}

// ------------------------------------ one projection per chunk (fused call) --
// A call that wants the loss and its gradients together has each chunk's
// normaliser complete as soon as that chunk's projection has run, so the
// chunk is projected once instead of once for log Z and again for dZ: the
// tile records per token z at its teacher entries, the provisional gradient
// dZ'' = 2^(y - R) with y = z log2(e) / tau in the dZ buffer (0 past V), R
// being the token's reference logit from k_prologue, and the partials (R,
// sum of 2^(y - R)) of log Z (a reference and a sum relative to it, like
// the (max, sum) partials of k_logits_lse).
// Once log Z is merged, the row factor (g/tau) M 2^(R - log2 Z) turns dZ''
// into (g/tau) M q; it is applied to the rows of dH and, through the
// transposed hidden rows, to dW, so dZ'' is never rewritten, except the
// teacher cells (k_row_finish writes (g/tau)(M q - p) / factor, Eq. 3) and the
// rare rows where a tile's sum of 2^(y - R) exceeded 2^kRefGap (k_row_finish
// rescales them).
// The [c, V] buffer is the same transient chunk the recompute schedule holds;
// nothing grows with N. Staging and teacher bookkeeping are those of k_dz.
template <typename T, int TS>
__global__ __launch_bounds__(Geo<TS>::kThreads, TS == 256 ? 1 : 2) void k_logits_dz(
    const T* __restrict__ W, const T* __restrict__ Hc, int D, int V, int rows, ProjTiles tiles,
    float k2, float* __restrict__ part_m, float* __restrict__ part_s, int nVT,
    const uint32_t* __restrict__ hits, const int* __restrict__ hoff, int K, T* dZ, int64_t ldz,
    float* zhit, const float* __restrict__ rowR, int* rowFlag, const int* __restrict__ nrow,
    int nrow_base) {
  typedef Geo<TS> G;
  constexpr int kThreads = G::kThreads, HT = TS / 2;  // HT: tokens staged at a time
  __shared__ __attribute__((aligned(16))) char lds[gemm_lds<T, TS>];
  int m0, n0;
  proj_tile<TS>(tiles, m0, n0);
  const int eb = Elt<T>::bytes;
  const int ld = D * eb;
  // with ignored tokens left out only the first *nrow - nrow_base rows hold
  // tokens: a tile of rows past them has nothing to compute, and rows past
  // them in the last tile read hidden rows of zeros (stored like the others,
  // with a row factor of 0)
  int trows = rows;
  if (nrow != nullptr) trows = min(rows, __builtin_amdgcn_readfirstlane(*nrow) - nrow_base);
  if (n0 >= trows) return;
  const int mrows = max(0, min(TS, V - m0)), nrows = min(TS, trows - n0);
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);

  const int64_t seg = (int64_t)(n0 / kTile) * kTile * K;
  const int* ho = hoff + (int64_t)(n0 / kTile) * (nVT + 1) + m0 / kTile;
  const int hb = ho[0], cnt = ho[1] - hb;
  const uint32_t fe = tid < cnt ? hits[seg + hb + tid] : 0u;
  // the tile's reference logits, loaded before the main loop: a load issued
  // in the epilogue would wait for every store issued before it (loads and
  // stores complete in order), serialising the row pass on its stores
  const float rref = (tid < TS && n0 + tid < rows) ? rowR[n0 + tid] : 0.f;

  AccTile<TS> acc;
  gemm<T, TS, false>(
      KcOp{reinterpret_cast<const char*>(W + (int64_t)m0 * D), (uint32_t)(mrows * ld), ld},
      KcOp{reinterpret_cast<const char*>(Hc + (int64_t)n0 * D), (uint32_t)(nrows * ld), ld}, 0,
      ld / kRowB, lds, acc);
  const bool full = m0 + TS <= V;

  float* st = reinterpret_cast<float*>(lds);
  // past the staging area: R of the tile's tokens (0 past the chunk)
  float* rs_r = reinterpret_cast<float*>(lds + stage_bytes<TS>);
  if (tid < TS) rs_r[tid] = rref;
  constexpr int NK = TS / 64;
  const int rho = lane >> 4, lam = lane & 15;  // row pass: 4 token rows per wave, 16 lanes each
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    stage_half<TS>(st, acc, h, wm, wn, lane);
    __syncthreads();
    // z at the teacher entries of this half, for C = sum_k p z (Eq. 2)
    auto rec = [&](uint32_t e, float) {
      int tl, v;
      if (!entry_cell<TS>(e, m0, n0, tl, v) || tl / HT != h) return;
      zhit[(int64_t)(n0 + tl) * K + (e >> 16)] = *stage_cell<TS>(st, tl & (HT - 1), v);
    };
    if (tid < cnt) rec(fe, 0.f);
    rest_entries<TS>(tid, cnt, hits + seg + hb, nullptr, rec);

    // 16 lanes per token row, lane lam holding columns 4 lam + 64 k + (0..3), k < NK.
    // The row's run of dZ'' is 2^(y - R) against the token's reference R; the
    // partials are (R, sum of 2^(y - R)) with the sum reduced within the 16
    // lanes (DPP). A run whose sum exceeds 2^kRefGap (so its values could
    // too) is stored against the run's own max m instead, with partials
    // (m, sum of 2^(y - m)), and its token is flagged for a row rescale.
    // Columns past V give 0 and count for neither.
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const int n = wave * 16 + 4 * gq + rho;  // token row of the half
      const int t = n0 + HT * h + n;
      f32x4_t zr[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k)
        zr[k] = *reinterpret_cast<const f32x4_t*>(stage_cell<TS>(st, n, 4 * lam + 64 * k));
      // rows past the chunk use a finite reference (nothing of them is stored)
      float ref = rs_r[HT * h + n];
      f32x4_t g[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k)
        g[k] = f32x4_t{fast_exp2(zr[k][0] * k2 - ref), fast_exp2(zr[k][1] * k2 - ref),
                       fast_exp2(zr[k][2] * k2 - ref), fast_exp2(zr[k][3] * k2 - ref)};
      // the column mask only on the last vocabulary tile (a wave-uniform
      // branch instead of per-element selects on every tile)
      if (!full) {
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          const int c = m0 + 4 * lam + 64 * k;
          g[k] = f32x4_t{c < V ? g[k][0] : 0.f, c + 1 < V ? g[k][1] : 0.f,
                         c + 2 < V ? g[k][2] : 0.f, c + 3 < V ? g[k][3] : 0.f};
        }
      }
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < NK; ++k) sum += (g[k][0] + g[k][1]) + (g[k][2] + g[k][3]);
      sum = row16_sum(sum);
      const bool own = !(sum <= kRefGapScale);
      if (__builtin_amdgcn_ballot_w64(own) != 0ull) {
        // rare: some row of the wave falls back to its own max (formed for
        // every row so that the 16-lane reductions run on a full wave)
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (full || m0 + 4 * lam + 64 * k + e < V) mx = fmaxf(mx, zr[k][e]);
        const float m = row16_max(mx) * k2;
        float s2 = 0.f;
        f32x4_t g2[NK];
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float ev = fast_exp2(zr[k][e] * k2 - m);
            if (!full && m0 + 4 * lam + 64 * k + e >= V) ev = 0.f;
            g2[k][e] = ev;
            s2 += ev;
          }
        s2 = row16_sum(s2);
        if (own) {
          ref = m;
          sum = s2;
#pragma unroll
          for (int k = 0; k < NK; ++k) g[k] = g2[k];
        }
      }
      if (t < rows) {
        T* dst = dZ + (int64_t)t * ldz + m0 + 4 * lam;
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          if constexpr (sizeof(T) == 2) {
            const u32x2_t pk2 = {pack_bf16x2(g[k][0], g[k][1]), pack_bf16x2(g[k][2], g[k][3])};
            *reinterpret_cast<u32x2_t*>(dst + 64 * k) = pk2;
          } else {
            *reinterpret_cast<f32x4_t*>(dst + 64 * k) = g[k];
          }
        }
        if (lam == 0) {
          put_partial<TS>(tiles, part_m, part_s, t, m0, ref, sum, ref);
          if (own) rowFlag[t] = 1;
        }
      }
    }
    __syncthreads();
  }
}

// l_t = H_t - C_t / tau + M_t log Z_t (Eq. 2) with C_t = sum_k p_k z_{t, idx_k},
// 0 on ignored rows; one wave per row and a partial sum per block of
// kLossRows rows in a fixed order, for the deterministic mean.
__global__ void k_row_loss(const float* zhit, const float* p, int K, const float* rowL2,
                           const float* rowM, const float* rowH, const uint8_t* ignore,
                           int64_t row0, const int* __restrict__ rowmap, int rows, float inv_tau,
                           float* loss_per_token, float* logz_out, float* block_partial) {
  __shared__ float red[kLossRows];
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int r = blockIdx.x * kLossRows + wave;
  float l = 0.f;
  // with a rowmap, row r is token rowmap[r] (loss_per_token and logz_out
  // indexed by token), and a row without a token (-1) has a loss of 0
  const int tok = (rowmap != nullptr && r < rows) ? rowmap[r] : 0;
  if (r < rows && tok >= 0) {
    float c = 0.f;
    for (int k = lane; k < K; k += 64) {
      // (both loads at once; a repeated index has p = 0 and a z that need not be
      // finite)
      const float pk = p[(int64_t)r * K + k], z = zhit[(int64_t)r * K + k];
      c += pk != 0.f ? pk * z : 0.f;
    }
    c = wave_sum(c);
    const bool valid = rowmap != nullptr || ignore == nullptr || ignore[row0 + r] == 0;
    l = valid ? rowH[r] - c * inv_tau + rowM[r] * rowL2[r] * kLn2 : 0.f;
    if (lane == 0) {
      if (loss_per_token) loss_per_token[rowmap != nullptr ? (int64_t)tok : r] = l;
      if (logz_out) logz_out[rowmap != nullptr ? (int64_t)tok : r] = rowL2[r] * kLn2;
    }
  }
  if (lane == 0) red[wave] = l;
  __syncthreads();
  if (threadIdx.x == 0) block_partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// The end of a chunk in the single-projection schedule, one wave per token
// (one pass instead of four launches): log2 Z merged from the tile partials
// (each a reference and a sum relative to it), the row factor that turns the
// stored 2^(y - mx) into (g/tau) M q, mx being the largest reference of the
// row's tiles (the token's reference logit unless a tile fell back to its own
// max); for a row with such a tile, every run brought to mx; the teacher
// cells (g/tau)(M q - p) (Eq. 3) in the row's stored scale (0 where the
// factor is 0, i.e. on ignored rows); and the token's loss (Eq. 2) with a
// partial per block of kLossRows rows as k_row_loss forms it. With a rowmap,
// row r is token rowmap[r] (loss_per_token is then indexed by token), and a
// row without a token (-1) only gets a row factor of 0 and a loss of 0.
template <typename T>
__global__ __launch_bounds__(256) void k_row_finish(
    const float* __restrict__ part_m, const float* __restrict__ part_s, int nVT, int vt_shift,
    const int* __restrict__ rowFlag, T* dZ, int64_t ldz, const int32_t* __restrict__ tidx,
    const float* __restrict__ p, const float* __restrict__ zhit, int K, int V, float k2,
    const float* __restrict__ rowM, const float* __restrict__ rowH,
    const float* __restrict__ rowCoef, const float* __restrict__ rowCoefM,
    const uint8_t* __restrict__ ignore, int64_t row0, const int* __restrict__ rowmap, int rows,
    float inv_tau, float* rowL2, float* rowFactor, float* loss_per_token, float* block_partial) {
  __shared__ float red[kLossRows];
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int r = blockIdx.x * kLossRows + wave;
  float l = 0.f;
  const int tok = (rowmap != nullptr && r < rows) ? rowmap[r] : 0;
  if (r < rows && tok < 0) {
    if (lane == 0) {
      rowL2[r] = 0.f;
      rowFactor[r] = 0.f;
    }
  } else if (r < rows) {
    const float* pm = part_m + (int64_t)r * nVT;
    const float* ps = part_s + (int64_t)r * nVT;
    // up to 1024 partials per row: they are loaded into registers
    // in one batch, with the row scalars, before any arithmetic (one round of
    // memory latency instead of one per pass); the sums keep the same order
    constexpr int kRF = 16;
    const bool in_regs = nVT <= 64 * kRF;
    float pmv[kRF], psv[kRF];
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < kRF; ++i) {
        const int j = lane + 64 * i;
        pmv[i] = j < nVT ? pm[j] : -INFINITY;
        psv[i] = j < nVT ? ps[j] : 0.f;
      }
    }
    const float cm = rowCoefM[r], cf = rowCoef[r];
    float mx = -INFINITY;
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < kRF; ++i) mx = fmaxf(mx, pmv[i]);
    } else {
      for (int j = lane; j < nVT; j += 64) mx = fmaxf(mx, pm[j]);
    }
    mx = wave_max(mx);
    float s = 0.f;
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < kRF; ++i)
        if (pmv[i] != -INFINITY) s += psv[i] * fast_exp2(pmv[i] - mx);
    } else {
      for (int j = lane; j < nVT; j += 64) {
        const float m = pm[j];
        if (m != -INFINITY) s += ps[j] * fast_exp2(m - mx);
      }
    }
    s = wave_sum(s);
    const float L2 = mx + log2f(s);
    const float f = cm * fast_exp2(mx - L2);
    if (lane == 0) {
      rowL2[r] = L2;
      rowFactor[r] = f;
    }
    T* row = dZ + (int64_t)r * ldz;
    if (rowFlag[r] != 0) {
      // rare: runs stored against different references
      constexpr int VPT = 16 / (int)sizeof(T);
      for (int64_t c0 = (int64_t)lane * VPT; c0 < ldz; c0 += 64 * VPT) {
        const float fr = fast_exp2(pm[c0 >> vt_shift] - mx);
        u32x4_t* q = reinterpret_cast<u32x4_t*>(row + c0);
        const u32x4_t v = *q;
        // built as a new vector (in-place element updates were miscompiled)
        if constexpr (sizeof(T) == 2) {
          uint32_t o[4];
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t x = v[w];
            o[w] = pack_bf16x2(__builtin_bit_cast(float, x << 16) * fr,
                               __builtin_bit_cast(float, x & 0xffff0000u) * fr);
          }
          *q = u32x4_t{o[0], o[1], o[2], o[3]};
        } else {
          *q = __builtin_bit_cast(u32x4_t, __builtin_bit_cast(f32x4_t, v) * fr);
        }
      }
      // the teacher cells below overwrite some of these elements: the wave's
      // rescale stores complete first (a workgroup-scope fence emits no wait
      // here, so the wait is explicit; the clobber keeps the compiler from
      // moving memory accesses across it)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    float c = 0.f;
    for (int k = lane; k < K; k += 64) {
      const int64_t e = (int64_t)r * K + k;
      const float pk = p[e], z = zhit[e];
      if (pk != 0.f) c += pk * z;
      const int v = tidx[e];
      if ((unsigned)v < (unsigned)V) {
        const float g = cm * fast_exp2(z * k2 - L2) - cf * pk;
        row[v] = (T)(f != 0.f ? g / f : 0.f);
      }
    }
    c = wave_sum(c);
    const bool valid = rowmap != nullptr || ignore == nullptr || ignore[row0 + r] == 0;
    l = valid ? rowH[r] - c * inv_tau + rowM[r] * L2 * kLn2 : 0.f;
    if (lane == 0 && loss_per_token) loss_per_token[rowmap != nullptr ? (int64_t)tok : r] = l;
  }
  if (lane == 0) red[wave] = l;
  __syncthreads();
  if (threadIdx.x == 0) block_partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// loss = (sum of the loss partials) / N_valid, in a fixed order: thread i of
// 256 sums pieces i, i + 256, ... of four partials, then a tree over the
// threads. partials is 16-byte aligned.
constexpr int kFinThreads = 256;
__device__ __forceinline__ void finalize_loss(const float* partials, int n, float inv_n,
                                              float* loss) {
  __shared__ float red[kFinThreads];
  const int tid = threadIdx.x;
  f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int i = tid; i < n / 4; i += kFinThreads) s += reinterpret_cast<const f32x4_t*>(partials)[i];
  float t = (s[0] + s[1]) + (s[2] + s[3]);
  if (tid < (n & 3)) t += partials[(n & ~3) + tid];
  red[tid] = t;
  __syncthreads();
  for (int o = kFinThreads / 2; o > 0; o >>= 1) {
    if (tid < o) red[tid] += red[tid + o];
    __syncthreads();
  }
  if (tid == 0) loss[0] = red[0] * inv_n;
}

// -------------------------------------------------------------------- dH ----
// dH_c[t, d] = sum_v dZ[t, v] W[v, d]: A = dZ (K = vocabulary contiguous),
// B = W read K-major (rows v, columns d); rows of W past V read as zeros. The
// tiles left over for the last round of workgroups are split along the
// vocabulary into fp32 partial tiles (see kd_split_rounds). With a rowmap, dZ row
// t is grad_hidden row rowmap[t] (-1: none), and only the first
// *nrow - nrow_base rows hold tokens: the tiles are those of these rows.
struct DhArgs {
  const void* dZ;
  int64_t ldz;
  const void* W;
  int V, rows, D, TN, ks_total;
  void* gH;
  int gh_f32;
  float* partial;
  int part_space;
  const float* rowscale;
  const int* rowmap;
  const int* nrow;
  int nrow_base;
  KdRounds sp;  // without nrow
};
// kd_split_rounds by a whole wave, a number of ranges per lane (all lanes active,
// the arguments the same). One after the other, with a division each, they took
// about 5 us of a masked dH and as much of its tail (77 x 768 x 32003 with a tenth
// ignored 93 us, now 84; six chunks of 5504 x 320 x 14960 773 us, now 487).
__device__ __forceinline__ KdRounds split_rounds(int tiles, int ksteps, int units, int part_cost,
                                                 int max_parts) {
  static_assert(kSplitMax == 64, "a number of ranges per lane");
  KdRounds r;
  r.dp = tiles / units * units;
  r.rem = tiles - r.dp;
  const int ranges = (int)(threadIdx.x & 63) + 1;
  const int t = kd_split_time(ranges, r.rem, ksteps, units, part_cost, max_parts);
  int best = t;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) best = min(best, __shfl_xor(best, o));
  // the fewest ranges of equals
  r.split = r.rem == 0 ? 1 : __builtin_ctzll(__builtin_amdgcn_ballot_w64(t == best)) + 1;
  return r;
}
// the tile rows that hold tokens and the launch's split
template <typename T, int TS>
__device__ __forceinline__ KdRounds dh_split(const DhArgs& a, int& n, int& TM) {
  n = a.nrow != nullptr ? min(a.rows, __builtin_amdgcn_readfirstlane(*a.nrow) - a.nrow_base) : a.rows;
  n = max(n, 0);
  TM = (n + TS - 1) / TS;
  if (a.nrow == nullptr) return a.sp;
  return split_rounds(TM * a.TN, a.ks_total, kd_units(TS), kd_part_cost(TS, sizeof(T) == 4),
                      kd_dh_max_parts(TM * a.TN, n, a.D, TS, a.part_space));
}

template <typename T, int TS>
__global__ __launch_bounds__(Geo<TS>::kThreads, TS == 256 ? 1 : 2) void k_dh(DhArgs a) {
  typedef Geo<TS> G;
  __shared__ __attribute__((aligned(16))) char lds[gemm_lds<T, TS>];
  int n, TM;
  const KdRounds sp = dh_split<T, TS>(a, n, TM);
  const int pid = blockIdx.x;
  int L, part = -1, kb = 0, ke = a.ks_total;  // part: of a split tile
  if (pid < sp.dp) {
    L = tile_order_xcd(pid, sp.dp);
  } else {
    // the last round: neighbours in the order take the same range of
    // neighbouring tiles, which share operand rows
    const int parts = sp.rem * sp.split;
    if (pid - sp.dp >= parts) return;
    const int q = tile_order_xcd(pid - sp.dp, parts);
    const int s = q / sp.rem;
    L = sp.dp + q - s * sp.rem;
    if (sp.split > 1) {
      part = s;
      kb = (int)((int64_t)a.ks_total * s / sp.split);
      ke = (int)((int64_t)a.ks_total * (s + 1) / sp.split);
    }
  }
  int mt, nt;
  tile_at(L, TM, a.TN, G::GM, mt, nt);
  const int m0 = mt * TS, n0 = nt * TS;
  const int D = a.D, rows = a.rows;
  const int eb = Elt<T>::bytes;
  const int lda = (int)(a.ldz * eb), ldb = D * eb;
  const T* dZ = static_cast<const T*>(a.dZ);
  AccTile<TS> acc;
  const int mrows = min(TS, rows - m0);
  // the row factors of the tile's rows, loaded before the main loop and
  // kept in LDS for the epilogue: a load there would wait for every store
  // issued before it (loads and stores complete in order)
  const int tid = threadIdx.x;
  const float rsv = (a.rowscale != nullptr && part < 0 && tid < TS && m0 + tid < rows)
                        ? a.rowscale[m0 + tid]
                        : 1.f;
  gemm<T, TS, true>(
      KcOp{reinterpret_cast<const char*>(dZ + (int64_t)m0 * a.ldz), (uint32_t)(mrows * lda), lda},
      KmOp{reinterpret_cast<const char*>(static_cast<const T*>(a.W) + n0),
           (int64_t)a.V * ldb - (int64_t)n0 * eb, ldb},
      kb, ke, lds, acc);
  const int lane = tid & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);
  if (part >= 0) {
    // into the range's [n, D] array or a tile of its own, rows past n out of the
    // resource's range; the wave's 64 columns all exist or none
    const bool rows_d = sp.dp == 0;
    const int pitch = rows_d ? D : TS;
    float* dst = a.partial + (rows_d ? ((int64_t)part * n + m0) * D + n0
                                     : (int64_t)((L - sp.dp) * sp.split + part) * TS * TS);
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(
        dst, 4u * (uint32_t)__builtin_amdgcn_readfirstlane(rows_d ? (n - m0) * D - n0
                                                                  : min(TS, n - m0) * TS));
    if (rows_d && n0 + wn * 64 >= D) return;
    const uint32_t o0 = 4u * (uint32_t)(G::acc_m(wm, 0, lane, 0) * pitch + G::acc_n(wn, 0, lane));
#pragma unroll
    for (int i = 0; i < G::NI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = acc.v[i][j][r];  // (a bit cast of the element itself takes element 0)
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), ro, o0 + 64u * j,
                                                4 * (16 * i + r) * pitch, 0);
        }
    return;
  }
  float* rsl = reinterpret_cast<float*>(lds);
  int* rml = reinterpret_cast<int*>(lds) + TS;
  if (tid < TS) {
    rsl[tid] = rsv;
    // the output row of each of the tile's rows (loaded here: nothing of the
    // unmasked call is kept live through the main loop for it)
    rml[tid] = (a.rowmap != nullptr && m0 + tid < rows) ? a.rowmap[m0 + tid] : m0 + tid;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < G::NI; ++i) {
    const f32x4_t sc = *reinterpret_cast<const f32x4_t*>(rsl + G::acc_m(wm, i, lane, 0));
    const i32x4_t om = *reinterpret_cast<const i32x4_t*>(rml + G::acc_m(wm, i, lane, 0));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int d = n0 + G::acc_n(wn, j, lane);
      if (d >= D) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (m0 + G::acc_m(wm, i, lane, r) >= rows) continue;
        const float v = acc.v[i][j][r] * sc[r];
        const int64_t o = om[r];  // the grad_hidden row
        if (o < 0) continue;
        if (a.gh_f32)
          static_cast<float*>(a.gH)[o * D + d] = v;
        else
          static_cast<T*>(a.gH)[o * D + d] = (T)v;
      }
    }
  }
}

// The split tiles of dH: their parts added in order, four features per thread.
template <typename T, int TS>
__device__ __forceinline__ void dh_reduce(int block, int blocks, const DhArgs& a) {
  int n, TM;
  const KdRounds sp = dh_split<T, TS>(a, n, TM);
  if (sp.split < 2) return;
  constexpr int Q = TS * TS / 4;  // pieces per tile
  const bool rows_d = sp.dp == 0;  // parts as [n, D] arrays
  const int total = rows_d ? n * (a.D / 4) : sp.rem * Q;
  const int64_t step = rows_d ? (int64_t)n * a.D : TS * TS;
  for (int i = block * 256 + (int)threadIdx.x; i < total; i += blocks * 256) {
    int t, d;
    const float* part = a.partial;
    if (rows_d) {
      t = i / (a.D / 4);
      d = i % (a.D / 4) * 4;
      part += (int64_t)i * 4;
    } else {
      const int q = i / Q, row = i % Q / (TS / 4), c = i % (TS / 4) * 4;
      int mt, nt;
      tile_at(sp.dp + q, TM, a.TN, Geo<TS>::GM, mt, nt);
      t = mt * TS + row;
      d = nt * TS + c;
      part += (int64_t)q * sp.split * (TS * TS) + row * TS + c;
    }
    if (t >= n || d >= a.D) continue;
    const int64_t o = a.rowmap != nullptr ? a.rowmap[t] : t;  // the grad_hidden row
    if (o < 0) continue;
    f32x4_t v = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int k = 0; k < sp.split; ++k) v += *reinterpret_cast<const f32x4_t*>(part + k * step);
    if (a.rowscale != nullptr) v *= a.rowscale[t];
    if (a.gh_f32 || sizeof(T) == 4) {
      *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.gH) + o * a.D + d) = v;
    } else {
      *reinterpret_cast<u32x2_t*>(static_cast<uint16_t*>(a.gH) + o * a.D + d) =
          u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    }
  }
}

// -------------------------------------------------------------------- dW ----
// The group's hidden rows transposed: Ht[d, t] = H[t, d] for t < tokens and 0
// for tokens <= t < ldt (ldt a multiple of 64), so that the dW contraction
// reads them with the tokens (its K dimension) contiguous. One 64 x 64 block
// per workgroup, 16-byte loads and stores on both sides. With a rowmap,
// column t is hidden row rowmap[t] (-1: zeros).
template <typename T>
__device__ __forceinline__ void transpose_rows(int bt, int bd, const T* __restrict__ H, int tokens,
                                               int D, T* __restrict__ Ht, int ldt,
                                               const float* __restrict__ rowscale,
                                               const int* __restrict__ rowmap) {
  constexpr int VPT = 16 / (int)sizeof(T);      // elements per 16-byte piece
  constexpr int PAD = 4 / (int)sizeof(T);       // one dword of padding per LDS row
  __shared__ T tile[64][64 + PAD];              // [token][feature]
  const int t0 = bt * 64, d0 = bd * 64;
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < 64 * 64 / VPT / 256; ++u) {
    const int q = tid + 256 * u;
    const int row = q / (64 / VPT), c = (q % (64 / VPT)) * VPT;
    u32x4_t v = u32x4_t{0u, 0u, 0u, 0u};
    const int64_t src = t0 + row >= tokens ? -1 : rowmap != nullptr ? rowmap[t0 + row] : t0 + row;
    if (src >= 0) v = *reinterpret_cast<const u32x4_t*>(H + src * D + d0 + c);
    T e[VPT];
    __builtin_memcpy(e, &v, 16);
    // a per-token factor of the gradient rows is applied to the hidden rows
    // here, so that dW = sum_t (factor_t H_t)^T dZ''_t
    const float f = (rowscale != nullptr && t0 + row < tokens) ? rowscale[t0 + row] : 1.f;
#pragma unroll
    for (int x = 0; x < VPT; ++x) tile[row][c + x] = rowscale ? (T)((float)e[x] * f) : e[x];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 64 * 64 / VPT / 256; ++u) {
    const int q = tid + 256 * u;
    const int d = q / (64 / VPT), c = (q % (64 / VPT)) * VPT;
    T e[VPT];
#pragma unroll
    for (int x = 0; x < VPT; ++x) e[x] = tile[c + x][d];
    u32x4_t v;
    __builtin_memcpy(&v, e, 16);
    *reinterpret_cast<u32x4_t*>(Ht + (int64_t)(d0 + d) * ldt + t0 + c) = v;
  }
}

// What is left between a group's dH and its dW, in one launch: blocks
// [0, nt) transpose the hidden rows for dW, the next nr add up the parts of a
// split dH, and one more forms the loss after the last chunk.
struct TailArgs {
  int nt, nr;
  // transpose
  const void* H;
  int tokens, D;
  void* Ht;
  int ldt;
  const float* rowscale;
  const int* rowmap;
  DhArgs dh;  // the dH launch whose parts are added up
  // loss
  const float* block_partial;
  int n_partials;
  const float* inv_nvalid;  // null: inv_n
  float inv_n;
  float* loss;
};
template <typename T, int DTS>
__global__ __launch_bounds__(256) void k_tail(TailArgs a) {
  const int b = blockIdx.x;
  if (b < a.nt) {
    const int td = a.D / 64;
    transpose_rows<T>(b / td, b % td, static_cast<const T*>(a.H), a.tokens, a.D,
                      static_cast<T*>(a.Ht), a.ldt, a.rowscale, a.rowmap);
  } else if (b < a.nt + a.nr) {
    dh_reduce<T, DTS>(b - a.nt, a.nr, a.dh);
  } else {
    finalize_loss(a.block_partial, a.n_partials, a.inv_nvalid ? a.inv_nvalid[0] : a.inv_n, a.loss);
  }
}

// grad_W[v, d] (+)= sum_t dZ[t, v] H[t, d] over the tokens of a group of
// chunks, computed as the tile C[d, v] = Ht[d, :] dZ[:, v]: A = the transposed
// hidden rows (K = tokens contiguous, zero past the group), B = dZ read
// K-major (rows = tokens; rows past the group read as zeros). Lane (g, c) of
// a wave holds C at four consecutive d of one v for each block, i.e. 16
// contiguous bytes of a grad_W row, so the tile goes to memory straight from
// the accumulators: with beta = 1 one half of the tile's old values is loaded,
// added, and the other half's loads are issued before the first half's stores
// (loads and stores complete in issue order, so waiting for those loads does
// not wait for the stores).
//
// SPLIT (for a tile count that leaves the last round of the compute units
// partly filled, or few tiles): blocks [0, nfull) compute the whole tiles of
// the full rounds, and the tiles left over are split into `split` token ranges
// (kd_split_rounds), neighbours in the order taking the same range of
// neighbouring tiles; range s of tile nfull + q is stored as an fp32 partial
// tile (pitch TS) at slot split q + s, and k_dw_fixup adds the parts to grad_W
// in a fixed order. Without SPLIT every block computes a whole tile (nfull,
// split and partial unused).
//
// With nrow (ignored tokens left out), only the group's first *nrow dZ rows
// hold tokens: the K range stops there, and the dZ rows past it read as
// zeros. The split is then the model's for that K range, at most the launch's:
// parts of a few steps cost more in partial tiles than they fill the chip
// (fwd and bwd of 11343 x 128 x 22099 with 12 tokens left: 124 us, now 114).
template <typename T>
__device__ __forceinline__ int dw_steps(int tokens, int ldt, const int* nrow) {
  constexpr int KS = kRowB / (int)sizeof(T);
  if (nrow != nullptr) tokens = min(tokens, __builtin_amdgcn_readfirstlane(*nrow));
  return min(ldt / KS, (tokens + KS - 1) / KS);
}
template <typename T, int TS>
__device__ __forceinline__ int dw_split(int split, int nks, int tiles, int nfull, const int* nrow) {
  if (nrow == nullptr) return split;
  return split_rounds(tiles, nks, kd_units(TS), kd_part_cost(TS, sizeof(T) == 4),
                      (tiles - nfull) * split)
      .split;
}
template <typename T, int TS, bool SPLIT>
__global__ __launch_bounds__(Geo<TS>::kThreads, TS == 256 ? 1 : 2) void k_dw(const T* __restrict__ Ht, int ldt,
                                                    const T* __restrict__ dZ, int64_t ldz,
                                                    int tokens, int V, int D, int TM, int TN,
                                                    int beta, float* __restrict__ gW, int nfull,
                                                    int split, float* __restrict__ partial,
                                                    const int* __restrict__ nrow) {
  typedef Geo<TS> G;
  constexpr int NI = G::NI;
  __shared__ __attribute__((aligned(16))) char lds[gemm_lds<T, TS>];
  const int nks = dw_steps<T>(tokens, ldt, nrow);
  if (nrow != nullptr) tokens = min(tokens, __builtin_amdgcn_readfirstlane(*nrow));
  const int pid = blockIdx.x;
  int L, ks0 = 0, ks1 = nks, slot = -1;
  if (!SPLIT) {
    L = tile_order_xcd(pid, TM * TN);
  } else if (pid < nfull) {
    L = tile_order_xcd(pid, nfull);
  } else {
    const int rem = TM * TN - nfull;
    split = dw_split<T, TS>(split, nks, TM * TN, nfull, nrow);
    if (pid - nfull >= rem * split) return;
    const int o = tile_order_xcd(pid - nfull, rem * split);
    const int s = o / rem, q = o - s * rem;
    L = nfull + q;
    if (split > 1) {
      slot = q * split + s;
      ks0 = (int)((int64_t)nks * s / split);
      ks1 = (int)((int64_t)nks * (s + 1) / split);
    }
  }
  int mt, nt;
  tile_at(L, TM, TN, G::GM, mt, nt);
  const int m0 = mt * TS, n0 = nt * TS;  // m: feature d, n: vocabulary v
  const int eb = Elt<T>::bytes;
  const int lda = ldt * eb, ldb = (int)(ldz * eb);
  const int mrows = min(TS, D - m0);
  AccTile<TS> acc;
  gemm<T, TS, true>(
      KcOp{reinterpret_cast<const char*>(Ht + (int64_t)m0 * ldt), (uint32_t)(mrows * lda), lda},
      KmOp{reinterpret_cast<const char*>(dZ + n0), (int64_t)tokens * ldb - (int64_t)n0 * eb, ldb},
      ks0, ks1, lds, acc);
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);
  // the tile's rows of grad_W (or of its partial slot, pitch TS) as one
  // resource: rows past V are out of range (loads give 0, stores are
  // dropped), features past D get an out-of-range offset
  const bool part = SPLIT && slot >= 0;
  const int pitch = part ? TS : D;
  const int vrows = __builtin_amdgcn_readfirstlane(part ? TS : min(TS, V - n0));
  const __amdgpu_buffer_rsrc_t ro =
      part ? make_rsrc(partial + (int64_t)slot * TS * TS, (uint32_t)TS * TS * 4u)
           : make_rsrc(gW + (int64_t)n0 * D, (uint32_t)vrows * (uint32_t)D * 4u);
  // block (i, j) sits at byte offset obase + 64 i (16 features) + 64 pitch j
  // (16 rows): the per-lane part is one register, 64 i goes into the
  // instruction's immediate offset and 64 pitch j into its scalar offset. D
  // is a multiple of 64, so whether block i's features exist is the same for
  // the whole wave.
  const int dw0 = (part ? 0 : m0) + wm * 16 * NI;
  const uint32_t obase =
      ((uint32_t)G::acc_n(wn, 0, lane) * (uint32_t)pitch + (uint32_t)(dw0 + 4 * (lane >> 4))) * 4u;
  const uint32_t jstep = 64u * (uint32_t)pitch;
  auto ld = [&](int i, int j) {
    return __builtin_bit_cast(
        f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(ro, obase + 64u * i, jstep * j, 0));
  };
  auto st = [&](int i, int j, f32x4_t v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), ro, obase + 64u * i,
                                           jstep * j, 0);
  };
  auto live = [&](int i) { return part || dw0 + 16 * i < D; };
  if (beta && !part) {
    f32x4_t old[NI / 2][4];
#pragma unroll
    for (int i = 0; i < NI / 2; ++i)
      if (live(i))
#pragma unroll
        for (int j = 0; j < 4; ++j) old[i][j] = ld(i, j);
#pragma unroll
    for (int i = 0; i < NI / 2; ++i)
      if (live(i))
#pragma unroll
        for (int j = 0; j < 4; ++j) acc.v[i][j] += old[i][j];
#pragma unroll
    for (int i = 0; i < NI / 2; ++i)
      if (live(NI / 2 + i))
#pragma unroll
        for (int j = 0; j < 4; ++j) old[i][j] = ld(NI / 2 + i, j);
#pragma unroll
    for (int i = 0; i < NI / 2; ++i)
      if (live(i))
#pragma unroll
        for (int j = 0; j < 4; ++j) st(i, j, acc.v[i][j]);
#pragma unroll
    for (int i = 0; i < NI / 2; ++i)
      if (live(NI / 2 + i))
#pragma unroll
        for (int j = 0; j < 4; ++j) st(NI / 2 + i, j, acc.v[NI / 2 + i][j] + old[i][j]);
  } else {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (live(i))
#pragma unroll
        for (int j = 0; j < 4; ++j) st(i, j, acc.v[i][j]);
  }
}

// The split tail tiles of k_dw: grad_W = (beta ? grad_W : 0) + (part 0 + part 1
// + ...), the parts in this order. One thread per 4 features of a vocabulary row of a tail
// tile (grid: tail tiles x blocks of rows).
template <typename T, int TS>
__global__ __launch_bounds__(256) void k_dw_fixup(const float* __restrict__ partial, int split,
                                                  int nfull, int TM, int TN, int V, int D,
                                                  int beta, float* __restrict__ gW, int tokens,
                                                  int ldt, const int* __restrict__ nrow) {
  split = dw_split<T, TS>(split, dw_steps<T>(tokens, ldt, nrow), TM * TN, nfull, nrow);
  if (split < 2) return;
  const int q = blockIdx.x;                      // tail tile
  constexpr int TPR = TS / 4;                    // threads per row
  const int row = blockIdx.y * (256 / TPR) + threadIdx.x / TPR;
  const int c4 = (threadIdx.x % TPR) * 4;        // first of 4 features in the tile
  int mt, nt;
  tile_at(nfull + q, TM, TN, Geo<TS>::GM, mt, nt);
  const int v = nt * TS + row, d = mt * TS + c4;
  if (v >= V || d >= D) return;
  f32x4_t sum = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll kDwMaxSplit
  for (int s = 0; s < split; ++s)
    sum += *reinterpret_cast<const f32x4_t*>(partial + ((int64_t)(q * split + s) * TS + row) * TS + c4);
  if (beta) sum += *reinterpret_cast<const f32x4_t*>(gW + (int64_t)v * D + d);
  *reinterpret_cast<f32x4_t*>(gW + (int64_t)v * D + d) = sum;
}

// ------------------------------------------------- ignored tokens left out --
// The tokens of a dW group [row0, row0 + rows) that are not ignored, in
// order: rowmap[j] = the j-th of them, -1 for j >= their count, *nrow = the
// count. One workgroup: thread i counts a contiguous run of the mask (16 bytes
// at a time where they are aligned), an exclusive scan of the counts over the
// threads gives each run its first slot. With inv_nvalid (the call's first
// group), N_valid of the whole mask [0, N) is counted as well and 1/N_valid
// (0 if none) written.
constexpr int kScanThreads = 1024;
__device__ __forceinline__ int zero_bytes(uint32_t v) {
  return ((v & 0xffu) == 0u) + ((v & 0xff00u) == 0u) + ((v & 0xff0000u) == 0u) +
         ((v & 0xff000000u) == 0u);
}
// zero bytes of [b, e)
__device__ __forceinline__ int count_zero(const uint8_t* m, int64_t b, int64_t e) {
  int c = 0;
  while (b < e && ((uintptr_t)(m + b) & 15u) != 0u) c += m[b++] == 0 ? 1 : 0;
#pragma unroll 4
  for (; b + 16 <= e; b += 16) {
    const u32x4_t w = *reinterpret_cast<const u32x4_t*>(m + b);
    c += (zero_bytes(w[0]) + zero_bytes(w[1])) + (zero_bytes(w[2]) + zero_bytes(w[3]));
  }
  while (b < e) c += m[b++] == 0 ? 1 : 0;
  return c;
}
__global__ __launch_bounds__(kScanThreads) void k_compact_scan(const uint8_t* __restrict__ ignore,
                                                               int64_t N, int64_t row0, int rows,
                                                               int* __restrict__ rowmap,
                                                               int* __restrict__ nrow,
                                                               float* __restrict__ inv_nvalid) {
  constexpr int NWV = kScanThreads / 64;
  __shared__ int sc[NWV], all[NWV];
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  // long runs are a multiple of 16 tokens: aligned when the mask is
  int per = (rows + kScanThreads - 1) / kScanThreads;
  if (per > 8) per = (per + 15) & ~15;
  const int b = (int)min((int64_t)rows, (int64_t)tid * per), e = min(rows, b + per);
  const uint8_t* m = ignore + row0;
  const int c = count_zero(m, b, e);
  const int incl = wave_incl_scan(c);
  if (lane == 63) sc[wave] = incl;
  const bool count = inv_nvalid != nullptr && rows < N;  // else the group is the whole mask
  if (count) {
    const int64_t per_all = ((N + kScanThreads - 1) / kScanThreads + 15) & ~(int64_t)15;
    const int64_t b0 = min(N, tid * per_all);
    int n = count_zero(ignore, b0, min(N, b0 + per_all));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o);
    if (lane == 0) all[wave] = n;
  }
  __syncthreads();
  int pos = incl - c, total = 0;
  for (int w = 0; w < NWV; ++w) {
    if (w < wave) pos += sc[w];
    total += sc[w];
  }
  for (int i = b; i < e; ++i)
    if (m[i] == 0) rowmap[pos++] = (int)(row0 + i);
  for (int j = total + tid; j < rows; j += kScanThreads) rowmap[j] = -1;
  if (tid == 0) {
    nrow[0] = total;
    if (inv_nvalid != nullptr) {
      int n = count ? 0 : total;
      for (int w = 0; w < (count ? NWV : 0); ++w) n += all[w];
      inv_nvalid[0] = n > 0 ? 1.0f / (float)n : 0.0f;
    }
  }
}

// ------------------------------------------------------------ index check --
// flag |= 1 if an index is outside [0, V); |= 2 if a row repeats an index.
__global__ void k_check_indices(const int32_t* idx, int64_t N, int K, int64_t V, int* flag) {
  const int64_t r = (int64_t)blockIdx.x * 4 + wave_id();
  const int lane = threadIdx.x & 63;
  if (r >= N) return;
  const int32_t* row = idx + r * K;
  int bad = 0;
  for (int k = lane; k < K; k += 64) {
    const int32_t v = row[k];
    if (v < 0 || (int64_t)v >= V) bad |= 1;
    for (int k2 = k + 1; k2 < K; ++k2)
      if (row[k2] == v) bad |= 2;
  }
  if (bad) atomicOr(flag, bad);
}


// ------------------------------------------------- upstream-gradient scale --
// y = g x elementwise, g a device scalar: the gradients of the mean loss
// times the upstream gradient of that mean (Algorithm 1's backward scales G
// by g; the loss is linear in g, so scaling the finished gradients is the
// same function). fp32 in; out in fp32 or bf16 (one rounding); in place when
// x and y are the same fp32 buffer. Bound by memory (2.36 GB of a 128256 x
// 3072 grad_W to bf16: 0.47 ms); both gradients share a launch, the first
// `blocks0` blocks taking the first. Each thread handles 8 elements, 16-byte
// accesses where the 8 are in range (the buffers are 16-byte aligned).
struct ScaleArg {
  const float* x;
  void* y;
  int64_t n;
  int bf16;
};
template <typename TO>
__device__ __forceinline__ void scale_f32(const float* x, TO* y, int64_t n, float s, int block,
                                          int blocks) {
  const int64_t stride = (int64_t)blocks * blockDim.x * 8;
  for (int64_t i = ((int64_t)block * blockDim.x + threadIdx.x) * 8; i < n; i += stride) {
    if (i + 8 <= n) {
      const f32x4_t a = *reinterpret_cast<const f32x4_t*>(x + i) * s;
      const f32x4_t b = *reinterpret_cast<const f32x4_t*>(x + i + 4) * s;
      if constexpr (sizeof(TO) == 2) {
        *reinterpret_cast<u32x4_t*>(y + i) =
            u32x4_t{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]),
                    pack_bf16x2(b[2], b[3])};
      } else {
        *reinterpret_cast<f32x4_t*>(y + i) = a;
        *reinterpret_cast<f32x4_t*>(y + i + 4) = b;
      }
    } else {
      for (int64_t k = i; k < n; ++k) y[k] = (TO)(x[k] * s);
    }
  }
}
__global__ void k_scale(ScaleArg a, ScaleArg b, int blocks0, const float* __restrict__ g) {
  const float s = g[0];
  const bool first = (int)blockIdx.x < blocks0;
  const ScaleArg c = first ? a : b;
  if (s == 1.f && c.x == c.y) return;  // in place by 1: the values stay
  const int block = first ? blockIdx.x : blockIdx.x - blocks0;
  const int blocks = first ? blocks0 : gridDim.x - blocks0;
  if (c.bf16)
    scale_f32(c.x, static_cast<__bf16*>(c.y), c.n, s, block, blocks);
  else
    scale_f32(c.x, static_cast<float*>(c.y), c.n, s, block, blocks);
}

}  // namespace kd

// ================================================================ launchers ==
using namespace kd;

#include <atomic>
#include <mutex>
#include <vector>

#include "../../include/kdtopk.h"

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------- event instrumentation ----
namespace {
enum ProfKind {
  P_PREP, P_LOGITS, P_MERGE, P_DZ, P_ROW_LOSS, P_DH, P_DW, P_TAIL, P_FILL,
  P_LOGITS_DZ, P_ROW_FINISH, P_DW_FIXUP, P_COMPACT, P_NKINDS
};
const char* const kProfNames[P_NKINDS] = {
    "prep", "logits_lse", "lse_merge", "dz", "row_loss", "dh", "dw", "tail", "fill",
    "logits_dz", "row_finish", "dw_fixup", "compact"};
struct ProfRec {
  int kind;
  hipEvent_t a, b;
  double flops;
};
std::atomic<int> g_prof_mode{0};  // 0 off, 1 every kernel, 2 contractions only
// set while the allocation-free entry point enqueues: no events are created
thread_local bool t_prof_suppressed = false;
std::mutex g_prof_mu;
std::vector<ProfRec> g_prof_recs;
std::vector<hipEvent_t> g_prof_pool;

hipEvent_t prof_event() {
  if (!g_prof_pool.empty()) {
    hipEvent_t e = g_prof_pool.back();
    g_prof_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Records an event pair around the launches in its scope when enabled.
struct ProfScope {
  int kind;
  double flops;
  hipStream_t s;
  hipEvent_t a = nullptr;
  ProfScope(int k, double f, hipStream_t st) : kind(k), flops(f), s(st) {
    const int mode = g_prof_mode.load(std::memory_order_relaxed);
    if (mode == 0 || (mode == 2 && f == 0.0) || t_prof_suppressed) return;
    std::lock_guard<std::mutex> g(g_prof_mu);
    a = prof_event();
    if (a) (void)hipEventRecord(a, s);
  }
  ~ProfScope() {
    if (!a) return;
    std::lock_guard<std::mutex> g(g_prof_mu);
    hipEvent_t b = prof_event();
    if (!b) {
      g_prof_pool.push_back(a);  // no pair: drop this record, keep the event
      return;
    }
    (void)hipEventRecord(b, s);
    g_prof_recs.push_back({kind, a, b, flops});
  }
};
}  // namespace

extern "C" kd_status kd_profile_enable(int mode) {
  if (mode < 0 || mode > 2) return KD_ERR_BAD_ARG;
  g_prof_mode.store(mode);
  return KD_OK;
}

extern "C" int kd_profile_read(kd_kernel_time* out, int max) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  double ms[P_NKINDS] = {0}, fl[P_NKINDS] = {0};
  int64_t n[P_NKINDS] = {0};
  int rc = 0;
  for (const ProfRec& r : g_prof_recs) {
    float t = 0.f;
    if (hipEventSynchronize(r.b) != hipSuccess || hipEventElapsedTime(&t, r.a, r.b) != hipSuccess)
      rc = -1;
    ms[r.kind] += t;
    fl[r.kind] += r.flops;
    n[r.kind] += 1;
    g_prof_pool.push_back(r.a);
    g_prof_pool.push_back(r.b);
  }
  g_prof_recs.clear();
  if (rc != 0) return rc;
  int w = 0;
  for (int k = 0; k < P_NKINDS && w < max; ++k) {
    if (n[k] == 0) continue;
    kd_kernel_time& o = out[w++];
    memset(o.name, 0, sizeof(o.name));
    strncpy(o.name, kProfNames[k], sizeof(o.name) - 1);
    o.launches = n[k];
    o.total_ms = ms[k];
    o.flops = fl[k];
  }
  return w;
}

// One projection launch: `count` 256x256 tiles from `first` on of the order
// (see ProjTiles). Vocabulary tiles go up to the padded width: every column of
// dZ is written.
template <typename T, int TS>
static void launch_projection(const KdChunkArgs& a, int first, int count, hipStream_t s) {
  if (count <= 0) return;
  const T* W = static_cast<const T*>(a.W);
  const T* Hc = static_cast<const T*>(a.Hc);
  const int TN = cdiv(a.rows, kTile);
  const ProjTiles t{a.nVT, TN, first, count, a.nP};
  const dim3 grid(count * (kTile / TS) * (kTile / TS)), block(Geo<TS>::kThreads);
  const float k2 = kLog2e * a.inv_tau;
  const double flops = 2.0 * (double)a.rows * (double)a.D * (double)a.V * count / (a.nVT * TN);
  if (a.one_projection) {
    ProfScope ps_(P_LOGITS_DZ, flops, s);
    hipLaunchKernelGGL((k_logits_dz<T, TS>), grid, block, 0, s, W, Hc, (int)a.D, (int)a.V, a.rows,
                       t, k2, a.part_m, a.part_s, a.nVT, a.hits, a.hoff, a.K,
                       static_cast<T*>(a.dZ), a.ldz, a.zhit, a.rowR, a.rowFlag, a.nrow,
                       a.nrow_base);
  } else if (a.mode != KD_MODE_BWD) {
    // no recompute follows (forward only, or a fused call that wants no
    // gradients): z at the teacher entries comes from this GEMM
    ProfScope ps_(P_LOGITS, flops, s);
    hipLaunchKernelGGL((k_logits_lse<T, TS>), grid, block, 0, s, W, Hc, (int)a.D, (int)a.V, a.rows,
                       t, k2, a.part_m, a.part_s, a.nVT, a.hits, a.hoff, a.K, a.zhit, a.nrow,
                       a.nrow_base);
  } else {
    // the backward of the split entry points: the logit recompute from the
    // saved log Z (Algorithm 1's backward)
    ProfScope ps_(P_DZ, flops, s);
    hipLaunchKernelGGL((k_dz<T, TS>), grid, block, 0, s, W, Hc, (int)a.D, (int)a.V, a.rows, t, k2,
                       a.rowL2, a.rowCoef, a.rowCoefM, a.hits, a.hitp, a.hoff, a.K, a.nVT,
                       static_cast<T*>(a.dZ), a.ldz, a.nrow, a.nrow_base);
  }
}

template <typename T>
static int launch_chunk_impl(const KdChunkArgs& a, hipStream_t s) {
  const int nbt = cdiv(a.rows, kTile);  // 256-token tiles (of the buckets too)
  const float k2 = kLog2e * a.inv_tau;
  const bool fwd = a.mode != KD_MODE_BWD;
  if (a.stages & KD_STAGE_PREP) {
    {
      ProfScope ps_(P_PREP, 0.0, s);
      PrologueArgs p{};
      p.tidx = a.tidx_in;
      p.tidx_out = a.tidx;
      p.tlogit = a.tlogit;
      p.ignore = a.ignore;
      p.row0 = a.row0;
      p.rowmap = a.rowmap;
      p.rows = a.rows;
      p.K = a.K;
      p.V = (int)a.V;
      p.D = (int)a.D;
      p.inv_tau = a.inv_tau;
      p.logprobs = a.teacher_logprobs;
      p.inv_nvalid = a.inv_nvalid;
      p.inv_n = a.inv_n;
      p.gscale = a.gscale;
      p.gtok = a.gtok;
      p.logz_in = fwd ? nullptr : a.logz_in;
      p.p_out = a.p;
      p.rowM = a.rowM;
      p.rowH = a.rowH;
      p.rowCoef = a.rowCoef;
      p.rowCoefM = a.rowCoefM;
      p.rowL2 = a.rowL2;
      p.hidden = a.hidden;
      p.W = a.W;
      p.k2 = k2;
      p.rowR = a.one_projection ? a.rowR : nullptr;
      p.rowFlag = a.rowFlag;
      p.hcomp = static_cast<char*>(const_cast<void*>(a.Hc));
      p.gH = static_cast<char*>(a.grad_hidden);
      p.gh_row_bytes = a.D * (a.gh_f32 ? 4 : (int64_t)sizeof(T));
      p.lpt = a.lpt_full;
      p.logz_out = a.logz_out;
      BucketArgs b{};
      b.tidx = a.tidx;
      b.p = a.p;
      b.rows = a.rows;
      b.K = a.K;
      b.V = (int)a.V;
      b.nVT = a.nVT;
      b.hits = a.hits;
      b.hitp = fwd ? nullptr : a.hitp;
      b.hoff = a.hoff;
      b.zhit = a.zhit;
      if (fwd && a.K <= kPrepMaxK) {
        b.tidx = a.rowmap != nullptr ? a.tidx_in : a.tidx_in + a.row0 * a.K;
        b.rowmap = a.rowmap;
        hipLaunchKernelGGL(k_prep<T>, dim3(nbt + cdiv(a.rows, kBucketThreads / 64)),
                           dim3(kBucketThreads), 0, s, p, b, nbt);
      } else {
        hipLaunchKernelGGL(k_prologue<T>, dim3(a.rows), dim3(64), (size_t)prologue_lds(a.K), s, p);
        const bool one = std::min(a.rows, kTile) * a.K <= kBucketThreads * kBucketRegs;
        hipLaunchKernelGGL(one ? k_bucket<true> : k_bucket<false>, dim3(nbt), dim3(kBucketThreads),
                           0, s, b);
      }
    }
  }
  if (!(a.stages & KD_STAGE_CHUNK)) return (int)hipGetLastError();
  // bf16: whole 256x256 tiles, and the order's last ones as 128x128 tiles
  const int large = sizeof(T) == 2 ? a.large_tiles : 0;
  if constexpr (sizeof(T) == 2) launch_projection<T, 256>(a, 0, large, s);
  launch_projection<T, 128>(a, large, a.nVT * nbt - large, s);
  if (a.one_projection) {
    // the merge of log Z with the row factors, the fallback rows, the teacher
    // cells and the row losses
    ProfScope ps_(P_ROW_FINISH, 0.0, s);
    hipLaunchKernelGGL(k_row_finish<T>, dim3(cdiv(a.rows, kLossRows)), dim3(64 * kLossRows), 0, s,
                       a.part_m, a.part_s, a.nP, a.nP == a.nVT ? 8 : 7, a.rowFlag,
                       static_cast<T*>(a.dZ), a.ldz, a.tidx, a.p, a.zhit, a.K, (int)a.V, k2,
                       a.rowM, a.rowH, a.rowCoef, a.rowCoefM, a.ignore, a.row0, a.rowmap, a.rows,
                       a.inv_tau, a.rowL2, a.rowFactor, a.loss_per_token, a.block_partial);
  } else if (fwd) {
    {
      ProfScope ps_(P_MERGE, 0.0, s);
      hipLaunchKernelGGL(k_lse_merge, dim3(cdiv(a.rows, 4)), dim3(256), 0, s, a.part_m, a.part_s,
                         a.rows, a.nP, a.rowL2, a.rowmap);
    }
    {
      ProfScope ps_(P_ROW_LOSS, 0.0, s);
      hipLaunchKernelGGL(k_row_loss, dim3(cdiv(a.rows, kLossRows)), dim3(64 * kLossRows), 0, s,
                         a.zhit, a.p, a.K, a.rowL2, a.rowM, a.rowH, a.ignore, a.row0, a.rowmap,
                         a.rows, a.inv_tau, a.loss_per_token, a.logz_out, a.block_partial);
    }
  }
  return (int)hipGetLastError();
}

extern "C" int kd_launch_chunk(const KdChunkArgs* a, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  return a->dtype == 1 ? launch_chunk_impl<__bf16>(*a, s) : launch_chunk_impl<float>(*a, s);
}

template <typename T, int TS>
static DhArgs dh_args(const KdDhArgs& a) {
  DhArgs d{};
  d.dZ = a.dZ;
  d.ldz = a.ldz;
  d.W = a.W;
  d.V = (int)a.V;
  d.rows = (int)a.tokens;
  d.D = (int)a.D;
  d.TN = cdiv(a.D, TS);
  d.ks_total = (int)(a.ldz * sizeof(T) / kRowB);
  d.gH = a.gH;
  d.gh_f32 = a.gh_f32;
  d.partial = a.partial;
  d.part_space = a.part_space;
  d.rowscale = a.rowscale;
  d.rowmap = a.rowmap;
  d.nrow = a.nrow;
  d.nrow_base = a.nrow_base;
  d.sp = kd_dh_rounds((int)a.tokens, (int)a.D, TS, d.ks_total, sizeof(T) == 4, a.part_space);
  return d;
}

template <typename T, int TS>
static int launch_dh_impl(const KdDhArgs& a, hipStream_t s) {
  const DhArgs d = dh_args<T, TS>(a);
  const int blocks = a.nrow == nullptr ? d.sp.dp + d.sp.rem * d.sp.split
                                       : kd_dh_blocks((int)a.tokens, (int)a.D, TS, d.ks_total,
                                                      sizeof(T) == 4, a.part_space);
  {
    ProfScope ps_(P_DH, 2.0 * (double)a.tokens * (double)a.D * (double)a.V, s);
    hipLaunchKernelGGL((k_dh<T, TS>), dim3(blocks), dim3(Geo<TS>::kThreads), 0, s, d);
  }
  return (int)hipGetLastError();
}

extern "C" int kd_launch_dh(const KdDhArgs* a, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a->dtype != 1) return launch_dh_impl<float, 128>(*a, s);
  return a->tile == 128 ? launch_dh_impl<__bf16, 128>(*a, s) : launch_dh_impl<__bf16, 256>(*a, s);
}

template <typename T, int TS>
static int launch_dw_impl(const KdDwArgs& a, hipStream_t s) {
  const int ldt = (int)(((a.tokens + 63) / 64) * 64);
  const T* Ht = static_cast<const T*>(a.Ht);
  constexpr int units = kd_units(TS);
  constexpr int kThreads = Geo<TS>::kThreads;
  const int TM = cdiv(a.D, TS), TN = cdiv(a.V, TS);
  const int tiles = TM * TN;
  // the last round is split along the tokens when the model says so and the
  // host provides the partial tiles' workspace
  const int nks = ldt * (int)sizeof(T) / kRowB;
  const KdRounds sp =
      kd_split_rounds(tiles, nks, units, kd_part_cost(TS, sizeof(T) == 4), a.max_parts);
  const int split = sp.split, nfull = split > 1 ? sp.dp : tiles;
  {
    ProfScope ps_(P_DW, 2.0 * (double)a.tokens * (double)a.D * (double)a.V, s);
    if (nfull < tiles)
      hipLaunchKernelGGL((k_dw<T, TS, true>), dim3(nfull + (tiles - nfull) * split), dim3(kThreads),
                         0, s, Ht, ldt, static_cast<const T*>(a.dZ), a.ldz,
                         (int)a.tokens, (int)a.V, (int)a.D, TM, TN, a.beta, a.gW, nfull, split,
                         a.partial, a.nrow);
    else
      hipLaunchKernelGGL((k_dw<T, TS, false>), dim3(tiles), dim3(kThreads), 0, s,
                         Ht, ldt, static_cast<const T*>(a.dZ), a.ldz,
                         (int)a.tokens, (int)a.V, (int)a.D, TM, TN, a.beta, a.gW, tiles, 1,
                         (float*)nullptr, a.nrow);
  }
  if (nfull < tiles) {
    ProfScope ps_(P_DW_FIXUP, 0.0, s);
    hipLaunchKernelGGL((k_dw_fixup<T, TS>), dim3(tiles - nfull, TS * TS / 1024), dim3(256), 0, s,
                       a.partial, split, nfull, TM, TN, (int)a.V, (int)a.D, a.beta, a.gW,
                       (int)a.tokens, ldt, a.nrow);
  }
  return (int)hipGetLastError();
}

extern "C" int kd_launch_dw(const KdDwArgs* a, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a->dtype != 1) return launch_dw_impl<float, 128>(*a, s);
  return a->tile == 128 ? launch_dw_impl<__bf16, 128>(*a, s) : launch_dw_impl<__bf16, 256>(*a, s);
}

template <typename T, int DTS>
static int launch_tail_impl(const KdTailArgs& a, hipStream_t s) {
  TailArgs t{};
  if (a.Ht != nullptr) {
    t.H = a.Hg;
    t.tokens = (int)a.tokens;
    t.Ht = a.Ht;
    t.ldt = (int)(((a.tokens + 63) / 64) * 64);
    t.rowscale = a.rowscale;
    t.rowmap = a.rowmap;
    t.nt = t.ldt / 64 * (int)(a.D / 64);
  }
  t.D = (int)a.D;
  if (a.dh != nullptr && a.dh->part_space > 0) {
    t.dh = dh_args<T, DTS>(*a.dh);
    const int rem = a.dh->nrow != nullptr ? std::min(cdiv(a.dh->tokens, DTS) * t.dh.TN, kd_units(DTS))
                    : t.dh.sp.split > 1   ? t.dh.sp.rem
                                          : 0;
    t.nr = std::min(rem * (DTS * DTS / 1024), 4096);
  }
  if (a.loss != nullptr) {
    t.block_partial = a.block_partial;
    t.n_partials = a.n_partials;
    t.inv_nvalid = a.inv_nvalid;
    t.inv_n = a.inv_n;
    t.loss = a.loss;
  }
  const int blocks = t.nt + t.nr + (a.loss != nullptr ? 1 : 0);
  if (blocks == 0) return 0;
  {
    ProfScope ps_(P_TAIL, 0.0, s);
    hipLaunchKernelGGL((k_tail<T, DTS>), dim3(blocks), dim3(256), 0, s, t);
  }
  return (int)hipGetLastError();
}

extern "C" int kd_launch_tail(const KdTailArgs* a, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a->dtype != 1) return launch_tail_impl<float, 128>(*a, s);
  return a->dh != nullptr && a->dh->tile == 128 ? launch_tail_impl<__bf16, 128>(*a, s)
                                                : launch_tail_impl<__bf16, 256>(*a, s);
}

extern "C" int kd_launch_compact(const KdCompactArgs* a, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a->rows <= 0) return 0;
  {
    ProfScope ps_(P_COMPACT, 0.0, s);
    hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(kScanThreads), 0, s, a->ignore, a->N, a->row0,
                       a->rows, a->rowmap, a->nrow, a->inv_nvalid);
  }
  return (int)hipGetLastError();
}

extern "C" int kd_launch_fill(float* p, int64_t n, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  {
    ProfScope ps_(P_FILL, 0.0, s);
    hipLaunchKernelGGL(k_fill_f32, dim3(std::min<int64_t>(cdiv(n, 256), 16384)), dim3(256), 0, s, p,
                       n, 0.0f);
  }
  return (int)hipGetLastError();
}

extern "C" int kd_launch_check_indices(const int32_t* idx, int64_t N, int K, int64_t V,
                                       int* flag, int* host_flag, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = hipMemsetAsync(flag, 0, sizeof(int), s);
  if (e != hipSuccess) return (int)e;
  if (N > 0)
    hipLaunchKernelGGL(k_check_indices, dim3(cdiv(N, 4)), dim3(256), 0, s, idx, N, K, V, flag);
  e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  e = hipMemcpyAsync(host_flag, flag, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return (int)e;
  return (int)hipStreamSynchronize(s);
}

// y = g x for one or two gradients (see k_scale): a count of 0 skips one
extern "C" int kd_launch_scale(const KdScaleArg* a, const KdScaleArg* b, const float* g,
                               void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto arg = [](const KdScaleArg* q) { return ScaleArg{q->x, q->y, q->n, q->out_bf16}; };
  auto blocks = [](int64_t n) { return (int)std::min<int64_t>((n + 2047) / 2048, 8192); };
  const int ba = blocks(a->n), bb = blocks(b->n);
  if (ba + bb == 0) return 0;
  hipLaunchKernelGGL(k_scale, dim3(ba + bb), dim3(256), 0, s, arg(a), arg(b), ba, g);
  return (int)hipGetLastError();
}

// ------------------------------------------------------ static scratch ------
// The workspace of the allocation-free entry point: one file-scope array per
// device, held until the process ends. In host code the array's name denotes
// a host-side stand-in, not device memory, so host code never uses it as an
// address: the device address comes from hipGetSymbolAddress, once per
// device with that device current, and only that address is passed to
// kernels. Every call on a device shares its array.
static __device__ __align__(256) char scratch[kd_scratch_bytes_max];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};
}  // namespace

extern "C" int kd_scratch_get(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (g_scratch[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (p == nullptr) return (int)hipErrorInvalidSymbol;
    g_scratch[dev] = p;
  }
  *ptr = g_scratch[dev];
  return 0;
}

extern "C" void kd_launch_suppress_profiling(int on) { t_prof_suppressed = on != 0; }
