// luffy_condense: per-bucket cosine threshold graph, representative
// selection and compaction.
//
// Kernels, in launch order:
//   norm_kernel          1/|x_t| per token (one wave per row); clears the
//                        degree counters and walk states; its first wave
//                        lays out every bucket's tiles and bitmask.
//   gram_screen_kernel   (long bf16 rows, large buckets) the tiles below decided
//                        from fp8 products and a few single ones.
//   gram_kernel_{bf16,f32}  persistent loop over the upper-triangle tiles
//                        (256 rows bf16, 64 rows fp32) of every bucket's Gram
//                        matrix.  The epilogue turns cos >= h into adjacency
//                        bits, writes both the tile and its transpose (every
//                        bitmask word is written exactly once) and adds each
//                        row's edge count to its degree.
//   gram_hist_screen_kernel, gram_hist_kernel_bf16  the same two with the
//                        previous block's record of pair classes: decided pairs
//                        keep their class, the others' classes are recorded.
//   greedy_round_kernel  first round of the parallel form of the greedy
//                        walk, 16 lanes per position: keeps every position
//                        with no undecided neighbour of higher priority.
//                        A position is claimed by its neighbours as soon
//                        as it is kept, in every pass: it absorbs them and
//                        offers itself (64-bit atomic max of degree,
//                        ~position), so an absorbed position ends with its
//                        first-visited kept neighbour.  On a union of
//                        cliques this round decides every position.
//   greedy_more_kernel   persistent pass with bounded coherent revisits of
//                        positions still undecided (dependency chains).
//   greedy_finish_kernel one workgroup per bucket: a few rounds, then one
//                        visit per position left in priority order (only
//                        when the pass before left a position undecided).
//   rep_local_kernel, rep_finalize_kernel  representative rows by a two-pass
//                        scan: rep_row, rep_token, rep_offsets.
//   greedy_small_kernel  (at most 4096 slots) the last four in one launch, after
//                        the first round.
//   gather_kernel        optional copy of the representative rows.
//
// The walk of Sec. 5.2 visits positions by priority (degree descending,
// position ascending) and keeps a position iff no neighbour of higher
// priority was kept.  In parallel: an undecided position whose kept
// neighbour exists is absorbed; one whose every higher-priority neighbour is
// absorbed is kept.  Both rules only read final decisions, so rounds may see
// each other's updates early without changing the result, and every round
// decides at least the highest-priority undecided position.
#include <algorithm>
#include <atomic>

#include "gemm_core.h"
#include "luffy_common.h"

namespace luffy {
namespace {

constexpr int kGreedyPasses = 32;   // visits of a blocked position in the round after the grid rounds
constexpr int kTile = 256;      // similarity tile of the bf16 path (GramGemm)
constexpr int kTileF32 = 64;    // similarity tile of the fp32 path
constexpr int kGramF32Blocks = 3;   // its blocks a CU (48 KB of operand ring each)
constexpr int kStateUndecided = 0, kStateKept = 1, kStateAbsorbed = 2;
constexpr int kTileQueues = 8;  // tile queues of the history similarity kernel, one per XCD

__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// first e with offsets[e] <= p < offsets[e+1]
__device__ __forceinline__ int bucket_of(const int32_t* __restrict__ offsets, int E, int p) {
  int lo = 0, hi = E;  // answer: (first i in [0,E] with offsets[i] > p) - 1
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (offsets[mid + 1] <= p) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Tile and bitmask layout of every bucket, by one wave (lane e: expert e,
// E <= 64).  Flags an error (and schedules no tile) when a bucket exceeds
// max_bucket or the bitmask exceeds the workspace.
__device__ __forceinline__ void gram_layout(const int32_t* __restrict__ offsets, int E, int max_bucket,
                                            int tile, long long cap_words, int32_t* __restrict__ tile_off,
                                            long long* __restrict__ bm_off, int* __restrict__ err) {
  const int lane = threadIdx.x & 63;
  const int n = lane < E ? offsets[lane + 1] - offsets[lane] : 0;
  const int nt = (n + tile - 1) / tile;
  const int tiles = nt * (nt + 1) / 2;
  const long long words = static_cast<long long>(n) * ((n + 63) / 64);
  int tincl = tiles;
  long long wincl = words;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int tu = __shfl_up(tincl, o, 64);
    const long long wu = __shfl_up(wincl, o, 64);
    if (lane >= o) {
      tincl += tu;
      wincl += wu;
    }
  }
  const long long wtotal = __shfl(wincl, 63, 64);
  const bool bad = __ballot(lane < E && (n < 0 || n > max_bucket)) != 0 || wtotal > cap_words;
  if (lane < E) {
    tile_off[lane] = bad ? 0 : tincl - tiles;
    bm_off[lane] = wincl - words;
  }
  if (lane == 63) {
    tile_off[E] = bad ? 0 : tincl;
    bm_off[E] = wincl;
    *err = bad ? 1 : 0;
  }
}

// fp8 copy of the token rows for the similarity screen (Sec. 3's cosine,
// estimated): row t is normalised and scaled by 2^8, x_n = x * inv_norm[t] *
// 256 (|x_n| = 256 up to the rounding of the norm, every value within
// +-256, inside the E4M3 range), rounded to E4M3 by the hardware conversion
// (values below the smallest normal, 2^-6, stored as 0, so no subnormal
// reaches the MFMA).  Rows are padded with zeros to dp values, a multiple of
// 128.  rowq[t] holds, all relative to |x_n| and taken from the decoded bytes,
// i.e. from the values the MFMA multiplies,
//   x  rho, the row's quantisation error |x_n - x^|,
//   y  the same over its first da values,
//   z  |x_n| over the values from da on (the part a product of the first da
//      values leaves out),
// each enlarged a little to cover the float32 sums.  Then for every pair
// c~ = x^_a . x^_b / 2^16 (the raw fp8 product scaled by a power of two) and
// the cosine c of the bf16 pass satisfy
//   |c - c~| <= (|x^_a| |e_b| + |e_a| |x_b|) / (|x_a| |x_b|) <= rho_a + rho_b + rho_a rho_b
// (e = x_n - x^, |x_n| = 256), up to float32 rounding; over the first da values
// alone the same holds with y for x, and the rest adds at most z_a z_b
// (Cauchy-Schwarz).  Row T of x8 (the pad row of partial tiles) is zero.  One
// wave a row (norm_kernel's QUANT pass); d and da are multiples of 64.
__device__ __forceinline__ void gram_quant_row(const uint16_t* __restrict__ x, int T, int d, int t, float inv,
                                               int dp, int da, uint8_t* __restrict__ x8, float4* __restrict__ rowq) {
  const int lane = threadIdx.x & 63;
  uint8_t* out = x8 + static_cast<size_t>(t) * dp;
  if (t == T) {
    for (int c = lane * 8; c < dp; c += 512) *reinterpret_cast<uint2*>(out + c) = make_uint2(0u, 0u);
    return;
  }
  const uint16_t* row = x + static_cast<size_t>(t) * d;
  if (inv == 0.f) {
    // a finite row whose squares over- or underflow: its cosines are 0 or NaN as
    // the bf16 products fall out, so no bound holds and its tiles are handed back
    uint32_t m = 0;
    for (int c = lane * 8; c < d; c += 512) {
      Pack16 v;
      v.u4 = *reinterpret_cast<const uint4*>(row + c);
#pragma unroll
      for (int i = 0; i < 8; ++i) m = max(m, static_cast<uint32_t>(v.h[i] & 0x7FFF));
    }
    if (__ballot(m >= 0x7F80u) == 0 && __ballot(m != 0) != 0) {
      for (int c = lane * 8; c < dp; c += 512) *reinterpret_cast<uint2*>(out + c) = make_uint2(0u, 0u);
      const float big = __builtin_inff();
      if (lane == 0) rowq[t] = make_float4(big, big, big, 0.f);
      return;
    }
  }
  const float sc = inv * 256.f;
  float se = 0.f, sx = 0.f, sea = 0.f, sxb = 0.f;   // error and square sums; error of the first da, squares of the rest
  for (int c = lane * 8; c < dp; c += 512) {
    if (c >= d) {
      *reinterpret_cast<uint2*>(out + c) = make_uint2(0u, 0u);
      continue;
    }
    Pack16 v;
    v.u4 = *reinterpret_cast<const uint4*>(row + c);
    float f[8], g[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      f[i] = bf16_to_f32(v.h[i]) * sc;
      g[i] = fabsf(f[i]) < 0x1p-6f ? 0.f : f[i];
    }
    int lo = __builtin_amdgcn_cvt_pk_fp8_f32(g[0], g[1], 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(g[2], g[3], lo, true);
    int hi = __builtin_amdgcn_cvt_pk_fp8_f32(g[4], g[5], 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(g[6], g[7], hi, true);
    *reinterpret_cast<uint2*>(out + c) = make_uint2(static_cast<uint32_t>(lo), static_cast<uint32_t>(hi));
    const float dq[8] = {__builtin_amdgcn_cvt_f32_fp8(lo, 0), __builtin_amdgcn_cvt_f32_fp8(lo, 1),
                         __builtin_amdgcn_cvt_f32_fp8(lo, 2), __builtin_amdgcn_cvt_f32_fp8(lo, 3),
                         __builtin_amdgcn_cvt_f32_fp8(hi, 0), __builtin_amdgcn_cvt_f32_fp8(hi, 1),
                         __builtin_amdgcn_cvt_f32_fp8(hi, 2), __builtin_amdgcn_cvt_f32_fp8(hi, 3)};
    float e8 = 0.f, x8s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float df = f[i] - dq[i];
      e8 = fmaf(df, df, e8);
      x8s = fmaf(f[i], f[i], x8s);
    }
    se += e8;
    sx += x8s;
    if (c < da) sea += e8;
    else sxb += x8s;
  }
  se = wave_sum_f32(se);
  sx = wave_sum_f32(sx);
  sea = wave_sum_f32(sea);
  sxb = wave_sum_f32(sxb);
  if (lane == 0) {
    constexpr float kUp = 1.f + 0x1p-9f;
    rowq[t] = sx > 0.f ? make_float4(sqrtf(se / sx) * kUp, sqrtf(sea / sx) * kUp, sqrtf(sxb / sx) * kUp, 0.f)
                       : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// NORMS = false: the norms were computed by the caller (luffy_route); only
// the clearing and the layout run.  QUANT (bf16): also the similarity
// screen's fp8 rows (gram_quant_row; rows 0..T, T the zero pad row).
template <bool BF16, bool NORMS, bool QUANT = false>
__global__ __launch_bounds__(256) void norm_kernel(const void* __restrict__ xv, int T, int d,
                                                   float* __restrict__ inv_norm, int S,
                                                   int32_t* __restrict__ deg, int32_t* __restrict__ state,
                                                   unsigned long long* __restrict__ claim,
                                                   const int32_t* __restrict__ offsets, int E, int max_bucket,
                                                   int tile, long long cap_words, int32_t* __restrict__ tile_off,
                                                   long long* __restrict__ bm_off, int* __restrict__ err,
                                                   unsigned long long* __restrict__ stats, int* __restrict__ queue,
                                                   int* __restrict__ left, int* __restrict__ list_count, int dp,
                                                   int da, uint8_t* __restrict__ x8, float4* __restrict__ rowq) {
  if (blockIdx.x == 0 && threadIdx.x < 64)
    gram_layout(offsets, E, max_bucket, tile, cap_words, tile_off, bm_off, err);
  if (stats && blockIdx.x == 0 && threadIdx.x >= 64 && threadIdx.x < 68) stats[threadIdx.x - 64] = 0ull;
  if (queue && blockIdx.x == 0 && threadIdx.x >= 128 && threadIdx.x < 128 + kTileQueues) queue[threadIdx.x - 128] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 192) *left = 0;
  // the similarity screen's count of listed tiles
  if (list_count && blockIdx.x == 0 && threadIdx.x == 200) *list_count = 0;
  // also clears the degree counters, walk states and claim keys of all S positions
  for (int p = blockIdx.x * 256 + threadIdx.x; p < S; p += gridDim.x * 256) {
    deg[p] = 0;
    state[p] = 0;
    claim[p] = 0ull;
  }
  if constexpr (!NORMS && !QUANT) return;
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if constexpr (QUANT) {
    static_assert(BF16, "fp8 rows of bf16 tokens");
    if (t == T) gram_quant_row(static_cast<const uint16_t*>(xv), T, d, t, 0.f, dp, da, x8, rowq);
    if (t >= T) return;
    if constexpr (!NORMS) {
      gram_quant_row(static_cast<const uint16_t*>(xv), T, d, t, inv_norm[t], dp, da, x8, rowq);
      return;
    }
  }
  if (t >= T) return;
  float s = 0.f;
  if constexpr (BF16) {
    const uint16_t* x = static_cast<const uint16_t*>(xv) + static_cast<size_t>(t) * d;
    for (int c = lane * 8; c < d; c += 512) {
      Pack16 v;
      v.u4 = *reinterpret_cast<const uint4*>(x + c);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float f = bf16_to_f32(v.h[i]);
        s = fmaf(f, f, s);
      }
    }
  } else {
    const float* x = static_cast<const float*>(xv) + static_cast<size_t>(t) * d;
    for (int c = lane * 4; c < d; c += 256) {
      const float4 v = *reinterpret_cast<const float4*>(x + c);
      s = fmaf(v.x, v.x, s);
      s = fmaf(v.y, v.y, s);
      s = fmaf(v.z, v.z, s);
      s = fmaf(v.w, v.w, s);
    }
  }
  s = wave_sum_f32(s);
  const float inv = s > 0.f ? 1.0f / sqrtf(s) : 0.f;
  if (lane == 0) inv_norm[t] = inv;
  if constexpr (QUANT) gram_quant_row(static_cast<const uint16_t*>(xv), T, d, t, inv, dp, da, x8, rowq);
}

struct TileCoord {
  int e, ti, tj, lo, n, W;
};

// Bucket of tile `tile` (the last e with tile_off[e] <= tile, skipping
// empty buckets), its first tile, first slot and size.  One load per lane
// (lane e holds bucket e, E <= 64) and a ballot: a single round trip instead
// of a walk of dependent loads.  Called by whole waves.  The _from form
// takes the three per-lane values already loaded (bucket_lookup_loads).
__device__ __forceinline__ void bucket_lookup_loads(const int32_t* __restrict__ tile_off,
                                                    const int32_t* __restrict__ offsets, int E, int& to, int& o0,
                                                    int& o1) {
  const int lane = threadIdx.x & 63;
  const bool in = lane < E;
  to = in ? tile_off[lane] : 0;
  o0 = in ? offsets[lane] : 0;
  o1 = in ? offsets[lane + 1] : 0;
}

__device__ __forceinline__ void locate_bucket_from(int tile, int to, int o0, int o1, int E, int& e, int& tbase,
                                                   int& lo, int& n) {
  const int lane = threadIdx.x & 63;
  const bool in = lane < E;
  e = __popcll(__ballot(in && lane >= 1 && to <= tile));   // wave-uniform, at most E - 1
  tbase = __builtin_amdgcn_readlane(to, e);
  lo = __builtin_amdgcn_readlane(o0, e);
  n = __builtin_amdgcn_readlane(o1, e) - lo;
}

__device__ __forceinline__ void locate_bucket(int tile, const int32_t* __restrict__ tile_off,
                                              const int32_t* __restrict__ offsets, int E, int& e, int& tbase,
                                              int& lo, int& n) {
  int to, o0, o1;
  bucket_lookup_loads(tile_off, offsets, E, to, o0, o1);
  locate_bucket_from(tile, to, o0, o1, E, e, tbase, lo, n);
}

__device__ __forceinline__ TileCoord decode_tile(int tile, const int32_t* __restrict__ tile_off,
                                                 const int32_t* __restrict__ offsets, int E) {
  TileCoord c;
  int tbase;
  locate_bucket(tile, tile_off, offsets, E, c.e, tbase, c.lo, c.n);
  const int q = tile - tbase;
  int tj = static_cast<int>((sqrtf(8.0f * q + 1.0f) - 1.0f) * 0.5f);
  while (tj * (tj + 1) / 2 > q) --tj;
  while ((tj + 1) * (tj + 2) / 2 <= q) ++tj;
  c.tj = tj;
  c.ti = q - tj * (tj + 1) / 2;
  c.W = (c.n + 63) / 64;
  return c;
}

// v_writelane_b32: `old` with lane `lane` replaced by the wave-uniform
// `value` (the LLVM intrinsic, which clang does not expose as a builtin).
__device__ int amdgcn_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane");

// Writes the words of one predicate of a 64 x 64 tile: row rl of tile-row ti
// at word tj (dw[rl]) and, off the diagonal, row rl of tile-row tj at word ti
// (tw[rl], the transposed tile).  A 64-column tile is one word.
__device__ __forceinline__ void write_tile_words(const TileCoord& c, const uint64_t* dw, const uint64_t* tw,
                                                 uint64_t* __restrict__ bitmask, long long base) {
  const int tid = threadIdx.x;
  if (tid >= 2 * kTileF32) return;
  const bool mirror = tid >= kTileF32;
  if (mirror && c.ti == c.tj) return;
  const int rl = mirror ? tid - kTileF32 : tid;
  const int a = (mirror ? c.tj : c.ti) * kTileF32 + rl;
  if (a < c.n) bitmask[base + static_cast<long long>(a) * c.W + (mirror ? c.ti : c.tj)] = mirror ? tw[rl] : dw[rl];
}

// Bit pieces of NM predicates (bit m of pr[v]) over one 32 x 32 block in the
// accumulator layout (lane l: column l % 32, value v: row 8 (v / 4) + v % 4 +
// 4 (l / 32)): row pieces (32 columns) and column pieces (32 rows) of the
// predicates, stored by lanes 0-31 at d[m][rrow][cb] and t[m][col][rb] (32-bit
// halves of 64-bit words).
template <int NM>
__device__ __forceinline__ void block_bits(const uint32_t (&pr)[16], uint32_t* d, uint32_t* t, int rrow0, int col0) {
  const int lane = threadIdx.x & 63, l31 = lane & 31, hi = lane >> 5;
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    int piece = 0;
    uint32_t col = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int rv = 8 * (v >> 2) + (v & 3);
      const bool p = (pr[v] >> m) & 1u;
      const uint64_t bm = __ballot(p);
      piece = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(bm)), rv, piece);
      piece = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(bm >> 32)), rv + 4, piece);
      col |= p ? 1u << rv : 0u;
    }
    col <<= 4 * hi;
    col |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(col), 32, 64));
    if (lane < 32) {
      d[(m * kTileF32 + rrow0 + l31) * 2 + (col0 >> 5)] = static_cast<uint32_t>(piece);
      t[(m * kTileF32 + col0 + l31) * 2 + (rrow0 >> 5)] = col;
    }
  }
}

// Tile order inside a bucket for the 256-row tiles: columns are taken in
// groups of 4; inside a group the tiles go row by row (ti major), first the
// full rows above the group's diagonal block, then its upper triangle.  Any
// 32 consecutive tiles then cover about 8 row blocks x 4 column blocks, so
// the blocks of one XCD that run them together share operand rows in L2.
__device__ __forceinline__ TileCoord decode_tile_grouped_from(int tile, int to, int o0, int o1, int E) {
  TileCoord c;
  int tbase;
  locate_bucket_from(tile, to, o0, o1, E, c.e, tbase, c.lo, c.n);
  c.W = (c.n + 63) / 64;
  const int nt = (c.n + kTile - 1) / kTile;
  const int q = tile - tbase;
  // tiles before column group g: 8g^2 + 2g
  int g = static_cast<int>((sqrtf(4.0f + 32.0f * q) - 2.0f) / 16.0f);
  while (g > 0 && 8 * g * g + 2 * g > q) --g;
  while (8 * (g + 1) * (g + 1) + 2 * (g + 1) <= q) ++g;
  const int r = q - (8 * g * g + 2 * g);
  const int wdt = min(4, nt - 4 * g);
  if (r < 4 * g * wdt) {
    c.ti = r / wdt;
    c.tj = 4 * g + r % wdt;
  } else {
    int r2 = r - 4 * g * wdt, i = 0;
    while (r2 >= wdt - i) { r2 -= wdt - i; ++i; }
    c.ti = 4 * g + i;
    c.tj = 4 * g + i + r2;
  }
  return c;
}

__device__ __forceinline__ TileCoord decode_tile_grouped(int tile, const int32_t* __restrict__ tile_off,
                                                         const int32_t* __restrict__ offsets, int E) {
  int to, o0, o1;
  bucket_lookup_loads(tile_off, offsets, E, to, o0, o1);
  return decode_tile_grouped_from(tile, to, o0, o1, E);
}

using GramGemm = GemmBig64;
static_assert(GramGemm::BM == kTile && GramGemm::BN == kTile, "similarity tile");


// Tokens of a tile's DMA rows (P rows of tile-row ti, Q rows of tile-row
// tj; rows past the bucket repeat its last row and are not fetched) and the
// tokens whose inverse norms this thread stages for the epilogue: entry i
// of the tile's 2*kTile (P rows, then Q rows) goes to thread i % THREADS,
// as its (i / THREADS)-th (-1 past the bucket).
template <class G>
// pad >= 0: rows past the bucket read row `pad` instead (a zero row, so
// that every fetched row is defined).
__device__ __forceinline__ void gram_tile_tokens(const TileCoord& c, const int32_t* __restrict__ perm_token,
                                                 int32_t (&ptok)[G::LP], int32_t (&qtok)[G::LQ],
                                                 int32_t (&itok)[2 * kTile / G::THREADS], int pad = -1) {
  static_assert((2 * kTile) % G::THREADS == 0, "inverse norms per thread");
  const int32_t* pt = perm_token + c.lo;
#pragma unroll
  for (int j = 0; j < G::LP; ++j) {
    const int r = c.ti * kTile + G::load_row(j);
    ptok[j] = pad >= 0 && r >= c.n ? pad : pt[min(r, c.n - 1)];
  }
#pragma unroll
  for (int j = 0; j < G::LQ; ++j) {
    const int r = c.tj * kTile + G::load_row(G::LP + j) - G::BM;
    qtok[j] = pad >= 0 && r >= c.n ? pad : pt[min(r, c.n - 1)];
  }
#pragma unroll
  for (int u = 0; u < 2 * kTile / G::THREADS; ++u) {
    const int i = static_cast<int>(threadIdx.x) + u * G::THREADS;
    const int r = i < kTile ? c.ti * kTile + i : c.tj * kTile + i - kTile;
    itok[u] = r < c.n ? pt[r] : -1;
  }
}

// Inverse norm staged for the epilogue: NaN for a row outside the bucket,
// which fails every comparison.
__device__ __forceinline__ float gram_stage_inv(const float* __restrict__ inv_norm, int32_t itok) {
  return itok >= 0 ? inv_norm[itok] : __builtin_nanf("");
}

// bits * 2 + (p >= h): the comparison's bit shifted in through the carry
// (an ordered compare: a NaN p shifts in 0).  A VALU read of VCC needs two
// wait states after the VALU write of it: the _next form fills them with the
// next element's product q = (a * b) * c, the last form with a nop.
__device__ __forceinline__ uint32_t shift_in_ge_next(uint32_t bits, float p, float h, float a, float b, float c,
                                                     float& q) {
  asm("v_cmp_le_f32 vcc, %3, %2\n\t"
      "v_mul_f32 %1, %4, %5\n\t"
      "v_mul_f32 %1, %6, %1\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, vcc"
      : "+v"(bits), "=&v"(q)
      : "v"(p), "s"(h), "v"(a), "v"(b), "v"(c)
      : "vcc");
  return bits;
}

// bits * 2 + (p >= h) and m = min(m, |h - p|) (a NaN p shifts in 0 and
// leaves m): the subtraction and the minimum fill the two wait states of
// the VCC read.
__device__ __forceinline__ uint32_t shift_in_ge_band(uint32_t bits, float p, float h, float& m) {
  float dif;
  asm("v_cmp_le_f32 vcc, %4, %3\n\t"
      "v_sub_f32 %2, %4, %3\n\t"
      "v_min_f32 %1, %1, |%2|\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, vcc"
      : "+v"(bits), "+v"(m), "=&v"(dif)
      : "v"(p), "s"(h)
      : "vcc");
  return bits;
}

__device__ __forceinline__ uint32_t shift_in_ge_last(uint32_t bits, float p, float h) {
  asm("v_cmp_le_f32 vcc, %2, %1\n\t"
      "s_nop 1\n\t"
      "v_addc_co_u32 %0, vcc, %0, %0, vcc"
      : "+v"(bits)
      : "v"(p), "s"(h)
      : "vcc");
  return bits;
}

// One step of the 32 x 32 bit transpose below: lanes i and i ^ S of a
// half-wave trade the S-bit fields in which bit S of the lane index and of
// the bit index differ.
template <int S>
__device__ __forceinline__ uint32_t transpose_step(uint32_t x, int i) {
  constexpr uint32_t m0 = S == 16 ? 0x0000FFFFu : S == 8 ? 0x00FF00FFu : S == 4 ? 0x0F0F0F0Fu
                        : S == 2 ? 0x33333333u : 0x55555555u;   // bits j with bit S of j clear
  // ds_swizzle bit mode within 32 lanes: and-mask 31, xor-mask S
  const uint32_t y = static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(static_cast<int>(x), 0x1F | (S << 10)));
  const bool up = (i & S) != 0;
  // lower lane: the partner's m0 fields move up by S; upper lane: its ~m0 fields move down by S
  const uint32_t t = __builtin_amdgcn_alignbit(y, y, up ? S : 32 - S);
  const uint32_t keep = up ? ~m0 : m0;
  return (x & keep) | (t & ~keep);
}

// 32 x 32 bit transpose within each half-wave: lane c holds word c of a
// square bit matrix (bit j: entry (j, c)); afterwards lane j holds the word
// with bit c = entry (j, c).
__device__ __forceinline__ uint32_t transpose32_bits(uint32_t x) {
  const int i = opaque_tid() & 31;   // per-lane masks recomputed here, not hoisted out of the tile loop
  x = transpose_step<16>(x, i);
  x = transpose_step<8>(x, i);
  x = transpose_step<4>(x, i);
  x = transpose_step<2>(x, i);
  return transpose_step<1>(x, i);
}

// Writes a 256 x 256 tile's adjacency words (4 per row, direct and, off the
// diagonal, mirrored) and adds each row's edge count to its degree, from the
// tile's bit pieces dbits[row][32-column group], tbits[column][32-row group].
__device__ __forceinline__ void write_gram_tile(const TileCoord& c, const uint32_t (*dbits)[kTile / 32],
                                                const uint32_t (*tbits)[kTile / 32], uint64_t* __restrict__ bitmask,
                                                long long base, int32_t* __restrict__ deg, int threads) {
  // degree: edges of each tile row (and, off the diagonal, of each mirrored row)
  for (int i = opaque_tid(); i < 2 * kTile; i += threads) {
    const bool mirror = i >= kTile;
    const int rl = mirror ? i - kTile : i;
    const uint32_t* pcs = mirror ? tbits[rl] : dbits[rl];
    int cnt = 0;
#pragma unroll
    for (int g = 0; g < kTile / 32; ++g) cnt += __popc(pcs[g]);
    const int r = (mirror ? c.tj : c.ti) * kTile + rl;
    if (cnt && r < c.n && (!mirror || c.ti != c.tj)) atomicAdd(&deg[c.lo + r], cnt);
  }
  // two words a thread
  auto store2 = [&](const uint32_t* pcs, int row, int wd) {
    if (row >= c.n || wd >= c.W) return;
    const uint4 v = *reinterpret_cast<const uint4*>(pcs);
    uint64_t* dst = bitmask + base + static_cast<long long>(row) * c.W + wd;
    if (wd + 1 < c.W) {
      __builtin_memcpy(dst, &v, 16);
    } else {
      const uint64_t lo = static_cast<uint64_t>(v.x) | (static_cast<uint64_t>(v.y) << 32);
      *dst = lo;
    }
  };
  for (int i = opaque_tid(); i < kTile * 2; i += threads) {
    const int rl = i >> 1, ww = 2 * (i & 1);
    store2(&dbits[rl][2 * ww], c.ti * kTile + rl, 4 * c.tj + ww);
    if (c.ti != c.tj) store2(&tbits[rl][2 * ww], c.tj * kTile + rl, 4 * c.ti + ww);
  }
}

// Column piece of a 32 x 32 block from a lane's 16 compare bits (bit v:
// accumulator v, row 8 (v / 4) + v % 4 + 4 (l / 32)): the bits spread to their
// rows and the two half-waves merged; a token with itself is dropped on a
// diagonal block.
__device__ __forceinline__ uint32_t spread_col_bits(uint32_t bits, int hi, bool diag, int l31) {
  // nibble k (accumulators 4k..4k+3) to bits 8k..8k+3, then this half's rows
  bits = (bits & 0xFFu) | ((bits & 0xFF00u) << 8);
  bits = (bits & 0x000F000Fu) | ((bits & 0x00F000F0u) << 4);
  bits <<= 4 * hi;
  uint32_t cw = bits | static_cast<uint32_t>(__shfl_xor(static_cast<int>(bits), 32, 64));
  if (diag) cw &= ~(1u << l31);
  return cw;
}

// Row pieces of a wave's pair of column blocks (bit transposes of their
// column pieces, one block per half-wave), stored at d[row][group].
__device__ __forceinline__ void store_row_bits(uint32_t col0, uint32_t col1, int hi, int l31, int abase, int bbase,
                                               uint32_t (*dbits)[kTile / 32]) {
  // lower half-wave: the first block, upper: the second (a select, not an
  // indexed read, which would put the words in memory)
  const uint32_t sel = col0 ^ ((col0 ^ col1) & (0u - static_cast<uint32_t>(hi)));
  const uint32_t rowbits = transpose32_bits(sel);
  dbits[abase + l31][(bbase + 32 * hi) >> 5] = rowbits;
}

// Similarity tiles on bf16 MFMA.  LIST = false: every upper-triangle tile of
// every bucket; LIST = true: the tiles the screen handed back.  The tile loop
// is software-pipelined: the next tile's bucket lookup is loaded
// before the current tile's K loop (nothing waits on it until the loop is
// over, so it does not hold up the loop's first stages, which the in-order
// load counter would otherwise tie to it); right after the K loop the next
// tile's row tokens are loaded, their latency hidden by this tile's
// compares, and its first DMA stages are issued before the rest of this
// tile's epilogue, which therefore keeps its bit pieces outside the operand
// ring.
template <bool LIST>
__global__ __launch_bounds__(GramGemm::THREADS) void gram_kernel_bf16(
    const uint16_t* __restrict__ X, int d, const int32_t* __restrict__ perm_token,
    const int32_t* __restrict__ offsets, int E, const float* __restrict__ inv_norm, float h,
    const int32_t* __restrict__ tile_off, const long long* __restrict__ bm_off,
    const int* __restrict__ err, uint64_t* __restrict__ bitmask, int32_t* __restrict__ deg,
    const int* __restrict__ list, const int* __restrict__ list_count) {
  using G = GramGemm;
  constexpr int NI = 2 * kTile / G::THREADS;   // inverse norms staged per thread
  static_assert(G::FN == 2, "column blocks are transposed in pairs");
  // One LDS array: the operand ring, then the inverse norms of the tile's P
  // rows (0..kTile-1) and Q rows (kTile..), then the tile's adjacency
  // pieces.  With separate LDS variables the compiler loses
  // the alias scopes that tell a stage's fragment reads from the DMA into
  // the other stage, and waits for each stage's DMA right after issuing it
  // (no overlap).
  constexpr int kInvOff = G::LDS_BYTES, kBitsOff = kInvOff + 2 * kTile * 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kBitsOff + 2 * kTile * (kTile / 32) * 4];
  float* inv_ab = reinterpret_cast<float*>(lds + kInvOff);
  uint32_t (*dbits)[kTile / 32] = reinterpret_cast<uint32_t (*)[kTile / 32]>(lds + kBitsOff);
  uint32_t (*tbits)[kTile / 32] = reinterpret_cast<uint32_t (*)[kTile / 32]>(lds + kBitsOff + kTile * (kTile / 32) * 4);
  const float* inv_a = inv_ab;
  const float* inv_b = inv_ab + kTile;
  if (*err) return;
  const int w = G::wave();
  const int wm = G::wave_m(w), wn = G::wave_n(w);
  const int total = LIST ? *list_count : tile_off[E];
  auto tile_of = [&](int item) { return LIST ? list[item] : item; };
  int item = xcd_virtual_block();
  if (item >= total) return;   // block-uniform, before any barrier
  TileCoord c = decode_tile_grouped(tile_of(item), tile_off, offsets, E);
  int32_t ptok[G::LP], qtok[G::LQ], itok[NI];
  uint32_t poff[G::LP], qoff[G::LQ];
  gram_tile_tokens<G>(c, perm_token, ptok, qtok, itok);
#pragma unroll
  for (int j = 0; j < G::LP; ++j) poff[j] = static_cast<uint32_t>(ptok[j]) * d;
#pragma unroll
  for (int j = 0; j < G::LQ; ++j) qoff[j] = static_cast<uint32_t>(qtok[j]) * d;
  float inv[NI];
#pragma unroll
  for (int u = 0; u < NI; ++u) inv[u] = gram_stage_inv(inv_norm, itok[u]);
  typename G::Pipe pipe;
  G::prefetch(X, poff, X, qoff, d, c.n - c.ti * kTile, c.n - c.tj * kTile, lds, pipe);
  for (;;) {
#pragma unroll
    for (int u = 0; u < NI; ++u) inv_ab[opaque_tid() + u * G::THREADS] = inv[u];   // visible after the K loop's first barrier
    const int nitem = item + gridDim.x;
    const int next = nitem < total ? tile_of(nitem) : 0;
    int nto = 0, no0 = 0, no1 = 0;
    if (nitem < total) bucket_lookup_loads(tile_off, offsets, E, nto, no0, no1);
    typename G::Acc acc;
    G::zero(acc);
    G::resume(pipe, lds, acc);   // ends with a barrier: the ring is free
    TileCoord cn = c;
    if (nitem < total) {
      cn = decode_tile_grouped_from(next, nto, no0, no1, E);
      gram_tile_tokens<G>(cn, perm_token, ptok, qtok, itok);
    }
    __builtin_amdgcn_sched_barrier(0);

    // Each (fm, fn) block is 32 x 32.  Lane l holds column bbase + l%32 and,
    // in accumulator v, row abase + rv(v) + 4*(l/32), rv(v) = 8(v/4) + v%4.
    // Each lane shifts its 16 compare bits into a word (accumulator v at bit
    // v) and spreads them to bits rv(v); lanes c and c+32 merge theirs with
    // one cross-half exchange, which gives the column pieces (the mirrored
    // tile's row words).  The row pieces are the bit transposes of the
    // column pieces: the two column blocks of a wave are transposed
    // together, one per half-wave.  Edge test: dot * (1/|a|) * (1/|b|) >= h
    // (rows outside the bucket carry a NaN scale), never a token with
    // itself.
    // lane values recomputed from the opaque thread index: hoisted out of
    // the tile loop they would stay live across the K loop
    const int el = opaque_tid() & 63;
    const int l31 = el & 31, hi = el >> 5;
    const bool same_tile = c.ti == c.tj;
#pragma unroll
    for (int fm = 0; fm < G::FM; ++fm) {
      const int abase = wm * G::WTM + 32 * fm;
      // this lane's 16 rows: abase + 8q + 4hi + r, as 4 runs of 4
      float ia[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 f = *reinterpret_cast<const float4*>(&inv_a[abase + 8 * q + 4 * hi]);
        ia[4 * q] = f.x;
        ia[4 * q + 1] = f.y;
        ia[4 * q + 2] = f.z;
        ia[4 * q + 3] = f.w;
      }
      uint32_t col[G::FN];
#pragma unroll
      for (int fn = 0; fn < G::FN; ++fn) {
        const int bbase = wn * G::WTN + 32 * fn;
        const int bl = bbase + l31;
        uint32_t bits = 0;
        const float ib = inv_b[bl];
        float p = acc[fm][fn][15] * ia[15] * ib;
#pragma unroll
        for (int v = 15; v >= 1; --v) {
          float q;
          bits = shift_in_ge_next(bits, p, h, acc[fm][fn][v - 1], ia[v - 1], ib, q);
          p = q;
        }
        bits = shift_in_ge_last(bits, p, h);
        col[fn] = spread_col_bits(bits, hi, same_tile && abase == bbase, l31);
        if (hi == 0) tbits[bl][abase >> 5] = col[fn];
      }
      store_row_bits(col[0], col[1], hi, l31, abase, wn * G::WTN, dbits);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (nitem < total) {
#pragma unroll
      for (int j = 0; j < G::LP; ++j) poff[j] = static_cast<uint32_t>(ptok[j]) * d;
#pragma unroll
      for (int j = 0; j < G::LQ; ++j) qoff[j] = static_cast<uint32_t>(qtok[j]) * d;
      // before the DMA: waiting for them then does not wait for the DMA
#pragma unroll
      for (int u = 0; u < NI; ++u) inv[u] = gram_stage_inv(inv_norm, itok[u]);
      G::prefetch(X, poff, X, qoff, d, cn.n - cn.ti * kTile, cn.n - cn.tj * kTile, lds, pipe);
    }
    // LDS-only barriers from here on: a full __syncthreads() would also wait
    // for the next tile's DMA
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's pieces are in LDS
    raw_barrier();
    write_gram_tile(c, dbits, tbits, bitmask, bm_off[c.e], deg, G::THREADS);
    if (nitem >= total) break;
    // every wave's reads of the pieces and of inv_ab are done before the next
    // tile overwrites them
    __builtin_amdgcn_s_waitcnt(0xC07F);
    raw_barrier();
    item = nitem;
    c = cn;
  }
}

// The similarity screen's arguments.
struct ScreenArgs {
  const uint8_t* x8;      // fp8 rows (E4M3, scaled by 2^8), pitch dp; row T is zero
  const float4* rowq;     // error bounds of every row (gram_quant_row)
  const uint16_t* x;      // the bf16 rows
  const float* inv_norm;
  int d, dp, da, T;
  float h;                // > 0
  int* list;              // tiles handed back to the bf16 pass
  int* list_count;
};

constexpr int kWavePairs = 64;    // pairs of a wave's part of a tile that can be looked at one by one
constexpr int kWaveFirst = 32;    // of them after the first da values
// Tiles a block takes whole after one that went on to phase 2 (gram_screen_kernel).
// 4 buckets of 8192 tokens, d = 2048, groups of 64: 279 us with one phase, 333 with
// every tile in two, 301 so; 8 of 2048, d = 4096, groups of 4 (some tiles go on):
// 102, 85 and 97; where no tile goes on there is no difference.
constexpr int kWholeTiles = 7;

// Wave-wide maximum and sum, the same in every lane: DPP rotations inside the
// rows of 16, then the four rows read as scalars (a cross-lane shuffle through
// LDS per step would take six dependent LDS round trips).
template <int N>
__device__ __forceinline__ float row_rotate(float x) {
  return __uint_as_float(static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(__float_as_uint(x)), 0x120 + N, 0xF, 0xF, false)));
}
__device__ __forceinline__ float lane_value(float x, int l) {
  return __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(__float_as_uint(x)), l)));
}
__device__ __forceinline__ float wave_max_dpp(float x) {
  x = fmaxf(x, row_rotate<8>(x));
  x = fmaxf(x, row_rotate<4>(x));
  x = fmaxf(x, row_rotate<2>(x));
  x = fmaxf(x, row_rotate<1>(x));
  return fmaxf(fmaxf(lane_value(x, 0), lane_value(x, 16)), fmaxf(lane_value(x, 32), lane_value(x, 48)));
}
__device__ __forceinline__ float wave_sum_dpp(float x) {
  x += row_rotate<8>(x);
  x += row_rotate<4>(x);
  x += row_rotate<2>(x);
  x += row_rotate<1>(x);
  return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// Accumulators of a 32 x 32 block on the diagonal that lie above it (bit v: row
// 8 (v / 4) + v % 4 + 4 hi < column l31), so that a pair is taken once.
__device__ __forceinline__ uint32_t above_diagonal(int l31, int hi) {
  const int q = l31 - 4 * hi;
  return q > 0 ? (1u << (4 * (q >> 3) + min(q & 7, 4))) - 1u : 0u;
}

// bits * 2 + (x < 0): the sign of a difference, without a compare (a NaN shifts in
// either).
__device__ __forceinline__ uint32_t shift_in_sign(uint32_t bits, float x) {
  return __builtin_amdgcn_alignbit(bits, __float_as_uint(x), 31);
}

// Sum over the lanes below this one, and over the wave: DPP shifts within the
// rows of 16, then the last lanes of rows broadcast to the rows after them.
__device__ __forceinline__ int wave_prefix_dpp(int x, int& total) {
  int s = x;
  s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, true);
  s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, true);
  s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, true);
  s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, true);
  s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xA, 0xF, true);
  s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xC, 0xF, true);
  total = __builtin_amdgcn_readlane(s, 63);
  return s - x;
}

// The pairs of a wave's part of a tile (FM x 2 blocks of 32 x 32) that are looked
// at one by one: left[fm] marks this lane's accumulators of blocks (fm, 0) and
// (fm, 1) in its low and high half (bit v: row 8 (v / 4) + v % 4 + 4 hi, column
// l31 of the block).  Counts the marked ones and, where they are at most `limit`,
// lists them in LDS (row << 8 | column; the wave's first row and column of the
// tile in row0, col0), each lane its own, so that the loops take a step for each
// pair of the fullest lane.  (Taken value by value with a ballot each, the 32
// pairs of a wave took 4 us.)
template <int FM>
__device__ __forceinline__ int list_pairs(const uint32_t (&left)[FM], int limit, int row0, int col0, uint32_t* pairs) {
  const int lane = opaque_tid() & 63;
  int mine = 0, total;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) mine += __popc(left[fm]);
  if (__ballot(mine != 0) == 0) return 0;   // the common case
  int at = wave_prefix_dpp(mine, total);
  if (total > limit) return total;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
    for (uint32_t m = left[fm]; m != 0; m &= m - 1) {
      const int b = __ffs(static_cast<int>(m)) - 1, v = b & 15;
      const int row = row0 + 32 * fm + 8 * (v >> 2) + (v & 3) + 4 * (lane >> 5);
      const int col = col0 + 32 * (b >> 4) + (lane & 31);
      pairs[at++] = static_cast<uint32_t>(row << 8 | col);
    }
  return total;
}

// Marks of a 32 x 32 block whose rows and columns are all taken: rows from row0 on
// and columns from col0 on of a tile of nra x nrb, those above the diagonal on a
// diagonal block.
__device__ __forceinline__ uint32_t valid_marks(int row0, int col0, int nra, int nrb, bool diagonal, int l31, int hi) {
  const int q = nra - row0 - 4 * hi;   // rows left: a prefix of the marks, as above_diagonal's
  uint32_t m = q >= 28 ? 0xFFFFu : q > 0 ? (1u << (4 * (q >> 3) + min(q & 7, 4))) - 1u : 0u;
  if (diagonal) m &= above_diagonal(l31, hi);
  return col0 + l31 < nrb ? m : 0u;
}

// The similarity screen: every upper-triangle tile decided from fp8 products
// where their error bound allows it, and from single products of two rows where
// a few pairs of it are too close.  The result is the one of the bf16 pass.
//
// Phase 1 multiplies only the first da values of the rows (ScreenArgs.da < dp).
// With c~ the estimate over them, a pair's cosine is below
// c~ + band + z_a z_b (band: the quantisation bound; z: what the rows keep
// beyond da), so a pair with c~ < h - band - max z max z is no edge.  Tokens of
// different meaning are nearly orthogonal, so what is left is little more than
// the tile's edges themselves (an expert's bucket of n tokens in groups of g
// has about 65536 (g - 1) / n of them per tile).  Each wave keeps the pairs left
// of its part of the tile; if no wave has more than kWaveFirst, their fp8
// products are taken one pair at a time.  Otherwise phase 2 multiplies the rest of
// the values for the whole tile, and the block's next kWholeTiles tiles take all
// values at once (a tile that goes on to phase 2 takes about 4 us longer than one
// that does not try: the compares, a barrier, the ring's refill; tiles of one call
// mostly go the same way).  A block without a next tile prefetches its phase 2
// in the next tile's place.  Either way a pair whose
// full estimate is further than band from h is decided, and a closer one gets
// its bf16 dot product.  A tile where a wave has more than kWavePairs of those,
// or one whose dot product is within float32 rounding of h, is listed for the
// bf16 pass and not written.
//
// Why: a whole fp8 tile is bound by its K loop (LDS traffic and MFMA issue,
// 2,670 cycles per 128 values) and the compares of its 65536 results; the first
// 512 of 2048 values leave about 60 pairs of a tile of the expert-parallel
// share (T = 32768, d = 2048, h = 0.9).
// That layer's similarity: whole fp8 products 519 us, this 328 (361 under the
// profiler); 16384 i.i.d. tokens of d = 4096: 103-111 -> 37-46 us.  Calls with about
// one tile a block whose tiles all go on lose 4 us against one phase (T = 4096, 8
// buckets, d = 2048, groups of 4 and more: 30 -> 34).
__global__ __launch_bounds__(GramGemm::THREADS) void gram_screen_kernel(
    ScreenArgs sa, const int32_t* __restrict__ perm_token, const int32_t* __restrict__ offsets, int E,
    const int32_t* __restrict__ tile_off, const long long* __restrict__ bm_off, const int* __restrict__ err,
    uint64_t* __restrict__ bitmask, int32_t* __restrict__ deg) {
  using G = GemmBig64F8;
  static_assert(G::BM == kTile && G::BN == kTile && G::THREADS == 2 * kTile && G::NWAVES == 8, "one row a thread");
  // one LDS array (see gram_kernel_bf16): the operand ring, the waves' row
  // bounds, the tokens of this tile and of the next (P rows, then Q rows), the
  // adjacency pieces, the bucket tables, every wave's pairs (row << 8 | column),
  // every wave's pairs still too close after their whole fp8 product, the pair
  // counts and the hand-back flag
  constexpr int kRedOff = G::LDS_BYTES, kTokOff = kRedOff + G::NWAVES * 16, kBitsOff = kTokOff + 4 * kTile * 4;
  constexpr int kTabOff = kBitsOff + 2 * kTile * (kTile / 32) * 4, kListOff = kTabOff + 3 * kMaxExperts * 4;
  constexpr int kCloseOff = kListOff + G::NWAVES * kWavePairs * 4, kCntOff = kCloseOff + G::NWAVES * kWavePairs * 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kCntOff + 48];
  float4* red = reinterpret_cast<float4*>(lds + kRedOff);
  uint32_t (*dbits)[kTile / 32] = reinterpret_cast<uint32_t (*)[kTile / 32]>(lds + kBitsOff);
  uint32_t (*tbits)[kTile / 32] = reinterpret_cast<uint32_t (*)[kTile / 32]>(lds + kBitsOff + kTile * (kTile / 32) * 4);
  int* tab = reinterpret_cast<int*>(lds + kTabOff);
  int* cnt = reinterpret_cast<int*>(lds + kCntOff);   // [w]: pairs of wave w; [8]: hand the tile back
  if (*err) return;
  const int w = G::wave();
  const int wm = G::wave_m(w), wn = G::wave_n(w);
  const int total = tile_off[E];
  int tile = xcd_virtual_block();
  if (tile >= total) return;   // block-uniform, before any barrier
  const uint16_t* X = reinterpret_cast<const uint16_t*>(sa.x8);
  const int K = sa.dp / 2, KA = sa.da / 2;   // 16-bit units, 64 a stage
  if (w == 0) {
    int to, o0, o1;
    bucket_lookup_loads(tile_off, offsets, E, to, o0, o1);
    const int l = opaque_tid();
    tab[l] = to;
    tab[kMaxExperts + l] = o0;
    tab[2 * kMaxExperts + l] = o1;
  }
  __syncthreads();
  auto decode = [&](int t) {
    const int l = opaque_tid() & 63;
    return decode_tile_grouped_from(t, tab[l], tab[kMaxExperts + l], tab[2 * kMaxExperts + l], E);
  };
  auto tokens = [&](int buf) { return reinterpret_cast<int32_t*>(lds + kTokOff) + buf * 2 * kTile; };
  // tokens of the tile's rows straight to LDS: wave w takes rows 64 (w % 4) .. of
  // P (w < 4) or Q; rows past the bucket repeat its last one
  auto fetch_tokens = [&](const TileCoord& t, int buf) {
    const int l = opaque_tid() & 63;
    const int r = (w < 4 ? t.ti : t.tj) * kTile + 64 * (w & 3) + l;
    const uint32_t off = static_cast<uint32_t>(t.lo + min(r, t.n - 1)) * 4u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        G::rsrc(perm_token),
        reinterpret_cast<__attribute__((address_space(3))) void*>((G::lds_ptr)(lds + kTokOff) + (buf * 2 * kTile + 64 * w) * 4),
        4, off, 0, 0, 0);
  };
  // row offsets of the tile's DMA (the zero row past the bucket) over nk units
  // from unit k0 on
  typename G::Pipe pipe;
  auto prepare = [&](const TileCoord& t, int buf, int k0, int nk) {
    const int32_t* tk = tokens(buf);
    uint32_t poff[G::LP], qoff[G::LQ];
#pragma unroll
    for (int j = 0; j < G::LP; ++j) {
      const int r = G::load_row(j);
      poff[j] = static_cast<uint32_t>(t.ti * kTile + r < t.n ? tk[r] : sa.T) * K;
    }
#pragma unroll
    for (int j = 0; j < G::LQ; ++j) {
      const int r = G::load_row(G::LP + j) - G::BM;
      qoff[j] = static_cast<uint32_t>(t.tj * kTile + r < t.n ? tk[kTile + r] : sa.T) * K;
    }
    G::prepare(X + k0, poff, X + k0, qoff, nk, kTile, kTile, pipe);
  };
  constexpr int kDma = G::STAGES * G::LOADS;   // loads of a tile's first stages
  // the same with the first stages issued
  auto start = [&](const TileCoord& t, int buf, int k0, int nk) {
    prepare(t, buf, k0, nk);
#pragma unroll
    for (int i = 0; i < kDma; ++i) G::issue_one(pipe, i, lds);
  };
  // error bounds of this thread's row (thread i: P row i, then Q row i - 256)
  auto bounds = [&](const TileCoord& t, int buf) {
    const int i = opaque_tid();
    const int r = (i < kTile ? t.ti : t.tj - 1) * kTile + i;
    return r < t.n ? sa.rowq[tokens(buf)[i]] : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  TileCoord c = decode(tile);
  fetch_tokens(c, 0);
  __syncthreads();   // (waits for the DMA too)
  float4 rq = bounds(c, 0);
  start(c, 0, 0, K);
  const float hs = sa.h * 65536.f;   // the threshold in units of the fp8 products (exact)
  int whole = 0;   // tiles that this block takes whole before it tries the first values again
  for (int buf = 0;; buf ^= 1) {
    const bool two = KA < K && whole == 0;
    pipe.nk = (two ? KA : K) / G::BK;
    const int ntile = tile + gridDim.x;
    const bool more = ntile < total;
    TileCoord cn = c;
    if (more) {
      cn = decode(ntile);
      fetch_tokens(cn, buf ^ 1);   // lands under the K loop
    }
    // staged for this tile, visible after the K loop's barriers
    {
      const float4 m = make_float4(wave_max_dpp(rq.x), wave_max_dpp(rq.y), wave_max_dpp(rq.z), 0.f);
      const int tid = opaque_tid();
      if ((tid & 63) == 0) red[w] = m;
      if (tid == 0) cnt[8] = 0;
      if (two) {   // (a whole tile's pieces are all written)
        uint4* z = reinterpret_cast<uint4*>(&dbits[0][0]);
        z[tid] = z[tid + G::THREADS] = make_uint4(0u, 0u, 0u, 0u);
      }
      static_assert(2 * G::THREADS * 16 == 2 * kTile * (kTile / 32) * 4, "cleared pieces");
    }
    typename G::Acc acc;
    G::zero(acc);
    G::resume(pipe, lds, acc);   // ends with a barrier: the ring is free
    if (more) {
      // the next tile's first stages are issued between this tile's compares
      // and land under the rest of its epilogue
      rq = bounds(cn, buf ^ 1);
      prepare(cn, buf ^ 1, 0, K);
      if (!two) {
#pragma unroll
        for (int i = 0; i < kDma; ++i) G::issue_one(pipe, i, lds);
      }
    } else if (two) {
      prepare(c, buf, KA, K - KA);   // no next tile: this one's second phase, if it comes to it
    }
    const int el = opaque_tid() & 63;
    const int l31 = el & 31, hi = el >> 5;
    const bool same_tile = c.ti == c.tj;
    float rho = 0.f, rho1 = 0.f, zp = 0.f, zq = 0.f;
#pragma unroll
    for (int i = 0; i < G::NWAVES; ++i) {
      const float4 f = red[i];
      rho = fmaxf(rho, f.x);
      rho1 = fmaxf(rho1, f.y);
      if (i < G::NWAVES / 2) zp = fmaxf(zp, f.z);
      else zq = fmaxf(zq, f.z);
    }
    const float band = (2.f * rho + rho * rho + 4e-3f) * 65536.f;
    // a row without a bound (gram_quant_row: all of its bounds infinite) hands its
    // tiles back whatever their products; the first phase's threshold would be a
    // NaN where such a row meets rows that are zero past the first da values
    const bool bounded = rho < __builtin_inff();   // block-uniform
    uint32_t* pairs = reinterpret_cast<uint32_t*>(lds + kListOff) + w * kWavePairs;
    const int nra = c.n - c.ti * kTile, nrb = c.n - c.tj * kTile;
    uint32_t left[G::FM] = {};   // the pairs left of this lane's part (list_pairs)
    static_assert(G::FN == 2, "two blocks a word");
    int np = 0;
    auto any_over = [&](int limit) {   // block-uniform
      if (el == 0) cnt[w] = np;
      __builtin_amdgcn_s_waitcnt(0xC07F);
      raw_barrier();
      return __ballot(el < G::NWAVES && cnt[el & 7] > limit) != 0;
    };
    bool full = !two || !bounded;   // block-uniform: the whole tile's products are taken
    if (two && bounded) {
      const float thr = (sa.h - (2.f * rho1 + rho1 * rho1 + 4e-3f) - zp * zq) * 65536.f;
#pragma unroll
      for (int fm = 0; fm < G::FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < G::FN; ++fn) {
          constexpr int PER = (kDma + G::FM * G::FN - 1) / (G::FM * G::FN);
#pragma unroll
          for (int i = 0; i < PER; ++i)
            if ((fm * G::FN + fn) * PER + i < kDma) G::issue_one(pipe, (fm * G::FN + fn) * PER + i, lds);
          const int abase = wm * G::WTM + 32 * fm, bbase = wn * G::WTN + 32 * fn;
          if (same_tile && abase > bbase) continue;   // the mirror's pairs
          // most blocks have no pair left: their largest value is tested first
          float mx = acc[fm][fn][0];
#pragma unroll
          for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[fm][fn][v]);
          if (__ballot(mx >= thr) == 0) continue;
          uint32_t hits = 0;
#pragma unroll
          for (int v = 15; v >= 0; --v) hits = shift_in_sign(hits, thr - acc[fm][fn][v]);
          left[fm] |= (hits & valid_marks(abase, bbase, nra, nrb, same_tile && abase == bbase, l31, hi)) << 16 * fn;
        }
      np = list_pairs(left, kWaveFirst, wm * G::WTM, wn * G::WTN, pairs);
      full = any_over(kWaveFirst);
      if (full) {
        // the rest of the values: the ring is taken back from the next tile
        if (more) {
          wait_vmcnt<0>();
          __builtin_amdgcn_s_waitcnt(0xC07F);
          raw_barrier();
          start(c, buf, KA, K - KA);
        }
        whole = kWholeTiles + 1;
        G::resume(pipe, lds, acc);
#pragma unroll
        for (int fm = 0; fm < G::FM; ++fm) left[fm] = 0;
      }
    }
    const bool first_only = !full;
    if (full) {
      // raw fp8 products of unit rows scaled by 2^8: c~ = acc / 2^16
#pragma unroll
      for (int fm = 0; fm < G::FM; ++fm) {
        const int abase = wm * G::WTM + 32 * fm;
        uint32_t col[G::FN];
#pragma unroll
        for (int fn = 0; fn < G::FN; ++fn) {
          const int bbase = wn * G::WTN + 32 * fn;
          // a token with itself is set to 0 (no edge for h > 0, and the word
          // drops it below anyway)
          if (same_tile && abase == bbase) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
              if (8 * (v >> 2) + (v & 3) + 4 * hi == l31) acc[fm][fn][v] = 0.f;
          }
          // a 32 x 32 block without an edge (every product below 2^16 h,
          // the common case) needs only its largest product: no bits, and
          // its least distance to 2^16 h is 2^16 h minus that product
          uint32_t bits = 0;
          float dmin = __builtin_inff();
          float mx = acc[fm][fn][0];
#pragma unroll
          for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[fm][fn][v]);
          if (__ballot(mx >= hs) == 0) {
            dmin = hs - mx;
          } else {
#pragma unroll
            for (int v = 15; v >= 0; --v) bits = shift_in_ge_band(bits, acc[fm][fn][v], hs, dmin);
          }
          if (__ballot(dmin < band) != 0 && !(same_tile && abase > bbase)) {
            uint32_t hits = 0;
#pragma unroll
            for (int v = 15; v >= 0; --v) hits = shift_in_sign(hits, fabsf(acc[fm][fn][v] - hs) - band);
            left[fm] |= (hits & valid_marks(abase, bbase, nra, nrb, same_tile && abase == bbase, l31, hi)) << 16 * fn;
          }
          col[fn] = spread_col_bits(bits, hi, same_tile && abase == bbase, l31);
          if (hi == 0) tbits[bbase + l31][abase >> 5] = col[fn];
        }
        store_row_bits(col[0], col[1], hi, l31, abase, wn * G::WTN, dbits);
      }
      np = list_pairs(left, kWavePairs, wm * G::WTM, wn * G::WTN, pairs);
      full = any_over(kWavePairs) || !bounded;   // from here on: hand the tile back
      if (two && more) start(cn, buf ^ 1, 0, K);
    }
    // the waves' lists taken as one, dealt to the waves a batch at a time
    int pre[G::NWAVES + 1];   // scalars: pairs before each wave's
    pre[0] = 0;
    if (!full) {
      const int mine = cnt[el & 7];
#pragma unroll
      for (int i = 0; i < G::NWAVES; ++i) pre[i + 1] = pre[i] + __builtin_amdgcn_readlane(mine, i);
    } else {
#pragma unroll
      for (int i = 0; i < G::NWAVES; ++i) pre[i + 1] = 0;
    }
    const int all = pre[G::NWAVES];
    const uint32_t* lists = reinterpret_cast<const uint32_t*>(lds + kListOff);
    auto item = [&](int i) {   // place of pair i (< all) in the lists
      int at = i;
#pragma unroll
      for (int q = 1; q < G::NWAVES; ++q)
        if (i >= pre[q]) at = q * kWavePairs + i - pre[q];
      return at;
    };
    uint32_t* close = reinterpret_cast<uint32_t*>(lds + kCloseOff) + w * kWavePairs;
    int nclose = 0;
    if (first_only) {
      // the whole fp8 products, eight pairs at a time; a decided edge is set, the
      // pairs still within the band are kept for the dot product.  (The first da
      // values once more: a sum kept from the accumulators would need each pair's
      // own register.)
      const int32_t* tk = tokens(buf);
      constexpr int NP = 8;
      for (int i0 = w * NP; i0 < all; i0 += G::NWAVES * NP) {
        const uint8_t *pa[NP], *pb[NP];
        float s[NP];
        const int my = item(min(i0 + (el & (NP - 1)), all - 1));
        const uint32_t pr = lists[my];
        const int ta = tk[pr >> 8], tb = tk[kTile + (pr & 255)];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          pa[u] = sa.x8 + static_cast<size_t>(__builtin_amdgcn_readlane(ta, u)) * sa.dp;
          pb[u] = sa.x8 + static_cast<size_t>(__builtin_amdgcn_readlane(tb, u)) * sa.dp;
          s[u] = 0.f;
        }
        // two 1 KB pieces of every row in flight (the loads' latency, not their
        // bytes, is what a batch waits for)
        for (int cc = el * 16; cc < sa.dp; cc += 2048) {
          uint4 a[2][NP], b[2][NP];
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int u = 0; u < NP; ++u) {
              const bool in = cc + 1024 * h2 < sa.dp;
              a[h2][u] = in ? *reinterpret_cast<const uint4*>(pa[u] + cc + 1024 * h2) : make_uint4(0u, 0u, 0u, 0u);
              b[h2][u] = in ? *reinterpret_cast<const uint4*>(pb[u] + cc + 1024 * h2) : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int u = 0; u < NP; ++u) {
              const uint32_t aw[4] = {a[h2][u].x, a[h2][u].y, a[h2][u].z, a[h2][u].w};
              const uint32_t bw[4] = {b[h2][u].x, b[h2][u].y, b[h2][u].z, b[h2][u].w};
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const auto a0 = __builtin_amdgcn_cvt_pk_f32_fp8(aw[q], false), a1 = __builtin_amdgcn_cvt_pk_f32_fp8(aw[q], true);
                const auto b0 = __builtin_amdgcn_cvt_pk_f32_fp8(bw[q], false), b1 = __builtin_amdgcn_cvt_pk_f32_fp8(bw[q], true);
                s[u] = fmaf(a0[0], b0[0], s[u]);
                s[u] = fmaf(a0[1], b0[1], s[u]);
                s[u] = fmaf(a1[0], b1[0], s[u]);
                s[u] = fmaf(a1[1], b1[1], s[u]);
              }
            }
        }
        float sum = 0.f;   // of pair i0 + el % NP
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          const float t = wave_sum_dpp(s[u]);
          sum = (el & (NP - 1)) == u ? t : sum;
        }
        const float d = sum - hs;
        const bool mine = el < NP && i0 + el < all;
        const bool near = mine && !(fabsf(d) >= band);   // (a NaN goes on to the dot product)
        if (mine && d >= band) {
          const int r = pr >> 8, q = pr & 255;
          atomicOr(&dbits[r][q >> 5], 1u << (q & 31));
          atomicOr(same_tile ? &dbits[q][r >> 5] : &tbits[q][r >> 5], 1u << (r & 31));
        }
        const uint64_t m = __ballot(near);
        if (near) close[nclose + __popcll(m & lanemask_lt())] = pr;
        nclose += __popcll(m);
      }
      asm volatile("" ::: "memory");   // the kept entries cross lanes
    }
    if (first_only ? nclose > 0 : all > 0) {
      // bf16 cosines, four pairs at a time; float32 sums of d products in any
      // two orders differ by less than 2 d 2^-24 of |a| |b|
      const float tie = static_cast<float>(2 * sa.d + 64) * 0x1p-24f;
      const int32_t* tk = tokens(buf);
      constexpr int NP = 4;
      const int n4 = first_only ? nclose : all, step = first_only ? NP : G::NWAVES * NP;
      for (int i0 = first_only ? 0 : w * NP; i0 < n4; i0 += step) {
        const uint16_t *pa[NP], *pb[NP];
        float s[NP];
        const int my = min(i0 + (el & (NP - 1)), n4 - 1);
        const uint32_t pr = first_only ? close[my] : lists[item(my)];
        const int ta = tk[pr >> 8], tb = tk[kTile + (pr & 255)];
        const float ia = sa.inv_norm[ta], ib = sa.inv_norm[tb];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          pa[u] = sa.x + static_cast<size_t>(__builtin_amdgcn_readlane(ta, u)) * sa.d;
          pb[u] = sa.x + static_cast<size_t>(__builtin_amdgcn_readlane(tb, u)) * sa.d;
          s[u] = 0.f;
        }
        for (int cc = el * 8; cc < sa.d; cc += 512) {
          Pack16 a[NP], b[NP];
#pragma unroll
          for (int u = 0; u < NP; ++u) {
            a[u].u4 = *reinterpret_cast<const uint4*>(pa[u] + cc);
            b[u].u4 = *reinterpret_cast<const uint4*>(pb[u] + cc);
          }
#pragma unroll
          for (int u = 0; u < NP; ++u)
#pragma unroll
            for (int q = 0; q < 8; ++q) s[u] = fmaf(bf16_to_f32(a[u].h[q]), bf16_to_f32(b[u].h[q]), s[u]);
        }
        float dot = 0.f;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          const float t = wave_sum_dpp(s[u]);
          dot = (el & (NP - 1)) == u ? t : dot;
        }
        const float cs = dot * ia * ib;
        if (el < NP && i0 + el < n4) {
          const int r = pr >> 8, q = pr & 255;
          uint32_t* dw = &dbits[r][q >> 5];
          uint32_t* tw = same_tile ? &dbits[q][r >> 5] : &tbits[q][r >> 5];
          if (fabsf(cs - sa.h) < tie) cnt[8] = 1;
          if (cs >= sa.h) {   // (a NaN cosine is no edge in either pass)
            atomicOr(dw, 1u << (q & 31));
            atomicOr(tw, 1u << (r & 31));
          } else {
            atomicAnd(dw, ~(1u << (q & 31)));
            atomicAnd(tw, ~(1u << (r & 31)));
          }
        }
      }
    }
    // LDS-only barriers: a full __syncthreads() would also wait for the next
    // tile's DMA (the pieces of the products passed any_over's)
    if (all > 0) {
      __builtin_amdgcn_s_waitcnt(0xC07F);
      raw_barrier();
    }
    if (!full && __builtin_amdgcn_readfirstlane(cnt[8]) == 0)
      write_gram_tile(c, dbits, tbits, bitmask, bm_off[c.e], deg, G::THREADS);
    else if (opaque_tid() == 0)
      sa.list[atomicAdd(sa.list_count, 1)] = tile;
    if (!more) {
      wait_vmcnt<0>();   // a second phase's first stages that were not needed
      break;
    }
    if (whole > 0) --whole;
    // every wave's reads of the tile's LDS state are done before the next
    // tile overwrites it
    __builtin_amdgcn_s_waitcnt(0xC07F);
    raw_barrier();
    tile = ntile;
    c = cn;
  }
}

// Values of a row the screen's first phase multiplies, a multiple of 128: the
// fewest that leave unrelated pairs (cosine about 0, estimate spread
// sqrt(f / d) over a share f of d values) well below h minus what the rows
// keep beyond them (about 1 - f, spread with the rows) and the quantisation
// bound (about 0.05 sqrt(f) + 0.004), or all of them (one phase) where that
// would be more than half.  Only speed depends on it.
int screen_first_values(int d, int dp, float h) {
  for (int da = 128; 2 * da <= d; da += 128) {
    const float f = static_cast<float>(da) / static_cast<float>(d);
    const float room = h - (1.f - f), sd = sqrtf(f / static_cast<float>(d));
    if (room >= 0.02f + 0.05f * sqrtf(f) + 6.f * sd) return da;
  }
  return dp;
}

// ------------------------------------------------------------ history
// Historical similarity (Sec. 5.1 step 2): a pair of tokens whose weight in
// the previous block was above S1 takes weight 1 here, one below S2 takes
// weight 0, and only the other pairs use their cosine.  A block leaves the
// next one a record of its own weights as two bit classes per pair of
// positions of one bucket, in the layout of the adjacency bitmask:
// hi (weight > S1) and lo (weight < S2), with hi taking precedence.  The
// record also keeps the block's token -> position map and bucket layout, so
// the next block, whose buckets differ, can find a pair (t, u) in it: the
// pair is decided when t and u shared a bucket there.
constexpr int kHistMagic = 0x4C594831;   // record format tag

struct HistRec {
  int32_t* info;        // magic, T, E, k, max_bucket
  int32_t* slot_pos;    // [T*k] position of slot (t, j) in the writing block, -1 if dropped
  int32_t* offsets;     // [E+1] its buckets
  long long* word_off;  // [E+1] first word of bucket e in hi and lo
  uint64_t* hi;         // [cap_words]
  uint64_t* lo;         // [cap_words]
};

HistRec carve_hist(Carver& c, int T, int E, int k, int max_bucket) {
  HistRec h;
  const long long S = static_cast<long long>(T) * k;
  const long long cap_words = S * ((static_cast<long long>(max_bucket) + 63) / 64);
  h.info = c.take<int32_t>(8);
  h.slot_pos = c.take<int32_t>(static_cast<size_t>(S));
  h.offsets = c.take<int32_t>(E + 1);
  h.word_off = c.take<long long>(E + 1);
  h.hi = c.take<uint64_t>(static_cast<size_t>(cap_words));
  h.lo = c.take<uint64_t>(static_cast<size_t>(cap_words));
  return h;
}


// Header of the record a block leaves: format, sizes, the token -> position
// map, bucket offsets and word offsets (after the layout).  A layout error
// (a bucket larger than max_bucket) leaves the record marked invalid, which
// makes the next block compute every pair.
__global__ __launch_bounds__(256) void hist_header_kernel(const int32_t* __restrict__ slot_pos, int T, int k,
                                                          const int32_t* __restrict__ offsets, int E, int max_bucket,
                                                          const long long* __restrict__ bm_off,
                                                          const int* __restrict__ err, HistRec out) {
  const long long S = static_cast<long long>(T) * k;
  for (long long i = blockIdx.x * 256ll + threadIdx.x; i < S; i += gridDim.x * 256ll) out.slot_pos[i] = slot_pos[i];
  if (blockIdx.x == 0) {
    if (threadIdx.x <= static_cast<unsigned>(E)) {
      out.offsets[threadIdx.x] = offsets[threadIdx.x];
      out.word_off[threadIdx.x] = bm_off[threadIdx.x];
    }
    if (threadIdx.x == 0) {
      out.info[0] = *err ? 0 : kHistMagic;
      out.info[1] = T;
      out.info[2] = E;
      out.info[3] = k;
      out.info[4] = max_bucket;
    }
  }
}

// Previous position of every slot of every position of this block, as
// (previous bucket << 24) | position inside it, -1 where the token had no
// kept slot there; every entry -1 when the record does not match (T, E, k,
// max_bucket) or is marked invalid.  One thread per position.
template <int K>
__global__ __launch_bounds__(256) void hist_cols_kernel(const int32_t* __restrict__ offsets, int E,
                                                        const int32_t* __restrict__ perm_token,
                                                        const int* __restrict__ err, HistRec in, int T,
                                                        int max_bucket, int32_t* __restrict__ colinfo) {
  __shared__ int poff[kMaxExperts + 1];
  __shared__ int rec_ok;
  if (*err) return;
  if (threadIdx.x == 0)
    rec_ok = in.info[0] == kHistMagic && in.info[1] == T && in.info[2] == E && in.info[3] == K &&
             in.info[4] == max_bucket;
  __syncthreads();
  const bool ok = rec_ok;
  if (ok && threadIdx.x <= static_cast<unsigned>(E)) poff[threadIdx.x] = in.offsets[threadIdx.x];
  __syncthreads();
  const int S = offsets[E];
  for (int p = blockIdx.x * 256 + threadIdx.x; p < S; p += gridDim.x * 256) {
    const int u = perm_token[p];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      int v = -1;
      if (ok) {
        const int q = in.slot_pos[static_cast<size_t>(u) * K + j];
        if (q >= 0) {
          const int pe = bucket_of(poff, E, q);
          v = (pe << 24) | (q - poff[pe]);
        }
      }
      colinfo[static_cast<size_t>(p) * K + j] = v;
    }
  }
}

// The previous block's classes of every pair of this block's buckets, in
// this block's bitmask layout: rb_hi / rb_lo bit c of row a of bucket e is
// set when tokens perm_token[lo+a] and perm_token[lo+c] shared a bucket in
// the previous block with class hi / lo there.  One block per kGatherRows
// rows of one bucket; each wave walks 64 columns of a 256-column chunk (the
// columns' previous positions from colinfo), and for each row reads the
// previous row's word of each matching column straight from memory (a row is
// a few KB, so its words stay in L1 / L2 while the block walks it).
constexpr int kGatherRows = 8;

template <int K>
__global__ __launch_bounds__(256) void hist_gather_kernel(const int32_t* __restrict__ offsets, int E,
                                                          const long long* __restrict__ bm_off,
                                                          const int* __restrict__ err, HistRec in,
                                                          const int32_t* __restrict__ colinfo,
                                                          uint64_t* __restrict__ rb_hi, uint64_t* __restrict__ rb_lo) {
  __shared__ int rinfo[kGatherRows][K];        // previous bucket of the rows' slots (-1: none)
  __shared__ long long rbase[kGatherRows][K];  // first word of that previous row
  __shared__ int tile_e, tile_a0, tile_rows;
  if (*err) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  constexpr int G = kGatherRows;
  if (w == 0) {
    // this block's bucket and first row: lane e holds bucket e's row groups
    const int n = lane < E ? offsets[lane + 1] - offsets[lane] : 0;
    const int g = (n + G - 1) / G;
    int incl = g;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    const int b = blockIdx.x;
    const int e = __popcll(__ballot(lane < E && incl <= b));
    const int es = e < E ? e : 0;
    const int excl = __shfl(incl - g, es, 64);
    const int ne = __shfl(n, es, 64);
    if (lane == 0) {
      tile_e = e < E ? e : -1;
      tile_a0 = (b - excl) * G;
      tile_rows = min(G, ne - tile_a0);
    }
  }
  __syncthreads();
  const int e = tile_e;
  if (e < 0) return;
  const int lo = offsets[e], n = offsets[e + 1] - lo, W = (n + 63) / 64;
  const int a0 = tile_a0, rows = tile_rows;
  if (tid < G * K) {
    const int i = tid / K, j = tid % K;
    const int ri = i < rows ? colinfo[static_cast<size_t>(lo + a0 + i) * K + j] : -1;
    long long base = 0;
    if (ri >= 0) {
      const int pe = ri >> 24, pl = ri & 0xFFFFFF;
      const int wq = (in.offsets[pe + 1] - in.offsets[pe] + 63) / 64;
      base = in.word_off[pe] + static_cast<long long>(pl) * wq;
    }
    rinfo[i][j] = ri < 0 ? -1 : (ri >> 24);
    rbase[i][j] = base;
  }
  __syncthreads();
  for (int c0 = 0; c0 < n; c0 += 256) {
    const int c = c0 + tid;
    int qv[K];
#pragma unroll
    for (int j = 0; j < K; ++j) qv[j] = c < n ? colinfo[static_cast<size_t>(lo + c) * K + j] : -1;
    const int wd = (c0 >> 6) + w;
    // the words of all G rows are loaded before any is used, so their
    // latencies overlap
    long long widx[G];
    int bit[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      widx[i] = -1;
      bit[i] = 0;
#pragma unroll
      for (int jr = K - 1; jr >= 0; --jr) {
        const int pe = i < rows ? rinfo[i][jr] : -1;
#pragma unroll
        for (int jc = K - 1; jc >= 0; --jc) {
          if (pe >= 0 && qv[jc] >= 0 && (qv[jc] >> 24) == pe) {
            const int q = qv[jc] & 0xFFFFFF;
            widx[i] = rbase[i][jr] + (q >> 6);
            bit[i] = q & 63;
          }
        }
      }
    }
    uint64_t vh[G], vl[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      vh[i] = widx[i] >= 0 ? in.hi[widx[i]] : 0ull;
      vl[i] = widx[i] >= 0 ? in.lo[widx[i]] : 0ull;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
      if (i >= rows) break;
      const uint64_t mh = __ballot((vh[i] >> bit[i]) & 1ull), ml = __ballot((vl[i] >> bit[i]) & 1ull);
      if (lane == 0 && wd < W) {
        const long long o = bm_off[e] + static_cast<long long>(a0 + i) * W + wd;
        rb_hi[o] = mh;
        rb_lo[o] = ml;
      }
    }
  }
}

// The same gather for buckets whose previous rows fit in LDS: the previous rows
// (both slots) of the block's G rows (8, or 4 where buckets may be large) are copied to LDS once, coalesced, hi and lo
// words side by side, and a lane (column) then takes both class bits of its
// previous position with one 8-byte LDS read.  The columns of a word keep their
// order from block to block, so most of a wave's reads fall on two or three
// words and are broadcasts.  A position is (previous bucket << 24) | place in it
// (colinfo), so its exclusive or with a row's previous bucket << 24 is the place
// itself where the buckets match and at least 2^24 where they do not; a token's
// two slots lie in different buckets, so at most one matches.  Neighbouring rows
// mostly come from the same previous bucket (a bucket holds its first choices,
// then its second ones), and the columns' places in it are then taken over from
// the row before.  The kernel is bound by its vector instructions, 8 to 25 per
// row and 64 columns (with a row's words in memory and 64-bit addresses about
// 60, and one-lane stores), and by a block's chain of loads before it starts,
// which the other block of the CU hides.  65536 slots in 32 buckets of up to
// 19,400, bound of 32768 (4 rows a block): 1005 -> 350-360 us (one block a CU 423,
// its rows copied one after the other 620); 16384 in 16 of at most 1280 (8 rows):
// 53 -> 25 us.
constexpr uint32_t kNoBucket = 0xC0000000u;   // matches no position
constexpr size_t kGatherLdsMax = 76 * 1024;   // two blocks in a CU's 160 KB

// Bytes of one previous row in LDS: 8 bytes per 32 positions and a zero entry
// (the last) for columns that were not in its bucket.
inline size_t hist_row_bytes(int max_bucket) { return (static_cast<size_t>(max_bucket) + 63) / 64 * 16 + 16; }

template <int K, int G>
__global__ __launch_bounds__(1024) void hist_gather_lds_kernel(const int32_t* __restrict__ offsets, int E,
                                                              const long long* __restrict__ bm_off,
                                                              const int* __restrict__ err, HistRec in, int row_bytes,
                                                              const int32_t* __restrict__ colinfo,
                                                              uint64_t* __restrict__ rb_hi,
                                                              uint64_t* __restrict__ rb_lo) {
  extern __shared__ __attribute__((aligned(16))) uint8_t rows_lds[];   // [row][slot][row_bytes]
  if (*err) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this block's bucket and first row: lane e holds bucket e's row groups
  const int o0 = lane < E ? offsets[lane] : 0;
  const int nl = lane < E ? offsets[lane + 1] - o0 : 0;
  const int g = (nl + G - 1) / G;
  int incl = g;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  const int b = blockIdx.x;
  const int e = __popcll(__ballot(lane < E && incl <= b));
  if (e >= E) return;
  const int lo = __builtin_amdgcn_readlane(o0, e), n = __builtin_amdgcn_readlane(nl, e), W = (n + 63) / 64;
  const int a0 = (b - (__builtin_amdgcn_readlane(incl, e) - __builtin_amdgcn_readlane(g, e))) * G;
  const int rows = min(G, n - a0);
  // previous bucket and first word of every row and slot (lane i K + j)
  int ri = -1, pw = 0;
  long long base = 0;
  if (lane < rows * K) {
    ri = colinfo[static_cast<size_t>(lo + a0) * K + lane];
    if (ri >= 0) {
      const int pe = ri >> 24;
      pw = (in.offsets[pe + 1] - in.offsets[pe] + 63) / 64;
      base = in.word_off[pe] + static_cast<long long>(ri & 0xFFFFFF) * pw;
    }
  }
  // entry 2 w (2 w + 1): low (high) half of word w of both classes, bit-reversed
  // so that a left shift by a place brings its bit to the sign
  const int zero_idx = row_bytes / 8 - 1;
  for (int r = w; r < G * K; r += static_cast<int>(blockDim.x) / 64) {   // a wave a row
    const int words = __builtin_amdgcn_readlane(pw, r);
    const long long at = (static_cast<long long>(__builtin_amdgcn_readlane(static_cast<int>(base >> 32), r)) << 32) |
                         static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(base), r));
    uint8_t* row = rows_lds + static_cast<size_t>(r) * row_bytes;
    constexpr int U = 4;   // pieces of the row in flight
    for (int i0 = lane; i0 < words; i0 += 64 * U) {
      uint64_t h[U], l[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in_row = i0 + 64 * u < words;
        h[u] = in_row ? in.hi[at + i0 + 64 * u] : 0ull;
        l[u] = in_row ? in.lo[at + i0 + 64 * u] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + 64 * u < words)
          *reinterpret_cast<uint4*>(row + 16 * (i0 + 64 * u)) =
              make_uint4(__brev(static_cast<uint32_t>(h[u])), __brev(static_cast<uint32_t>(l[u])),
                         __brev(static_cast<uint32_t>(h[u] >> 32)), __brev(static_cast<uint32_t>(l[u] >> 32)));
    }
    if (lane == 0) *reinterpret_cast<uint2*>(row + 8 * zero_idx) = make_uint2(0u, 0u);
  }
  uint32_t P[G][K];   // scalars
#pragma unroll
  for (int i = 0; i < G; ++i)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const int v = __builtin_amdgcn_readlane(ri, i * K + j);
      P[i][j] = v >= 0 ? static_cast<uint32_t>(v) & 0xFF000000u : kNoBucket;
    }
  __syncthreads();
  // the lane that stores: row lane % G of class hi (lanes 0 .. G - 1) or lo (G .. 2 G - 1)
  const bool store = lane < 2 * G && (lane & (G - 1)) < rows;
  uint64_t* dst = (lane < G ? rb_hi : rb_lo) + bm_off[e] + static_cast<long long>(a0 + (lane & (G - 1))) * W;
  // two words (128 columns) a wave and pass: 16 bytes a storing lane
  for (int wd = 2 * w; wd < W; wd += blockDim.x / 32) {
    int ww[2][2] = {};   // [word][half]: lane i: row i's hi word; lane 8 + i: its lo word
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const int c = (wd + h2) * 64 + lane;
      uint32_t qv[K];
#pragma unroll
      for (int j = 0; j < K; ++j) qv[j] = c < n ? static_cast<uint32_t>(colinfo[static_cast<size_t>(lo + c) * K + j]) : ~0u;
      // the columns' places in the row's previous bucket (slot j), kept while
      // the bucket stays the same from row to row; offset of their entry
      uint32_t m[K], at[K];
      bool miss = false;   // a column was not in the first slot's bucket (wave-uniform)
      auto places = [&](uint32_t bucket, int j) {
        uint32_t x = qv[0] ^ bucket;
        if constexpr (K == 2) x = min(x, qv[1] ^ bucket);
        m[j] = x;
        at[j] = 8u * min(x >> 5, static_cast<uint32_t>(zero_idx));
      };
      uint2 v[G];
      uint32_t pos[G];
#pragma unroll
      for (int i = 0; i < G; ++i) {
        if (i == 0 || P[i][0] != P[i - 1][0]) {
          places(P[i][0], 0);
          miss = __ballot(m[0] >= (1u << 24)) != 0;
        }
        const uint8_t* row = rows_lds + static_cast<uint32_t>(i * K) * row_bytes;
        uint32_t off = at[0];
        pos[i] = m[0];
        if constexpr (K == 2) {
          // the row's first slot takes precedence over its second
          if (miss) {
            places(P[i][1], 1);
            const bool second = m[0] >= (1u << 24);
            off = second ? at[1] + row_bytes : off;
            pos[i] = second ? m[1] : m[0];
          }
        }
        v[i] = *reinterpret_cast<const uint2*>(row + off);
      }
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const uint64_t mh = __ballot(static_cast<int>(v[i].x << (pos[i] & 31)) < 0);
        const uint64_t ml = __ballot(static_cast<int>(v[i].y << (pos[i] & 31)) < 0);
        ww[h2][0] = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(mh)), i, ww[h2][0]);
        ww[h2][1] = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(mh >> 32)), i, ww[h2][1]);
        ww[h2][0] = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(ml)), G + i, ww[h2][0]);
        ww[h2][1] = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(ml >> 32)), G + i, ww[h2][1]);
      }
    }
    if (store) {
      const uint4 o = make_uint4(ww[0][0], ww[0][1], ww[1][0], ww[1][1]);
      if (wd + 1 < W) __builtin_memcpy(dst + wd, &o, 16);
      else __builtin_memcpy(dst + wd, &o, 8);
    }
  }
}

// Constants of a block's pair weights: a decided pair's weight is 1 or 0,
// which gives its edge (w >= h) and its classes for the next block
// (w > S1, w < S2) without a cosine.
struct HistParams {
  float h, S1, S2;
  uint64_t* out_hi;   // record words of this block (nullptr: no record)
  uint64_t* out_lo;
  const uint64_t* rb_hi;   // previous classes in this block's layout (nullptr: none)
  const uint64_t* rb_lo;
  unsigned long long* stats;   // undecided pairs, decided pairs, tiles computed, tiles skipped
  int* queue;                  // kTileQueues tile counters, zero at launch
};

// Words of one row piece from its (hi, lo) previous classes, for a tile
// whose pairs are all decided: edge, class hi and class lo of every pair
// under the valid mask vm.
__device__ __forceinline__ void decided_words(uint64_t hi, uint64_t lo, uint64_t vm, const HistParams& hp,
                                              uint64_t& edge, uint64_t& rh, uint64_t& rl) {
  const uint64_t one = hi & vm, zero = lo & ~hi & vm;
  edge = (1.0f >= hp.h ? one : 0ull) | (0.0f >= hp.h ? zero : 0ull);
  rh = (1.0f > hp.S1 ? one : 0ull) | (0.0f > hp.S1 ? zero : 0ull);
  rl = (1.0f < hp.S2 ? one : 0ull) | (0.0f < hp.S2 ? zero : 0ull);
}

// Columns of word wd (global word index) of a row that are pairs inside the
// bucket: columns < n, the row's own position excluded.
__device__ __forceinline__ uint64_t pair_mask(int row, int wd, int n) {
  const int c0 = wd * 64;
  uint64_t m = n - c0 >= 64 ? ~0ull : (n - c0 <= 0 ? 0ull : (1ull << (n - c0)) - 1);
  if (row >= c0 && row < c0 + 64) m &= ~(1ull << (row - c0));
  return m;
}

// bf16 similarity with history.  Per tile: the previous classes of its pairs
// (rows of tile-row ti, words of tile-column tj) are read into LDS; the
// undecided and decided pairs above the diagonal are counted; a tile whose
// pairs are all decided skips the product and derives its words from the
// classes alone (its mirror from the mirrored classes, which are the same
// pairs); any other tile runs the product and takes, pair by pair, weight 1
// or 0 where the previous block decided it and the cosine elsewhere.  The
// record of this block (classes of every weight) is written beside the
// adjacency words, direct and mirrored.
// LIST: only the tiles the history screen handed back (which has counted their
// pairs).
template <bool HIN, bool HOUT, bool LIST = false>
__global__ __launch_bounds__(GramGemm::THREADS) void gram_hist_kernel_bf16(
    const uint16_t* __restrict__ X, int d, const int32_t* __restrict__ perm_token,
    const int32_t* __restrict__ offsets, int E, const float* __restrict__ inv_norm, HistParams hp,
    const int32_t* __restrict__ tile_off, const long long* __restrict__ bm_off,
    const int* __restrict__ err, uint64_t* __restrict__ bitmask, int32_t* __restrict__ deg,
    const int* __restrict__ list, const int* __restrict__ list_count) {
  using G = GramGemm;
  __shared__ __attribute__((aligned(16))) uint8_t lds[G::LDS_BYTES];
  __shared__ __attribute__((aligned(16))) float inv_a[kTile];
  __shared__ float inv_b[kTile];
  __shared__ __attribute__((aligned(16))) uint64_t rbw[2][kTile][4];   // previous classes of the tile's pairs
  __shared__ unsigned long long cnt_s[2];
  constexpr int NM = HOUT ? 3 : 1;   // masks built per tile: edge, then class hi and class lo
  // after the K loop the operand buffers hold the masks' pieces:
  // dbits[m][row][32-column group], tbits[m][column][32-row group]
  auto dbits = reinterpret_cast<uint32_t (*)[kTile][kTile / 32]>(lds);
  auto tbits = reinterpret_cast<uint32_t (*)[kTile][kTile / 32]>(lds + NM * kTile * kTile / 8);
  static_assert(2 * NM * kTile * kTile / 8 <= G::LDS_BYTES, "mask pieces fit the operand buffer");
  if (*err) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = G::wave_m(w), wn = G::wave_n(w);
  const int total = LIST ? *list_count : tile_off[E];
  // Tiles cost very different times (skipped or computed), so blocks take
  // them from queues: queue x holds the x-th eighth of the tile order, a
  // block first drains the queue of its own XCD (blocks are dealt to the
  // XCDs round-robin), then the others'.  Listed tiles are all computed and are
  // taken in turn: eight empty queues alone took 27 us.
  __shared__ int next_tile;
  const int home = blockIdx.x % kTileQueues;
  int qi = 0;
  for (int item = LIST ? xcd_virtual_block() : 0;; item += gridDim.x) {
    if (tid == 0) {
      int t = -1;
      if (LIST && item < total) t = list[item];
      while (!LIST && qi < kTileQueues) {
        const int x = (home + qi) % kTileQueues;
        const int t0 = static_cast<int>(static_cast<long long>(total) * x / kTileQueues);
        const int t1 = static_cast<int>(static_cast<long long>(total) * (x + 1) / kTileQueues);
        const int v = atomicAdd(&hp.queue[x], 1);
        if (t0 + v < t1) {
          t = t0 + v;
          break;
        }
        ++qi;
      }
      next_tile = t;
    }
    __syncthreads();
    if (next_tile < 0) break;
    const int tile = next_tile;
    const TileCoord c = decode_tile_grouped(tile, tile_off, offsets, E);
    const int32_t* pt = perm_token + c.lo;
    const long long bmo = bm_off[c.e];
    const int nrow_a = c.n - c.ti * kTile, nrow_b = c.n - c.tj * kTile;
    const bool same_tile = c.ti == c.tj;
    // previous classes of the tile's pairs; count undecided / decided pairs
    // above the diagonal
    if (tid < 2) cnt_s[tid] = 0;
    __syncthreads();
    int undecided = 0;
    {
      unsigned long long nu = 0, nd = 0;
      for (int i = tid; i < kTile * 4; i += G::THREADS) {
        const int rl = i >> 2, ww = i & 3;
        const int a = c.ti * kTile + rl, wd = 4 * c.tj + ww;
        uint64_t h1 = 0, l1 = 0, vm = 0;
        if (a < c.n && wd < c.W) {
          vm = pair_mask(a, wd, c.n);
          if constexpr (HIN) {
            h1 = hp.rb_hi[bmo + static_cast<long long>(a) * c.W + wd];
            l1 = hp.rb_lo[bmo + static_cast<long long>(a) * c.W + wd];
          }
        }
        rbw[0][rl][ww] = h1;
        rbw[1][rl][ww] = l1;
        const uint64_t und = ~(h1 | l1) & vm;
        undecided |= und != 0;
        // pairs above the diagonal only (columns > row) on a diagonal tile
        uint64_t up = ~0ull;
        if (same_tile) {
          const int c0 = wd * 64;
          up = a < c0 ? ~0ull : (a >= c0 + 63 ? 0ull : ~((2ull << (a - c0)) - 1));
        }
        nu += __popcll(und & up);
        nd += __popcll(vm & ~und & up);
      }
      if (nu) atomicAdd(&cnt_s[0], nu);
      if (nd) atomicAdd(&cnt_s[1], nd);
    }
    undecided = __syncthreads_or(undecided);
    if (!LIST && tid == 0) {
      atomicAdd(&hp.stats[0], cnt_s[0]);
      atomicAdd(&hp.stats[1], cnt_s[1]);
      atomicAdd(&hp.stats[undecided ? 2 : 3], 1ull);
    }
    if (!undecided) {
      // every pair decided: no product; direct words from rbw, mirrored
      // words from the mirrored classes (same pairs, read from rb)
      for (int i = tid; i < 2 * kTile * 4; i += G::THREADS) {
        const bool mirror = i >= kTile * 4;
        if (mirror && same_tile) continue;
        const int j = mirror ? i - kTile * 4 : i;
        const int rl = j >> 2, ww = j & 3;
        const int a = (mirror ? c.tj : c.ti) * kTile + rl, wd = 4 * (mirror ? c.ti : c.tj) + ww;
        if (a >= c.n || wd >= c.W) continue;
        const long long o = bmo + static_cast<long long>(a) * c.W + wd;
        const uint64_t h1 = mirror ? hp.rb_hi[o] : rbw[0][rl][ww];
        const uint64_t l1 = mirror ? hp.rb_lo[o] : rbw[1][rl][ww];
        uint64_t edge, rh, rlw;
        decided_words(h1, l1, pair_mask(a, wd, c.n), hp, edge, rh, rlw);
        bitmask[o] = edge;
        if constexpr (HOUT) {
          hp.out_hi[o] = rh;
          hp.out_lo[o] = rlw;
        }
        if (edge) atomicAdd(&deg[c.lo + a], __popcll(edge));
      }
      __syncthreads();
      continue;
    }
    uint32_t poff[G::LP], qoff[G::LQ];
#pragma unroll
    for (int j = 0; j < G::LP; ++j)
      poff[j] = static_cast<uint32_t>(pt[min(c.ti * kTile + G::load_row(j), c.n - 1)]) * d;
#pragma unroll
    for (int j = 0; j < G::LQ; ++j)
      qoff[j] = static_cast<uint32_t>(pt[min(c.tj * kTile + G::load_row(G::LP + j) - G::BM, c.n - 1)]) * d;
    for (int i = tid; i < 2 * kTile; i += G::THREADS) {
      if (i < kTile) inv_a[i] = inv_norm[pt[min(c.ti * kTile + i, c.n - 1)]];
      else inv_b[i - kTile] = inv_norm[pt[min(c.tj * kTile + i - kTile, c.n - 1)]];
    }
    G::Acc acc;
    G::zero(acc);
    G::run(X, poff, X, qoff, d, nrow_a, nrow_b, lds, acc);  // ends with a barrier

    // Epilogue as in gram_kernel_bf16, for NM predicates per pair:
    //   weight w = 1 (class hi), 0 (class lo) or the cosine;
    //   edge = w >= h; next classes w > S1, w < S2.
    const int l31 = lane & 31, hi = lane >> 5;
    const uint32_t* rbh32 = reinterpret_cast<const uint32_t*>(&rbw[0][0][0]);
    const uint32_t* rbl32 = reinterpret_cast<const uint32_t*>(&rbw[1][0][0]);
    const bool e1 = 1.0f >= hp.h, e0 = 0.0f >= hp.h;
    const bool h1c = 1.0f > hp.S1, h0c = 0.0f > hp.S1, l1c = 1.0f < hp.S2, l0c = 0.0f < hp.S2;
#pragma unroll
    for (int fm = 0; fm < G::FM; ++fm) {
      const int abase = wm * G::WTM + 32 * fm;
      const float nan = __builtin_nanf("");
      float ia[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int al0 = abase + 8 * q + 4 * hi;
        const float4 f = *reinterpret_cast<const float4*>(&inv_a[al0]);
        const float fv[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) ia[4 * q + r] = al0 + r < nrow_a ? fv[r] : nan;
      }
#pragma unroll
      for (int fn = 0; fn < G::FN; ++fn) {
        const int bbase = wn * G::WTN + 32 * fn;
        const int bl = bbase + l31;
        const float ib = bl < nrow_b ? inv_b[bl] : nan;
        const bool diag = same_tile && abase == bbase;   // wave-uniform
        uint32_t colbits[NM], piece[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) colbits[m] = piece[m] = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int rv = 8 * (v >> 2) + (v & 3);
          const int row = abase + rv + 4 * hi;
          const bool hb = (rbh32[row * 8 + (bbase >> 5)] >> l31) & 1u;
          const bool lb = (rbl32[row * 8 + (bbase >> 5)] >> l31) & 1u;
          const float cs = acc[fm][fn][v] * ia[v] * ib;
          const bool self = diag && rv + 4 * hi == l31;
          bool pr[NM];
          pr[0] = !self && (hb ? e1 : (lb ? e0 : cs >= hp.h));
          if constexpr (HOUT) {
            pr[1] = !self && (hb ? h1c : (lb ? h0c : cs > hp.S1));
            pr[2] = !self && (hb ? l1c : (lb ? l0c : cs < hp.S2));
          }
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            const uint64_t bm = __ballot(pr[m]);
            piece[m] = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(bm)), rv, piece[m]);
            piece[m] = amdgcn_writelane(static_cast<int>(static_cast<uint32_t>(bm >> 32)), rv + 4, piece[m]);
            colbits[m] |= pr[m] ? 1u << rv : 0u;
          }
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          colbits[m] <<= 4 * hi;
          const uint32_t tv = colbits[m] | static_cast<uint32_t>(__shfl_xor(static_cast<int>(colbits[m]), 32, 64));
          if (lane < 32) {
            dbits[m][abase + l31][bbase >> 5] = piece[m];
            tbits[m][bl][abase >> 5] = tv;
          }
        }
      }
    }
    __syncthreads();
    for (int i = tid; i < 2 * kTile; i += G::THREADS) {
      const bool mirror = i >= kTile;
      const int rl = mirror ? i - kTile : i;
      const uint32_t* pcs = mirror ? tbits[0][rl] : dbits[0][rl];
      int cnt = 0;
#pragma unroll
      for (int g = 0; g < kTile / 32; ++g) cnt += __popc(pcs[g]);
      const int r = (mirror ? c.tj : c.ti) * kTile + rl;
      if (cnt && r < c.n && (!mirror || !same_tile)) atomicAdd(&deg[c.lo + r], cnt);
    }
    for (int i = tid; i < kTile * 4; i += G::THREADS) {
      const int rl = i >> 2, ww = i & 3;
      const int a = c.ti * kTile + rl, wd = 4 * c.tj + ww;
      const int bb = c.tj * kTile + rl, wt = 4 * c.ti + ww;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        uint64_t* dst = m == 0 ? bitmask : (m == 1 ? hp.out_hi : hp.out_lo);
        const uint64_t dv = static_cast<uint64_t>(dbits[m][rl][2 * ww]) |
                            (static_cast<uint64_t>(dbits[m][rl][2 * ww + 1]) << 32);
        if (a < c.n && wd < c.W) dst[bmo + static_cast<long long>(a) * c.W + wd] = dv;
        if (!same_tile) {
          const uint64_t tv = static_cast<uint64_t>(tbits[m][rl][2 * ww]) |
                              (static_cast<uint64_t>(tbits[m][rl][2 * ww + 1]) << 32);
          if (bb < c.n && wt < c.W) dst[bmo + static_cast<long long>(bb) * c.W + wt] = tv;
        }
      }
    }
    __syncthreads();
  }
}

// Words wd and wd + 1 of bitmask row `row` for the pairs of a tile: previous
// classes (if any) decide a pair's weight, its cosine's predicates e, g, l (weight
// >= h, > S1, < S2; bit pieces of 64 columns) the others.  Returns the row's
// edges among them.
__device__ __forceinline__ int store_hist_words(const HistParams& hp, uint64_t* __restrict__ bitmask, long long base,
                                                int row, int wd, int n, int W, const uint32_t* e, const uint32_t* g,
                                                const uint32_t* l) {
  if (row >= n || wd >= W) return 0;
  const long long o = base + static_cast<long long>(row) * W + wd;
  const int nw = min(2, W - wd);
  uint64_t oe[2], oh[2], ol[2];
  int edges = 0;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint64_t vm = u < nw ? pair_mask(row, wd + u, n) : 0ull;
    uint64_t one = 0, zero = 0;
    if (hp.rb_hi && u < nw) {
      one = hp.rb_hi[o + u];
      zero = hp.rb_lo[o + u];
    }
    decided_words(one, zero, vm, hp, oe[u], oh[u], ol[u]);
    const uint64_t und = ~(one | zero) & vm;
    auto word = [&](const uint32_t* p) { return static_cast<uint64_t>(p[2 * u]) | (static_cast<uint64_t>(p[2 * u + 1]) << 32); };
    oe[u] |= und & word(e);
    oh[u] |= und & word(g);
    ol[u] |= und & word(l);
    edges += __popcll(oe[u]);
  }
  if (nw == 2) {
    __builtin_memcpy(bitmask + o, oe, 16);
    __builtin_memcpy(hp.out_hi + o, oh, 16);
    __builtin_memcpy(hp.out_lo + o, ol, 16);
  } else {
    bitmask[o] = oe[0];
    hp.out_hi[o] = oh[0];
    hp.out_lo[o] = ol[0];
  }
  return edges;
}

// History similarity on the fp8 screen's rows (see gram_screen_kernel): a tile
// with an undecided pair takes its whole fp8 product, whose band decides a
// pair's three predicates (>= h, > S1, < S2) where its estimate is further than
// the band from all three thresholds; the few pairs closer to one get their
// bf16 dot product, and a tile with more than kWavePairs of them in a wave, or
// a dot product within float32 rounding of a threshold, is listed for the bf16
// pass.  The predicates' bit pieces of a tile are merged with its previous
// classes word by word as they are stored; most 32 x 32 blocks lie below every
// threshold as a whole and need no compares.  A tile whose pairs are all
// decided skips the product.  The tile loop is pipelined as the screen's, with
// one stage of the next tile's operands in flight: the other stage's LDS holds
// the pieces.  Where cosines crowd the thresholds, so that a block's tiles are
// handed back one after the other, it hands the next ones back at once (1, 3, then
// 7 of them) before it takes a product again.
// Why: the bf16 kernel spent 77,000 cycles of a 256 x 256 tile of d = 2048 on
// its K loop and as many on 3 predicates with two bit lookups a pair; fp8 halves
// the first and the word-level merge leaves one compare a predicate.  A later
// block of T = 32768, d = 2048, E = 32 (Zipf): 1405 -> 700 us, and 34 for the fp8
// rows and 6 for the bf16 pass, which nothing goes back to.
__global__ __launch_bounds__(GramGemm::THREADS) void gram_hist_screen_kernel(
    ScreenArgs sa, HistParams hp, const int32_t* __restrict__ perm_token, const int32_t* __restrict__ offsets, int E,
    const int32_t* __restrict__ tile_off, const long long* __restrict__ bm_off, const int* __restrict__ err,
    uint64_t* __restrict__ bitmask, int32_t* __restrict__ deg) {
  using G = GemmBig64F8;
  constexpr int kPieces = kTile * (kTile / 32) * 4;   // bytes of one mask's pieces, direct or transposed
  static_assert(G::STAGES == 2 && 6 * kPieces <= G::STAGE_BYTES && G::THREADS == 2 * kTile && G::NWAVES == 8,
                "three masks' pieces in the second stage");
  // one LDS array (see gram_kernel_bf16): the operand ring, whose second stage
  // holds the pieces d[m], then t[m], between K loops; the waves' row bounds,
  // the tokens of this tile and of the next, the bucket tables, every wave's
  // close pairs, their counts and the flags
  constexpr int kRedOff = G::LDS_BYTES, kTokOff = kRedOff + G::NWAVES * 4 + 32, kTabOff = kTokOff + 4 * kTile * 4;
  constexpr int kListOff = kTabOff + 3 * kMaxExperts * 4, kCntOff = kListOff + G::NWAVES * kWavePairs * 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kCntOff + 48];
  float* red = reinterpret_cast<float*>(lds + kRedOff);
  auto pieces = [&](int m, bool t) {
    return reinterpret_cast<uint32_t (*)[kTile / 32]>(lds + G::STAGE_BYTES + (m + (t ? 3 : 0)) * kPieces);
  };
  int* tab = reinterpret_cast<int*>(lds + kTabOff);
  int* cnt = reinterpret_cast<int*>(lds + kCntOff);   // [w]: pairs of wave w; [8]: hand back; [9]: undecided pairs
  if (*err) return;
  const int w = G::wave();
  const int wm = G::wave_m(w), wn = G::wave_n(w);
  const int total = tile_off[E];
  int tile = xcd_virtual_block();
  if (tile >= total) return;   // block-uniform, before any barrier
  const uint16_t* X = reinterpret_cast<const uint16_t*>(sa.x8);
  const int K = sa.dp / 2;   // 16-bit units, 64 a stage
  if (w == 0) {
    int to, o0, o1;
    bucket_lookup_loads(tile_off, offsets, E, to, o0, o1);
    const int l = opaque_tid();
    tab[l] = to;
    tab[kMaxExperts + l] = o0;
    tab[2 * kMaxExperts + l] = o1;
  }
  __syncthreads();
  auto decode = [&](int t) {
    const int l = opaque_tid() & 63;
    return decode_tile_grouped_from(t, tab[l], tab[kMaxExperts + l], tab[2 * kMaxExperts + l], E);
  };
  auto tokens = [&](int buf) { return reinterpret_cast<int32_t*>(lds + kTokOff) + buf * 2 * kTile; };
  auto fetch_tokens = [&](const TileCoord& t, int buf) {
    const int l = opaque_tid() & 63;
    const int r = (w < 4 ? t.ti : t.tj) * kTile + 64 * (w & 3) + l;
    const uint32_t off = static_cast<uint32_t>(t.lo + min(r, t.n - 1)) * 4u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        G::rsrc(perm_token),
        reinterpret_cast<__attribute__((address_space(3))) void*>((G::lds_ptr)(lds + kTokOff) + (buf * 2 * kTile + 64 * w) * 4),
        4, off, 0, 0, 0);
  };
  typename G::Pipe pipe;
  auto prepare = [&](const TileCoord& t, int buf) {
    const int32_t* tk = tokens(buf);
    uint32_t poff[G::LP], qoff[G::LQ];
#pragma unroll
    for (int j = 0; j < G::LP; ++j) {
      const int r = G::load_row(j);
      poff[j] = static_cast<uint32_t>(t.ti * kTile + r < t.n ? tk[r] : sa.T) * K;
    }
#pragma unroll
    for (int j = 0; j < G::LQ; ++j) {
      const int r = G::load_row(G::LP + j) - G::BM;
      qoff[j] = static_cast<uint32_t>(t.tj * kTile + r < t.n ? tk[kTile + r] : sa.T) * K;
    }
    G::prepare(X, poff, X, qoff, K, kTile, kTile, pipe);
  };
  auto issue_stage = [&](int st) {
#pragma unroll
    for (int i = 0; i < G::LOADS; ++i) G::issue_one(pipe, st * G::LOADS + i, lds);
  };
  auto bound = [&](const TileCoord& t, int buf) {
    const int i = opaque_tid();
    const int r = (i < kTile ? t.ti : t.tj - 1) * kTile + i;
    return r < t.n ? sa.rowq[tokens(buf)[i]].x : 0.f;
  };
  TileCoord c = decode(tile);
  fetch_tokens(c, 0);
  __syncthreads();   // (waits for the DMA too)
  float rq = bound(c, 0);
  prepare(c, 0);
  issue_stage(0);
  const float te = sa.h * 65536.f, tg = hp.S1 * 65536.f, tl = hp.S2 * 65536.f;
  const float tmin = fminf(fminf(te, tg), tl);
  unsigned long long nu = 0, nd = 0, tiles = 0, skipped = 0;
  // computed tiles handed back in a row (1, 2, 4, .. at most 8), and the tiles to
  // hand back without their product after them
  int strike = 0, direct = 0;
  for (int buf = 0;; buf ^= 1) {
    const int ntile = tile + gridDim.x;
    const bool more = ntile < total;
    const long long base = bm_off[c.e];
    const bool same_tile = c.ti == c.tj;
    issue_stage(1);
    TileCoord cn = c;
    if (more) {
      cn = decode(ntile);
      fetch_tokens(cn, buf ^ 1);   // lands under the K loop
    }
    // the tile's undecided and decided pairs above the diagonal
    int undecided = 0;
    {
      const int i = opaque_tid(), rl = i >> 1;
      const int a = c.ti * kTile + rl;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int wd = 4 * c.tj + 2 * (i & 1) + u;
        if (a < c.n && wd < c.W) {
          const uint64_t vm = pair_mask(a, wd, c.n);
          uint64_t dec = 0;
          if (hp.rb_hi) {
            const long long o = base + static_cast<long long>(a) * c.W + wd;
            dec = hp.rb_hi[o] | hp.rb_lo[o];
          }
          const uint64_t und = ~dec & vm;
          undecided |= und != 0;
          uint64_t up = ~0ull;
          if (same_tile) {
            const int c0 = wd * 64;
            up = a < c0 ? ~0ull : (a >= c0 + 63 ? 0ull : ~((2ull << (a - c0)) - 1));
          }
          nu += __popcll(und & up);
          nd += __popcll(vm & ~und & up);
        }
      }
      const float m = wave_max_dpp(rq);
      if ((i & 63) == 0) red[w] = m;
      if (i < 2) cnt[8 + i] = 0;
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);
    raw_barrier();
    if (__ballot(undecided) != 0 && (opaque_tid() & 63) == 0) cnt[9] = 1;
    __builtin_amdgcn_s_waitcnt(0xC07F);
    raw_barrier();
    const bool left = !hp.rb_hi || __builtin_amdgcn_readfirstlane(cnt[9]) != 0;   // block-uniform
    tiles += left;
    skipped += !left;
    const bool compute = left && direct == 0;
    if (left && direct > 0) --direct;
    typename G::Acc acc;
    G::zero(acc);
    if (compute) {
      G::resume(pipe, lds, acc);   // ends with a barrier: the ring is free
    } else {
      wait_vmcnt<0>();
      raw_barrier();
    }
    if (more) {
      rq = bound(cn, buf ^ 1);
      prepare(cn, buf ^ 1);
      issue_stage(0);
    }
    const int el = opaque_tid() & 63;
    const int l31 = el & 31, hi = el >> 5;
    bool back = left && !compute;   // block-uniform: too many close pairs
    if (compute) {
      float rho = 0.f;
#pragma unroll
      for (int i = 0; i < G::NWAVES; ++i) rho = fmaxf(rho, red[i]);
      const float band = (2.f * rho + rho * rho + 4e-3f) * 65536.f;
      uint32_t* pairs = reinterpret_cast<uint32_t*>(lds + kListOff) + w * kWavePairs;
      const int nra = c.n - c.ti * kTile, nrb = c.n - c.tj * kTile;
      uint32_t close[G::FM] = {};   // the close pairs of this lane's part (list_pairs)
      static_assert(G::FN == 2, "two blocks a word");
#pragma unroll
      for (int fm = 0; fm < G::FM; ++fm) {
        const int abase = wm * G::WTM + 32 * fm;
        uint32_t col[3][G::FN];
#pragma unroll
        for (int fn = 0; fn < G::FN; ++fn) {
          const int bbase = wn * G::WTN + 32 * fn;
          float mx = acc[fm][fn][0];
#pragma unroll
          for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[fm][fn][v]);
          uint32_t be = 0, bg = 0, bl = 0;   // bl: not below S2
          float dmin = __builtin_inff();
          // (a NaN product sets no bit of any of the three)
          if (__ballot(!(mx < tmin - band)) != 0) {
#pragma unroll
            for (int v = 15; v >= 0; --v) {
              be = shift_in_ge_band(be, acc[fm][fn][v], te, dmin);
              bg = shift_in_ge_band(bg, acc[fm][fn][v], tg, dmin);
              bl = shift_in_ge_band(bl, acc[fm][fn][v], tl, dmin);
            }
            if (__ballot(dmin < band) != 0 && !(same_tile && abase > bbase)) {
              uint32_t hits = 0;
#pragma unroll
              for (int v = 15; v >= 0; --v) {
                const float p = acc[fm][fn][v];
                hits = shift_in_sign(hits, fminf(fabsf(p - te), fminf(fabsf(p - tg), fabsf(p - tl))) - band);
              }
              close[fm] |= (hits & valid_marks(abase, bbase, nra, nrb, same_tile && abase == bbase, l31, hi)) << 16 * fn;
            }
          }
          uint32_t nan = 0;
#pragma unroll
          for (int v = 15; v >= 0; --v) nan = 2 * nan + (acc[fm][fn][v] != acc[fm][fn][v] ? 1u : 0u);
          col[0][fn] = spread_col_bits(be, hi, false, l31);
          col[1][fn] = spread_col_bits(bg, hi, false, l31);
          col[2][fn] = spread_col_bits(~(bl | nan) & 0xFFFFu, hi, false, l31);
#pragma unroll
          for (int m = 0; m < 3; ++m)
            if (hi == 0) pieces(m, true)[bbase + l31][abase >> 5] = col[m][fn];
        }
#pragma unroll
        for (int m = 0; m < 3; ++m) store_row_bits(col[m][0], col[m][1], hi, l31, abase, wn * G::WTN, pieces(m, false));
      }
      const int np = list_pairs(close, kWavePairs, wm * G::WTM, wn * G::WTN, pairs);
      if (el == 0) cnt[w] = np;
      __builtin_amdgcn_s_waitcnt(0xC07F);
      raw_barrier();
      const int mine = cnt[el & 7];
      // (so does a row without a bound, see gram_screen_kernel)
      back = __ballot(el < G::NWAVES && mine > kWavePairs) != 0 || !(rho < __builtin_inff());
      int pre[G::NWAVES + 1];
      pre[0] = 0;
#pragma unroll
      for (int i = 0; i < G::NWAVES; ++i) pre[i + 1] = back ? 0 : pre[i] + __builtin_amdgcn_readlane(mine, i);
      const int all = pre[G::NWAVES];
      // bf16 cosines, four pairs a wave at a time (see gram_screen_kernel)
      const float tie = static_cast<float>(2 * sa.d + 64) * 0x1p-24f;
      const uint32_t* lists = reinterpret_cast<const uint32_t*>(lds + kListOff);
      const int32_t* tk = tokens(buf);
      constexpr int NP = 4;
      for (int i0 = w * NP; i0 < all; i0 += G::NWAVES * NP) {
        const uint16_t *pa[NP], *pb[NP];
        float s[NP];
        const int it = min(i0 + (el & (NP - 1)), all - 1);
        int at = it;
#pragma unroll
        for (int q = 1; q < G::NWAVES; ++q)
          if (it >= pre[q]) at = q * kWavePairs + it - pre[q];
        const uint32_t pr = lists[at];
        const int ta = tk[pr >> 8], tb = tk[kTile + (pr & 255)];
        const float ia = sa.inv_norm[ta], ib = sa.inv_norm[tb];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          pa[u] = sa.x + static_cast<size_t>(__builtin_amdgcn_readlane(ta, u)) * sa.d;
          pb[u] = sa.x + static_cast<size_t>(__builtin_amdgcn_readlane(tb, u)) * sa.d;
          s[u] = 0.f;
        }
        for (int cc = el * 8; cc < sa.d; cc += 512) {
          Pack16 a[NP], b[NP];
#pragma unroll
          for (int u = 0; u < NP; ++u) {
            a[u].u4 = *reinterpret_cast<const uint4*>(pa[u] + cc);
            b[u].u4 = *reinterpret_cast<const uint4*>(pb[u] + cc);
          }
#pragma unroll
          for (int u = 0; u < NP; ++u)
#pragma unroll
            for (int q = 0; q < 8; ++q) s[u] = fmaf(bf16_to_f32(a[u].h[q]), bf16_to_f32(b[u].h[q]), s[u]);
        }
        float dot = 0.f;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          const float t = wave_sum_dpp(s[u]);
          dot = (el & (NP - 1)) == u ? t : dot;
        }
        const float cs = dot * ia * ib;
        if (el < NP && i0 + el < all) {
          const int r = pr >> 8, q = pr & 255;
          if (fabsf(cs - sa.h) < tie || fabsf(cs - hp.S1) < tie || fabsf(cs - hp.S2) < tie) cnt[8] = 1;
          const bool is[3] = {cs >= sa.h, cs > hp.S1, cs < hp.S2};
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            uint32_t* dw = &pieces(m, false)[r][q >> 5];
            uint32_t* tw = same_tile ? &pieces(m, false)[q][r >> 5] : &pieces(m, true)[q][r >> 5];
            if (is[m]) {
              atomicOr(dw, 1u << (q & 31));
              atomicOr(tw, 1u << (r & 31));
            } else {
              atomicAnd(dw, ~(1u << (q & 31)));
              atomicAnd(tw, ~(1u << (r & 31)));
            }
          }
        }
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);
      raw_barrier();
    }
    back = back || __builtin_amdgcn_readfirstlane(cnt[8]) != 0;
    if (compute) {
      strike = !back ? 0 : strike ? min(2 * strike, 8) : 1;
      direct = max(strike - 1, 0);
    }
    if (back) {
      if (opaque_tid() == 0) sa.list[atomicAdd(sa.list_count, 1)] = tile;
    } else {
      // (a skipped tile's pieces are stale and masked out: no pair is undecided)
      const int i = opaque_tid(), rl = i >> 1, ww = 2 * (i & 1);
#pragma unroll
      for (int mir = 0; mir < 2; ++mir) {
        if (mir && same_tile) break;
        const int row = (mir ? c.tj : c.ti) * kTile + rl, wd = 4 * (mir ? c.ti : c.tj) + ww;
        int edges = store_hist_words(hp, bitmask, base, row, wd, c.n, c.W, &pieces(0, mir)[rl][2 * ww],
                                          &pieces(1, mir)[rl][2 * ww], &pieces(2, mir)[rl][2 * ww]);
        edges += __shfl_xor(edges, 1, 64);
        if (edges && (i & 1) == 0) atomicAdd(&deg[c.lo + row], edges);
      }
    }
    if (!more) break;
    // every wave's reads of the tile's LDS state are done before the next
    // tile overwrites it
    __builtin_amdgcn_s_waitcnt(0xC07F);
    raw_barrier();
    tile = ntile;
    c = cn;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    nu += __shfl_xor(static_cast<long long>(nu), o, 64);
    nd += __shfl_xor(static_cast<long long>(nd), o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    if (nu) atomicAdd(&hp.stats[0], nu);
    if (nd) atomicAdd(&hp.stats[1], nd);
  }
  if (threadIdx.x == 0) {
    if (tiles) atomicAdd(&hp.stats[2], tiles);
    if (skipped) atomicAdd(&hp.stats[3], skipped);
  }
}

// float32 similarity, with or without history (Sec. 5.1 step 2): 64 x 64
// tiles on float32 MFMA (GemmF32; the products and sums are float32, as with
// vector FMA, at twice its unpacked rate and without its LDS reads per
// multiply-add).  Bound by the MFMA rate for large buckets, by a tile's
// latency for small ones; three blocks a CU overlap one tile's loads and
// epilogue with another's products.  On 8 buckets of about 750 rows
// (d = 512): vector FMA tiles (4 x 4 a thread) 89 us, these 32 us; on 4 of 128
// rows (d = 256): 23 and 10 us.
// HIST: each pair takes weight 1 or 0 where the previous block decided it and
// its cosine elsewhere (every tile computed); HOUT: the record words are
// written beside the adjacency words.
template <bool HIST, bool HIN, bool HOUT>
__global__ __launch_bounds__(GemmF32::THREADS, kGramF32Blocks) void gram_kernel_f32(
    const float* __restrict__ X, int d, const int32_t* __restrict__ perm_token,
    const int32_t* __restrict__ offsets, int E, const float* __restrict__ inv_norm, HistParams hp,
    const int32_t* __restrict__ tile_off, const long long* __restrict__ bm_off,
    const int* __restrict__ err, uint64_t* __restrict__ bitmask, int32_t* __restrict__ deg) {
  using G = GemmF32;
  static_assert(G::BM == kTileF32 && G::BN == kTileF32 && G::FM == 1 && G::FN == 1, "float32 similarity tile");
  constexpr int NM = HOUT ? 3 : 1;
  // one LDS array: the operand ring; the inverse norms of the tile's rows and
  // columns; the predicates' words, direct and transposed; the previous
  // classes of the tile's rows
  constexpr int kInvOff = G::LDS_BYTES, kDOff = kInvOff + 2 * kTileF32 * 4, kTOff = kDOff + NM * kTileF32 * 8;
  constexpr int kRbOff = kTOff + NM * kTileF32 * 8;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kRbOff + (HIN ? 2 * kTileF32 * 8 : 0)];
  float* inv = reinterpret_cast<float*>(lds + kInvOff);
  uint64_t* dw = reinterpret_cast<uint64_t*>(lds + kDOff);
  uint64_t* tw = reinterpret_cast<uint64_t*>(lds + kTOff);
  uint64_t* rbw = reinterpret_cast<uint64_t*>(lds + kRbOff);
  if (*err) return;
  const int tid = threadIdx.x, lane = tid & 63, w = G::wave();
  const int arow = G::wave_m(w) * 32, brow = G::wave_n(w) * 32;
  const int l31 = lane & 31, hi = lane >> 5;
  const int total = tile_off[E];
  for (int tile = xcd_virtual_block(); tile < total; tile += gridDim.x) {
    const TileCoord c = decode_tile(tile, tile_off, offsets, E);
    const int32_t* pt = perm_token + c.lo;
    const long long bmo = bm_off[c.e];
    uint32_t poff[G::LP], qoff[G::LQ];
#pragma unroll
    for (int j = 0; j < G::LP; ++j)
      poff[j] = static_cast<uint32_t>(pt[min(c.ti * kTileF32 + G::load_row(j), c.n - 1)]) * 2u * d;
#pragma unroll
    for (int j = 0; j < G::LQ; ++j)
      qoff[j] = static_cast<uint32_t>(pt[min(c.tj * kTileF32 + G::load_row(G::LP + j) - G::BM, c.n - 1)]) * 2u * d;
    if (tid < 2 * kTileF32) {
      const int r = (tid < kTileF32 ? c.ti * kTileF32 : (c.tj - 1) * kTileF32) + tid;
      inv[tid] = inv_norm[pt[min(r, c.n - 1)]];
    } else if (HIN && tid < 3 * kTileF32) {
      // previous classes: tile-row rows, word tj
      const int rl = tid - 2 * kTileF32, a = c.ti * kTileF32 + rl;
      rbw[rl] = a < c.n ? hp.rb_hi[bmo + static_cast<long long>(a) * c.W + c.tj] : 0ull;
      rbw[kTileF32 + rl] = a < c.n ? hp.rb_lo[bmo + static_cast<long long>(a) * c.W + c.tj] : 0ull;
    }
    typename G::Acc acc;
    G::zero(acc);
    G::run(reinterpret_cast<const uint16_t*>(X), poff, reinterpret_cast<const uint16_t*>(X), qoff, 2 * d,
           c.n - c.ti * kTileF32, c.n - c.tj * kTileF32, lds, acc);   // its barriers publish inv and rbw
    const int bl = brow + l31, b = c.tj * kTileF32 + bl;
    const float ib = inv[kTileF32 + bl];
    uint32_t pr[16];
    unsigned nu = 0, nd = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int al = arow + 8 * (v >> 2) + (v & 3) + 4 * hi, a = c.ti * kTileF32 + al;
      const bool pair = a < c.n && b < c.n && a != b;
      float wv = acc[0][0][v] * inv[al] * ib;
      if constexpr (HIST) {
        bool hb = false, lb = false;
        if constexpr (HIN) {
          hb = (rbw[al] >> bl) & 1ull;
          lb = (rbw[kTileF32 + al] >> bl) & 1ull;
        }
        wv = hb ? 1.0f : (lb ? 0.0f : wv);
        if (pair && a < b) {
          if (hb || lb) ++nd;
          else ++nu;
        }
      }
      pr[v] = pair && wv >= hp.h ? 1u : 0u;
      if constexpr (HOUT) pr[v] |= (pair && wv > hp.S1 ? 2u : 0u) | (pair && wv < hp.S2 ? 4u : 0u);
    }
    if constexpr (HIST) {
      if (nu) atomicAdd(&hp.stats[0], static_cast<unsigned long long>(nu));
      if (nd) atomicAdd(&hp.stats[1], static_cast<unsigned long long>(nd));
      if (tid == 0) atomicAdd(&hp.stats[2], 1ull);
    }
    block_bits<NM>(pr, reinterpret_cast<uint32_t*>(dw), reinterpret_cast<uint32_t*>(tw), arow, brow);
    __syncthreads();
    if (tid < 2 * kTileF32) {
      const bool mirror = tid >= kTileF32;
      const int rl = mirror ? tid - kTileF32 : tid;
      const int cnt = __popcll(mirror ? tw[rl] : dw[rl]);
      const int r = (mirror ? c.tj : c.ti) * kTileF32 + rl;
      if (cnt && r < c.n && (!mirror || c.ti != c.tj)) atomicAdd(&deg[c.lo + r], cnt);
    }
    write_tile_words(c, dw, tw, bitmask, bmo);
    if constexpr (HOUT) {
      write_tile_words(c, dw + kTileF32, tw + kTileF32, hp.out_hi, bmo);
      write_tile_words(c, dw + 2 * kTileF32, tw + 2 * kTileF32, hp.out_lo, bmo);
    }
    __syncthreads();
  }
}

// Decides position p if its neighbours allow it; returns true when p is
// still undecided afterwards (uniform over the GW-lane group that visits p,
// GW = 16 or 64, aligned inside the wave).  The group walks the adjacency
// row 4*GW words at a time (four word loads in flight per lane), gathers the
// state and degree of up to 8 neighbours at a time before testing them, and
// stops after the first batch of words that shows a kept neighbour (p is
// absorbed) or an undecided neighbour of higher priority (p stays
// undecided for a later round).  The grid
// rounds use plain loads (FRESH = false): a state written by another XCD in
// the same launch may be seen late, which only delays a decision (states
// change once, from undecided to final).  The single-workgroup finishing
// pass, which relies on seeing the previous iteration's decisions, reads
// the states with coherent atomic loads (FRESH = true).
// U words a lane of a GW-lane group, from word b0 of a row on: looks up the
// state and degree of every neighbour they hold and notes a kept
// neighbour or an undecided one of higher priority.
template <bool FRESH, int GW, int U>
__device__ __forceinline__ void greedy_scan(int b0, int p, int dp, int lo, int n, int W,
                                            const uint64_t* __restrict__ row, const int32_t* __restrict__ deg,
                                            const int32_t* state, bool& kept_nb, bool& blocked) {
  const int gl = threadIdx.x & (GW - 1);
  const int wd0 = b0 + gl;
  uint64_t wv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) wv[u] = wd0 + GW * u < W ? row[wd0 + GW * u] : 0ull;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    uint64_t bits = wv[u];
    const int cbase = (wd0 + GW * u) * 64;
    while (bits) {
      int q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        q[i] = -1;
        if (bits) {
          const int b = __ffsll(static_cast<long long>(bits)) - 1;
          bits &= bits - 1;
          if (cbase + b < n) q[i] = lo + cbase + b;   // no bit lies past the bucket
        }
      }
      int st[8], dq[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        st[i] = q[i] >= 0 ? (FRESH ? load_flag(&state[q[i]]) : state[q[i]]) : kStateAbsorbed;
        dq[i] = q[i] >= 0 ? deg[q[i]] : 0;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (st[i] == kStateKept) kept_nb = true;
        else if (st[i] == kStateUndecided && (dq[i] > dp || (dq[i] == dp && q[i] < p))) blocked = true;
      }
    }
  }
}

// A kept position q offers itself to every neighbour, as soon as it is
// kept: it marks the neighbour absorbed (a neighbour of a kept position is
// never kept, so it ends absorbed) and keeps in claim[b] the largest key
// (degree << 32 | ~position), i.e. the neighbour's first kept neighbour in
// walk order.  The maximum does not depend on when each kept position makes
// its claims, so every pass that keeps a position claims for it at once and
// no pass over the kept rows is needed afterwards.  The GW lanes of q's group
// share the row, four words a lane at a time.
template <int GW>
__device__ __forceinline__ void greedy_claim(int q, int dq, int lo, int n, int W,
                                             const uint64_t* __restrict__ row, int32_t* state,
                                             unsigned long long* __restrict__ claim) {
  const int gl = threadIdx.x & (GW - 1);
  const unsigned long long key = (static_cast<unsigned long long>(dq) << 32) |
                                 static_cast<unsigned int>(~static_cast<unsigned int>(q));
  constexpr int U = 4;
  for (int wd0 = gl; wd0 < W; wd0 += U * GW) {
    uint64_t wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) wv[u] = wd0 + GW * u < W ? row[wd0 + GW * u] : 0ull;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint64_t bits = wv[u];
      const int cbase = (wd0 + GW * u) * 64;
      while (bits) {
        const int b = __ffsll(static_cast<long long>(bits)) - 1;
        bits &= bits - 1;
        if (cbase + b < n) {
          store_flag(&state[lo + cbase + b], kStateAbsorbed);
          atomicMax(&claim[lo + cbase + b], key);
        }
      }
    }
  }
}

// Visit of undecided position p by a GW-lane group: kept if no neighbour is
// kept or undecided with higher priority (it then claims its neighbours at
// once), absorbed if a neighbour is kept, else left undecided (returns
// true).  The row is scanned in chunks and the
// group stops at its first kept or blocking neighbour: the first chunk has
// 4 words a lane (most rows stop there), later ones 8, so that a row
// scanned to its end (every neighbour of lower priority) takes half the
// dependent round trips.
template <bool FRESH, int GW>
__device__ __forceinline__ bool greedy_visit(int p, int lo, int n, int W,
                                             const uint64_t* __restrict__ row,
                                             const int32_t* __restrict__ deg, int32_t* state,
                                             unsigned long long* __restrict__ claim) {
  const int lane = threadIdx.x & 63;
  const int gl = lane & (GW - 1);
  const int gshift = lane & ~(GW - 1);
  const uint64_t gmask = GW == 64 ? ~0ull : ((1ull << (GW & 63)) - 1);
  const int dp = deg[p];
  bool kept_nb = false, blocked = false;
  greedy_scan<FRESH, GW, 4>(0, p, dp, lo, n, W, row, deg, state, kept_nb, blocked);
  for (int b0 = 4 * GW; b0 < W && !((__ballot(kept_nb || blocked) >> gshift) & gmask); b0 += 8 * GW)
    greedy_scan<FRESH, GW, 8>(b0, p, dp, lo, n, W, row, deg, state, kept_nb, blocked);
  const bool any_kept = ((__ballot(kept_nb) >> gshift) & gmask) != 0;
  const bool any_blocked = ((__ballot(blocked) >> gshift) & gmask) != 0;
  if (any_kept) {
    if (gl == 0) store_flag(&state[p], kStateAbsorbed);
    return false;
  }
  if (!any_blocked) {
    if (gl == 0) store_flag(&state[p], kStateKept);
    greedy_claim<GW>(p, dp, lo, n, W, row, state, claim);
    return false;
  }
  return true;
}

constexpr int kVisitLanes = 16;                       // lanes per position in the grid passes
constexpr int kVisitPerBlock = 256 / kVisitLanes;     // positions per 256-thread block

// Bucket offsets of the current call in LDS (E <= 64).
__device__ __forceinline__ void load_offsets(const int32_t* __restrict__ offsets, int E, int* soff) {
  if (threadIdx.x <= static_cast<unsigned>(E)) soff[threadIdx.x] = offsets[threadIdx.x];
  __syncthreads();
}

// The first round over all positions (16 lanes each); also publishes the
// degrees.  On a union of cliques it decides every position: the first
// member of each clique in walk order is kept and claims the others.
__global__ __launch_bounds__(256) void greedy_round_kernel(
    const int32_t* __restrict__ offsets, int E, const long long* __restrict__ bm_off,
    const int* __restrict__ err, const uint64_t* __restrict__ bitmask,
    const int32_t* __restrict__ deg, int32_t* state, unsigned long long* __restrict__ claim,
    int32_t* __restrict__ degree_out) {
  __shared__ int soff[kMaxExperts + 1];
  if (*err) return;
  load_offsets(offsets, E, soff);
  const int p = blockIdx.x * kVisitPerBlock + (threadIdx.x / kVisitLanes);
  const int gl = threadIdx.x & (kVisitLanes - 1);
  if (p >= soff[E]) return;
  if (degree_out && gl == 0) degree_out[p] = deg[p];
  // every state starts undecided and is written in this round only by p's
  // own visit or as absorbed by a kept neighbour's claims; p's visit can
  // then only find it absorbed again or leave it, so it is not read
  const int e = bucket_of(soff, E, p);
  const int lo = soff[e], n = soff[e + 1] - lo, W = (n + 63) / 64;
  greedy_visit<false, kVisitLanes>(p, lo, n, W, bitmask + bm_off[e] + static_cast<long long>(p - lo) * W, deg,
                                   state, claim);
}

// The round after the grid rounds: a persistent grid, 16 lanes per
// position, that passes over every position (each group reads the states of
// 16 consecutive positions with one load; decided ones cost nothing more)
// and revisits a blocked one a bounded number of times, reading
// the states coherently, so a dependency chain of length L resolves in
// about L visits inside one launch instead of L launches (graphs whose
// chains the grid rounds leave unfinished).  left[0] records that a
// position is still undecided after it, for the finishing pass.
__global__ __launch_bounds__(256) void greedy_more_kernel(
    const int32_t* __restrict__ offsets, int E, const long long* __restrict__ bm_off,
    const int* __restrict__ err, const uint64_t* __restrict__ bitmask,
    const int32_t* __restrict__ deg, int32_t* state, unsigned long long* __restrict__ claim,
    int* __restrict__ left) {
  __shared__ int soff[kMaxExperts + 1];
  if (*err) return;
  load_offsets(offsets, E, soff);
  const int gl = threadIdx.x & (kVisitLanes - 1);
  const int gshift = threadIdx.x & 63 & ~(kVisitLanes - 1);
  const int S = soff[E];
  // a group reads the states of kVisitLanes consecutive positions with one
  // load and visits the undecided ones among them (most are decided by now)
  for (int base = (blockIdx.x * kVisitPerBlock + static_cast<int>(threadIdx.x) / kVisitLanes) * kVisitLanes;
       base < S; base += gridDim.x * kVisitPerBlock * kVisitLanes) {
    const int pq = base + gl;
    const bool und = pq < S && load_flag(&state[pq]) == kStateUndecided;
    uint32_t m = static_cast<uint32_t>((__ballot(und) >> gshift) & ((1ull << kVisitLanes) - 1));
    // every pass visits each position the group still has: one of them may wait
    // for another (visited to the end one after the other, such a position spent
    // all its passes first: 8192 tokens with one mixture of two groups in twenty,
    // threshold 0.45: 70 us, now 12)
    for (int pass = 0; m && pass < kGreedyPasses; ++pass) {
      if (pass > 0) __builtin_amdgcn_s_sleep(32);
      for (uint32_t todo = m; todo; todo &= todo - 1) {
        const int p = base + __ffs(todo) - 1;
        const int e = bucket_of(soff, E, p);
        const int lo = soff[e], n = soff[e + 1] - lo, W = (n + 63) / 64;
        const uint64_t* row = bitmask + bm_off[e] + static_cast<long long>(p - lo) * W;
        if (!greedy_visit<true, kVisitLanes>(p, lo, n, W, row, deg, state, claim)) m &= ~(todo & (0u - todo));
      }
    }
    if (m && gl == 0) store_flag(&left[0], 1);
  }
}

// One workgroup per bucket decides what the grid rounds left.  The
// undecided positions are gathered into a list in LDS (a coalesced pass over
// the bucket's states); at most kFinishRounds rounds then visit only the
// listed positions, 16 lanes each (64 at a time), keeping those still
// undecided for the next round (a round decides at least the
// highest-priority undecided position; on clustered data one or two rounds
// decide all).  What is left after them (dependency chains, such as a path
// of similar tokens) is sorted by priority (degree descending, position
// ascending; a bitonic sort in LDS) and visited once each in that order by
// one wave: every higher-priority neighbour of a position is decided by its
// turn, so each visit decides its position, and the work is bounded by one
// visit per position instead of one per position and round.  A bucket with
// more undecided positions than the list holds first runs rounds over all
// its positions until the rest fits the list.
constexpr int kFinishList = 16384;
constexpr int kFinishRounds = 16;

// By the 1024 threads of a block; every thread returns from it.
template <int LIST>
__device__ __forceinline__ void greedy_finish_bucket(int lo, int n, const uint64_t* __restrict__ rows,
                                                     const int32_t* __restrict__ deg, int32_t* state,
                                                     unsigned long long* __restrict__ claim, int (*list)[LIST],
                                                     int* cnt) {
  if (n == 0) return;
  const int W = (n + 63) / 64;
  const int tid = threadIdx.x;
  int m;
  for (;;) {
    if (tid < 2) cnt[tid] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += 1024) {
      if (load_flag(&state[lo + i]) == kStateUndecided) {
        const int slot = atomicAdd(&cnt[0], 1);
        if (slot < LIST) list[0][slot] = i;
      }
    }
    __syncthreads();
    m = cnt[0];
    if (m == 0) return;
    if (m <= LIST) break;
    // more than the list holds: a round over all positions, one wave each
    const int wv = tid >> 6;
    for (int pl = wv; pl < n; pl += 16) {
      const int p = lo + pl;
      if (load_flag(&state[p]) != kStateUndecided) continue;
      greedy_visit<true, 64>(p, lo, n, W, rows + static_cast<long long>(pl) * W, deg, state, claim);
    }
    __syncthreads();
  }
  int cur = 0;
  {
    const int grp = tid / kVisitLanes;
    constexpr int kGroups = 1024 / kVisitLanes;
    for (int it = 0; it < kFinishRounds && m > 0; ++it) {
      for (int idx = grp; idx < m; idx += kGroups) {
        const int pl = list[cur][idx];
        greedy_visit<true, kVisitLanes>(lo + pl, lo, n, W, rows + static_cast<long long>(pl) * W, deg, state,
                                        claim);
      }
      if (tid == 0) cnt[cur ^ 1] = 0;
      __syncthreads();
      for (int idx = tid; idx < m; idx += 1024) {
        const int pl = list[cur][idx];
        if (load_flag(&state[lo + pl]) == kStateUndecided) list[cur ^ 1][atomicAdd(&cnt[cur ^ 1], 1)] = pl;
      }
      __syncthreads();
      cur ^= 1;
      m = cnt[cur];
      __syncthreads();
    }
  }
  if (m == 0) return;
  // sort the m positions left by priority: list[cur] positions, list[cur ^ 1]
  // their degrees; padded to a power of two with entries after every real one
  int* pos = list[cur];
  int* dg = list[cur ^ 1];
  int P = 1;
  while (P < m) P <<= 1;
  for (int i = tid; i < P; i += 1024) {
    if (i < m) dg[i] = deg[lo + pos[i]];
    else { pos[i] = 0x7fffffff; dg[i] = -1; }
  }
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = tid; i < P; i += 1024) {
        const int l = i ^ j;
        if (l > i) {
          // a_first: entry i comes before entry l (higher degree, then lower position)
          const bool a_first = dg[i] > dg[l] || (dg[i] == dg[l] && pos[i] < pos[l]);
          const bool up = (i & k) == 0;
          if (up != a_first) {
            const int tp = pos[i], td = dg[i];
            pos[i] = pos[l];
            dg[i] = dg[l];
            pos[l] = tp;
            dg[l] = td;
          }
        }
      }
      __syncthreads();
    }
  }
  if (tid < 64) {
    for (int idx = 0; idx < m; ++idx) {
      const int pl = pos[idx];
      greedy_visit<true, 64>(lo + pl, lo, n, W, rows + static_cast<long long>(pl) * W, deg, state, claim);
    }
  }
}

__global__ __launch_bounds__(1024) void greedy_finish_kernel(
    const int32_t* __restrict__ offsets, int E, const long long* __restrict__ bm_off,
    const int* __restrict__ err, const uint64_t* __restrict__ bitmask,
    const int32_t* __restrict__ deg, int32_t* state, unsigned long long* __restrict__ claim,
    const int* __restrict__ left) {
  __shared__ int list[2][kFinishList];
  __shared__ int cnt[2];
  if (*err) return;
  if (load_flag(&left[0]) == 0) return;   // the grid rounds decided every position
  const int e = blockIdx.x;
  greedy_finish_bucket<kFinishList>(offsets[e], offsets[e + 1] - offsets[e], bitmask + bm_off[e], deg, state, claim,
                                    list, cnt);
}

// Small calls (at most kSmallSlots positions): the positions that the first round
// leaves undecided, and the representative rows by the block that finishes last.
// Four launches of 4 to 5 us each, whose work is mostly a few reads, become one
// (512 positions: 19.5 -> 7.9 us; the last block takes about 1 us per 1024
// positions, so that 16384 would take 22.6 us).
// One block decides a bucket of up to kSmallAlone positions as greedy_finish_kernel
// does.  The undecided positions of a larger one are dealt to several blocks, 16
// lanes each, that revisit them as greedy_more_kernel does, and the last block
// finishes what they leave: a graph of thousands of undecided positions with full
// rows (a bucket of 4096 tokens with cosines around h) takes one block 140 to 490
// us, these 26 to 84, the four launches 48 to 110; 4096 tokens in groups of 8, with
// nothing left undecided: 8, 9 and 18 us.
// Blocks hand their decisions over through agent-scope atomics: every state and
// claim written here is one, every wave waits for its own (the barrier alone does
// not) before its block counts itself done (release), so the last block (acquire)
// reads them all.
constexpr int kSmallSlots = 4096;
constexpr int kSmallAlone = 1024;
constexpr int kSmallList = 4096;   // undecided positions of a bucket listed at a time

// Blocks of greedy_small_kernel for a bucket of n positions.
__host__ __device__ __forceinline__ int small_share(int n) { return n <= kSmallAlone ? 1 : (n + 255) / 256; }

// Share b of B of a bucket's undecided positions (every B-th position, whatever
// the other blocks have decided by then): each 16-lane group revisits its own a
// bounded number of times; cnt[1] records that one stayed undecided.
__device__ __forceinline__ void greedy_share_bucket(int b, int B, int lo, int n, const uint64_t* __restrict__ rows,
                                                    const int32_t* __restrict__ deg, int32_t* state,
                                                    unsigned long long* __restrict__ claim, int* list, int* cnt) {
  const int W = (n + 63) / 64, tid = threadIdx.x;
  if (tid < 2) cnt[tid] = 0;
  __syncthreads();
  for (int i = b + B * tid; i < n; i += B * 1024)
    if (load_flag(&state[lo + i]) == kStateUndecided) list[atomicAdd(&cnt[0], 1)] = i;
  __syncthreads();
  const int m = cnt[0];
  constexpr int kGroups = 1024 / kVisitLanes;
  bool still = false;
  for (int pass = 0; pass < kGreedyPasses; ++pass) {
    if (pass > 0) __builtin_amdgcn_s_sleep(32);
    still = false;
    for (int idx = tid / kVisitLanes; idx < m; idx += kGroups) {
      const int pl = list[idx];
      if (load_flag(&state[lo + pl]) == kStateUndecided)
        still |= greedy_visit<true, kVisitLanes>(lo + pl, lo, n, W, rows + static_cast<long long>(pl) * W, deg, state, claim);
    }
    if (!still) break;
  }
  if (still) cnt[1] = 1;
}

// SHARED: block y of bucket x has share y of it; blocks past the bucket's do nothing.
template <bool SHARED>
__global__ __launch_bounds__(1024) void greedy_small_kernel(
    const int32_t* __restrict__ offsets, int E, const long long* __restrict__ bm_off, const int* __restrict__ err,
    const uint64_t* __restrict__ bitmask, const int32_t* __restrict__ deg, int32_t* state,
    unsigned long long* __restrict__ claim, int* __restrict__ done, const int32_t* __restrict__ perm_token,
    int32_t* __restrict__ rep_of_pos, int32_t* __restrict__ rep_row, int32_t* __restrict__ rep_token,
    int32_t* __restrict__ rep_offsets) {
  __shared__ __attribute__((aligned(16))) int list[2][kSmallList];
  __shared__ int cnt[2], wsum[kSmallSlots / 64 / 64];
  __shared__ bool last, rest;
  const int failed = *err;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  auto finish = [&](int e) {
    greedy_finish_bucket<kSmallList>(offsets[e], offsets[e + 1] - offsets[e], bitmask + bm_off[e], deg, state, claim,
                                     list, cnt);
  };
  const int e = blockIdx.x;
  bool shared = false;   // block-uniform
  int blocks = E;        // that count themselves done
  if constexpr (SHARED) {
    // (a bucket larger than max_bucket, a layout error, has the whole grid column)
    auto of_bucket = [&](int n) { return min(small_share(n), static_cast<int>(gridDim.y)); };
    const int n = offsets[e + 1] - offsets[e], of = of_bucket(n);
    if (static_cast<int>(blockIdx.y) >= of) return;
    if (wv == 0) {
      int all;
      wave_prefix_dpp(lane < E ? of_bucket(offsets[lane + 1] - offsets[lane]) : 0, all);
      blocks = all;
    }
    shared = of > 1 && !failed;
    if (shared)
      greedy_share_bucket(blockIdx.y, of, offsets[e], n, bitmask + bm_off[e], deg, state, claim, &list[0][0], cnt);
  }
  if (!shared && !failed) finish(e);
  // this wave's states and claims are done; the counting thread's release writes
  // the L2 back for the whole block (a fence by every wave, which repeats that,
  // costs a 512-token layer 3 us: 62.0 against 58.9)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    // low half: blocks done; high half: those that left a position undecided
    int mine = 1;
    if (shared && cnt[1]) mine = 0x10001;
    const int sum = mine + __hip_atomic_fetch_add(done, mine, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    last = (sum & 0xFFFF) == blocks;
    rest = (sum >> 16) != 0;
  }
  __syncthreads();
  if (!last) return;
  if (SHARED && rest) {   // block-uniform
    for (int i = 0; i < E; ++i) {
      finish(i);
      __syncthreads();
    }
  }
  // representatives (bit p % 64 of word p / 64) and their exclusive counts
  uint64_t* mask = reinterpret_cast<uint64_t*>(&list[0][0]);
  int* pre = &list[1][0];
  static_assert(kSmallSlots / 64 * 8 <= static_cast<int>(sizeof(list[0])) &&
                    kSmallSlots / 64 + 1 <= kSmallList && kSmallSlots / 64 <= 1024, "masks in LDS");
  const int S = offsets[E];
  constexpr int PER = kSmallSlots / 1024;
  int q[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int p = i * 1024 + tid;
    q[i] = p;
    if (p < S && !failed && load_flag(&state[p]) == kStateAbsorbed) {
      const unsigned long long c = __hip_atomic_load(&claim[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      q[i] = static_cast<int>(~static_cast<unsigned int>(c & 0xffffffffull));
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int p = i * 1024 + tid;
    if (i * 1024 >= S) break;   // (block-uniform)
    const uint64_t m = __ballot(p < S && q[i] == p);
    if (lane == 0) mask[p >> 6] = m;
    if (p < S) rep_of_pos[p] = q[i];
  }
  __syncthreads();
  // exclusive prefix of the words' counts, a word a thread (one wave)
  const int words = (S + 63) / 64;
  int own = 0, incl = 0;
  if (tid < kSmallSlots / 64) {
    own = tid < words ? __popcll(mask[tid]) : 0;
    incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o, 64);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wv] = incl;
  }
  __syncthreads();
  if (tid < kSmallSlots / 64) {
    int before = 0;
    for (int i = 0; i < wv; ++i) before += wsum[i];
    pre[tid] = before + incl - own;
    if (tid == kSmallSlots / 64 - 1) pre[kSmallSlots / 64] = before + incl;
  }
  __syncthreads();
  auto rank = [&](int p) {   // representatives before position p (p <= S)
    const int w = p >> 6;
    return w >= words ? pre[kSmallSlots / 64] : pre[w] + __popcll(mask[w] & ((1ull << (p & 63)) - 1));
  };
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int p = i * 1024 + tid;
    if (i * 1024 >= S) break;
    if (p < S) {
      const int row = rank(q[i]);
      rep_row[p] = row;
      if (q[i] == p) rep_token[row] = perm_token[p];
    }
  }
  if (tid <= E) rep_offsets[tid] = rank(offsets[tid]);
}

// Representative rows, in two passes over 1024-position blocks.
// rep_local_kernel: the duplicate->representative map, then the rank of each
// representative inside its block (wave ballots + LDS prefix of the 16 wave
// counts) and the block's count.
__global__ __launch_bounds__(1024) void rep_local_kernel(const int32_t* __restrict__ offsets, int E,
                                                        const int* __restrict__ err,
                                                        const int32_t* __restrict__ state,
                                                        const unsigned long long* __restrict__ claim,
                                                        int32_t* __restrict__ rep_of_pos,
                                                        int32_t* __restrict__ local,
                                                        int32_t* __restrict__ bsum, int slot_cap) {
  __shared__ int wcnt[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int p = blockIdx.x * 1024 + tid;
  // state and claim of this position are read together with the slot count
  // (positions past the arrays' T*k entries read nothing)
  const bool mine = p < slot_cap;
  const int st = mine ? state[p] : 0;
  const unsigned long long cl = mine ? claim[p] : 0ull;
  const int failed = *err;
  const int S = offsets[E];
  const int base = blockIdx.x * 1024;
  if (base >= S) return;
  // rep_of_pos: absorbed -> claimed representative; otherwise itself (also
  // after a layout error, when nothing was decided)
  bool f = false;
  if (p < S) {
    const bool absorbed = !failed && st == kStateAbsorbed;
    rep_of_pos[p] = absorbed ? static_cast<int>(~static_cast<unsigned int>(cl & 0xffffffffull)) : p;
    f = !absorbed;
  }
  const uint64_t bal = __ballot(f);
  if (lane == 0) wcnt[wv] = __popcll(bal);
  __syncthreads();
  int before = 0, total = 0;
  for (int i = 0; i < 16; ++i) {
    const int v = wcnt[i];
    before += i < wv ? v : 0;
    total += v;
  }
  if (p < S) local[p] = before + __popcll(bal & lanemask_lt());
  if (tid == 0) bsum[blockIdx.x] = total;
}

// rep_finalize_kernel: every block prefixes the block counts in LDS, then
// writes rep_token, rep_row (through the representative's own block prefix)
// and, in block 0, rep_offsets.
__global__ __launch_bounds__(1024) void rep_finalize_kernel(
    const int32_t* __restrict__ offsets, int E, const int32_t* __restrict__ rep_of_pos,
    const int32_t* __restrict__ perm_token, const int32_t* __restrict__ local,
    const int32_t* __restrict__ bsum, int32_t* __restrict__ rep_row, int32_t* __restrict__ rep_token,
    int32_t* __restrict__ rep_offsets, int slot_cap) {
  extern __shared__ int bpre[];   // one entry per block of the grid, plus one
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // this thread's position: its representative and token are read before
  // the block-count scan (positions past the arrays' T*k entries read
  // nothing; those past the kept slot count are read and not used)
  const int p = blockIdx.x * 1024 + tid;
  const bool mine = p < slot_cap;
  const int q_pre = mine ? rep_of_pos[p] : 0;
  const int tok_pre = mine ? perm_token[p] : 0;
  const int S = offsets[E];
  const int nb = (S + 1023) / 1024;
  // exclusive prefix of bsum[0..nb) into bpre, 1024 at a time
  int carry = 0;
  for (int c0 = 0; c0 < nb; c0 += 1024) {
    const int i = c0 + tid;
    const int v = i < nb ? bsum[i] : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o, 64);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int wb = 0, tot = 0;
    for (int k = 0; k < 16; ++k) {
      wb += k < wv ? wsum[k] : 0;
      tot += wsum[k];
    }
    if (i < nb) bpre[i] = carry + wb + incl - v;
    carry += tot;
    __syncthreads();
  }
  if (tid == 0) bpre[nb] = carry;
  __syncthreads();
  if (p < S) {
    const int q = q_pre;
    const int row = bpre[q >> 10] + local[q];
    rep_row[p] = row;
    if (q == p) rep_token[row] = tok_pre;
  }
  if (blockIdx.x == 0 && tid <= E) {
    const int o = offsets[tid];
    rep_offsets[tid] = o < S ? bpre[o >> 10] + local[o] : bpre[nb];
  }
}

__global__ __launch_bounds__(256) void gather_kernel(const uint8_t* __restrict__ x, size_t row_bytes,
                                                     const int32_t* __restrict__ rep_offsets, int E,
                                                     const int32_t* __restrict__ rep_token,
                                                     uint8_t* __restrict__ x_rep) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rep_offsets[E]) return;
  const uint4* src = reinterpret_cast<const uint4*>(x + static_cast<size_t>(rep_token[r]) * row_bytes);
  uint4* dst = reinterpret_cast<uint4*>(x_rep + static_cast<size_t>(r) * row_bytes);
  for (size_t i = lane; i < row_bytes / 16; i += 64) dst[i] = src[i];
}

struct CondenseWs {
  float* inv_norm;
  int32_t* tile_off;
  long long* bm_off;
  int* err;
  int32_t* deg;
  int32_t* state;
  unsigned long long* claim;
  int32_t* local;
  int32_t* bsum;
  uint64_t* bitmask;
  long long cap_words;
  // history calls only: the previous block's classes in this block's
  // layout, and the pair / tile counters when the caller passes none
  uint64_t* rb_hi = nullptr;
  uint64_t* rb_lo = nullptr;
  unsigned long long* stats = nullptr;
  int* left;                    // a position stayed undecided after the greedy rounds (small calls: the
                                // finished blocks of greedy_small_kernel)
  int32_t* colinfo = nullptr;   // previous positions of every slot of every position
  int* queue = nullptr;         // tile queues of the similarity kernel
  // the fp8 screen (calls whose shape allows it): fp8 rows
  // (and a zero row), their error bounds, the tiles left to the bf16 pass and
  // their count
  uint8_t* x8 = nullptr;
  float4* rowq = nullptr;
  int* list = nullptr;
  int* list_count = nullptr;
};

// Process-wide switch of the fp8 similarity screen (on by default).
std::atomic<int> g_gram_screen{1};

// Shapes whose similarity call may take the fp8 screen: long rows, and buckets
// of MFMA-bound size on average (T k / E >= 512).  Below that the extra pass
// over x and the looks at single pairs cost more than the products they save:
// at d = 1024, 16 buckets of about 1100 tokens, bf16 products 34 us, screen 64
// (its band, 0.067, covers same-group cosines of 0.999 against h = 0.95).
bool gram_screen_shape(int T, int d, int E, int k) {
  return d >= 2048 && static_cast<long long>(T) * k >= 512ll * E &&
         static_cast<long long>(T + 1) * ((d + 127) / 128 * 128) <= 0xFFFF0000ll;
}
// A threshold the screen can decide most unrelated pairs against: their cosines
// spread about 0 by 1 / sqrt(d), their estimates are off by up to about 0.06 (the
// band of rows that fill their range evenly), and a wave's part of a tile holds
// 8192 of them, of which 64 may fall inside the band.  Nearer to 0 every tile goes
// back and the bf16 kernel alone is the faster one.  History, 16 buckets of 2048,
// d = 2048 (line at 0.126), S2 = 0.10 / 0.12 / 0.13 / 0.2: with the screen 416 /
// 350 / 219 / 195 us, without 248 each; 8 of 1024, d = 4096 (0.107), S2 = 0.10 /
// 0.11: 293 / 133 and 132.  Plain, 4 of 2048, d = 4096, h = 0.10 / 0.12: 223 / 85
// and 105.
bool screen_room(int d, float t) { return fabsf(t) >= 0.06f + 3.f / sqrtf(static_cast<float>(d)); }
// Pitch of the fp8 rows: whole 128-value stages.
int screen_pitch(int d) { return (d + 127) / 128 * 128; }

// Upper bound of the number of similarity tiles: sum over buckets of
// t_e (t_e + 1) / 2 with t_e = ceil(n_e / kTile) <= ceil(max_bucket / kTile)
// and sum t_e <= S / kTile + E.
long long gram_tile_bound(long long S, int E, int max_bucket) {
  const long long tmax = (static_cast<long long>(max_bucket) + kTile - 1) / kTile;
  return (S / kTile + E) * (tmax + 1) / 2 + 1;
}

CondenseWs carve_condense(Carver& c, int T, int d, int E, int k, int max_bucket, bool history = false) {
  CondenseWs w;
  const long long S = static_cast<long long>(T) * k;
  w.inv_norm = c.take<float>(T);
  w.tile_off = c.take<int32_t>(E + 1);
  w.bm_off = c.take<long long>(E + 1);
  w.err = c.take<int>(1);
  w.deg = c.take<int32_t>(S);
  w.state = c.take<int32_t>(S);
  w.claim = c.take<unsigned long long>(S);
  w.local = c.take<int32_t>(S);
  w.bsum = c.take<int32_t>((S + 1023) / 1024 + 1);
  w.left = c.take<int>(1);
  w.cap_words = S * ((static_cast<long long>(max_bucket) + 63) / 64);
  w.bitmask = c.take<uint64_t>(static_cast<size_t>(w.cap_words));
  if (history) {
    w.rb_hi = c.take<uint64_t>(static_cast<size_t>(w.cap_words));
    w.rb_lo = c.take<uint64_t>(static_cast<size_t>(w.cap_words));
    w.stats = c.take<unsigned long long>(4);
    w.colinfo = c.take<int32_t>(static_cast<size_t>(S) * k);
    w.queue = c.take<int>(kTileQueues);
  }
  if (gram_screen_shape(T, d, E, k)) {
    w.x8 = c.take<uint8_t>(static_cast<size_t>(T + 1) * screen_pitch(d));
    w.rowq = c.take<float4>(T);
    w.list_count = c.take<int>(1);
    w.list = c.take<int>(static_cast<size_t>(gram_tile_bound(S, E, max_bucket)));
  }
  return w;
}

// Arguments of a call with historical similarity.
struct HistCall {
  const int32_t* slot_pos;   // this block's slot positions (for its record)
  const void* in;            // previous block's record or nullptr
  void* out;                 // this block's record or nullptr
  float S1, S2;
  unsigned long long* stats;
};

}  // namespace
}  // namespace luffy

using namespace luffy;

namespace {

int condense_check(const char* fn, const void* x, int T, int d, int dtype, const int32_t* perm_token,
                   const int32_t* offsets, int E, int k, int max_bucket, float threshold, const int32_t* rep_of_pos,
                   const int32_t* rep_row, const int32_t* rep_offsets, const int32_t* rep_token) {
  if (!x || !perm_token || !offsets || !rep_of_pos || !rep_row || !rep_offsets || !rep_token)
    return fail(LUFFY_E_INVALID, "%s: null pointer argument", fn);
  if (T <= 0 || d <= 0 || E <= 0 || max_bucket < 0)
    return fail(LUFFY_E_INVALID, "%s: T=%d d=%d E=%d max_bucket=%d", fn, T, d, E, max_bucket);
  if (k != 1 && k != 2) return fail(LUFFY_E_INVALID, "%s: k=%d must be 1 or 2", fn, k);
  if (dtype != LUFFY_F32 && dtype != LUFFY_BF16) return fail(LUFFY_E_INVALID, "%s: unknown dtype %d", fn, dtype);
  if (threshold != threshold) return fail(LUFFY_E_INVALID, "%s: threshold is NaN", fn);
  if (E > kMaxExperts) return fail(LUFFY_E_UNSUPPORTED, "%s: E=%d > %d", fn, E, kMaxExperts);
  if (d % 64 != 0) return fail(LUFFY_E_UNSUPPORTED, "%s: d=%d not a multiple of 64", fn, d);
  if (d > 32768) return fail(LUFFY_E_UNSUPPORTED, "%s: d=%d > 32768", fn, d);
  if (static_cast<long long>(T) * d * elem_bytes(dtype) > 0xFFFF0000ll)
    return fail(LUFFY_E_UNSUPPORTED, "%s: x exceeds 4 GiB - 64 KiB", fn);
  if (static_cast<long long>(T) * k > (1ll << 24)) return fail(LUFFY_E_UNSUPPORTED, "%s: T*k > 2^24", fn);
  return LUFFY_OK;
}

// Every launch of a condense call; hc is null for a call without history.
void condense_enqueue(const void* x, int T, int d, int dtype, const int32_t* perm_token, const int32_t* offsets,
                      int E, int k, int max_bucket, float threshold, int32_t* rep_of_pos, int32_t* rep_row,
                      int32_t* rep_offsets, int32_t* rep_token, void* x_rep, int32_t* degree,
                      const float* inv_norm, const CondenseWs& ws, const HistCall* hc, hipStream_t s) {
  const int S = T * k;
  const bool bf16 = dtype == LUFFY_BF16;
  unsigned long long* stats = hc ? (hc->stats ? hc->stats : ws.stats) : nullptr;
  // norms from the caller when given (the gate pass already read x)
  const float* inv_norm_use = inv_norm ? inv_norm : ws.inv_norm;
  // the fp8 similarity screen: its rows are written by the norm pass
  // (a history call without a record out keeps the bf16 kernel)
  const bool screen = (!hc || (hc->out && screen_room(d, hc->S1) && screen_room(d, hc->S2))) && bf16 && ws.x8 &&
                      threshold > 0.f && screen_room(d, threshold) &&
                      g_gram_screen.load(std::memory_order_relaxed);
  const int norm_blocks = screen ? std::max((S + 255) / 256, (T + 4) / 4)
                                 : inv_norm ? std::max(1, (S + 255) / 256) : (T + 3) / 4;
  const int dp = screen_pitch(d), da = !screen ? 0 : hc ? dp : screen_first_values(d, dp, threshold);
  {
    const int tile = bf16 ? kTile : kTileF32;
#define LUFFY_NORM_ARGS x, T, d, inv_norm ? const_cast<float*>(inv_norm) : ws.inv_norm, S, ws.deg, ws.state, ws.claim, \
                        offsets, E, max_bucket, tile, ws.cap_words, ws.tile_off, ws.bm_off, ws.err, stats, ws.queue,   \
                        ws.left, ws.list_count, dp, da, ws.x8, ws.rowq
    if (bf16 && screen) {
      if (inv_norm) launch("norm", norm_kernel<true, false, true>, norm_blocks, 256, 0, s, LUFFY_NORM_ARGS);
      else launch("norm", norm_kernel<true, true, true>, norm_blocks, 256, 0, s, LUFFY_NORM_ARGS);
    } else if (bf16) {
      if (inv_norm) launch("norm", norm_kernel<true, false>, norm_blocks, 256, 0, s, LUFFY_NORM_ARGS);
      else launch("norm", norm_kernel<true, true>, norm_blocks, 256, 0, s, LUFFY_NORM_ARGS);
    } else {
      if (inv_norm) launch("norm", norm_kernel<false, false>, norm_blocks, 256, 0, s, LUFFY_NORM_ARGS);
      else launch("norm", norm_kernel<false, true>, norm_blocks, 256, 0, s, LUFFY_NORM_ARGS);
    }
#undef LUFFY_NORM_ARGS
  }
  if (!hc) {
    const uint16_t* xb = static_cast<const uint16_t*>(x);
    if (screen) {
      // the screen over every tile, then the bf16 pass over the tiles it left
      const ScreenArgs sa{ws.x8, ws.rowq, xb, inv_norm_use, d, dp, da, T, threshold, ws.list, ws.list_count};
      launch("gram", gram_screen_kernel, persistent_grid(), GramGemm::THREADS, 0, s, sa, perm_token, offsets, E,
             ws.tile_off, ws.bm_off, ws.err, ws.bitmask, ws.deg);
      launch("gram_recheck", gram_kernel_bf16<true>, persistent_grid(), GramGemm::THREADS, 0, s, xb, d, perm_token,
             offsets, E, inv_norm_use, threshold, ws.tile_off, ws.bm_off, ws.err, ws.bitmask, ws.deg, ws.list,
             ws.list_count);
    } else if (bf16)
      launch("gram", gram_kernel_bf16<false>, persistent_grid(), GramGemm::THREADS, 0, s, xb, d, perm_token, offsets,
             E, inv_norm_use, threshold, ws.tile_off, ws.bm_off, ws.err, ws.bitmask, ws.deg, nullptr, nullptr);
    else {
      HistParams hp{};
      hp.h = threshold;
      launch("gram", gram_kernel_f32<false, false, false>, kGramF32Blocks * persistent_grid(), GemmF32::THREADS, 0, s,
             static_cast<const float*>(x), d, perm_token, offsets, E, inv_norm_use, hp, ws.tile_off, ws.bm_off, ws.err,
             ws.bitmask, ws.deg);
    }
  } else {
    Carver cin(const_cast<void*>(hc->in)), cout(hc->out);
    const HistRec rin = carve_hist(cin, T, E, k, max_bucket);
    const HistRec rout = carve_hist(cout, T, E, k, max_bucket);
    if (hc->in) {
      const int blocks = (S + kGatherRows - 1) / kGatherRows + E;
      const int cblocks = std::max(1, std::min(1024, (S + 255) / 256));
      // the rows in LDS where they fit a CU: 8 rows a block by four waves while
      // four blocks fit, 8 by 16 waves while two do, else 4 by 16 waves (buckets
      // of up to 38,848 tokens at k = 2 then still give a CU two blocks, whose
      // row copies and lookups overlap); larger buckets read the rows from memory
      const size_t row_lds = hist_row_bytes(max_bucket);
      const int row_bytes = static_cast<int>(row_lds);
      const bool eight = 8 * k * row_lds <= kGatherLdsMax;
      const int grows = eight ? 8 : 4, gthreads = eight && 8 * k * row_lds <= kGatherLdsMax / 2 ? 256 : 1024;
      const size_t glds = grows * k * row_lds;
      const int gblocks = (S + grows - 1) / grows + E;
#define LUFFY_GATHER(K_, G_) launch("hist_gather", hist_gather_lds_kernel<K_, G_>, gblocks, gthreads, glds, s, offsets, E, \
                                    ws.bm_off, ws.err, rin, row_bytes, ws.colinfo, ws.rb_hi, ws.rb_lo)
      if (k == 1)
        launch("hist_cols", hist_cols_kernel<1>, cblocks, 256, 0, s, offsets, E, perm_token, ws.err, rin, T,
               max_bucket, ws.colinfo);
      else
        launch("hist_cols", hist_cols_kernel<2>, cblocks, 256, 0, s, offsets, E, perm_token, ws.err, rin, T,
               max_bucket, ws.colinfo);
      if (glds <= kGatherLdsMax) {
        if (k == 1) { if (eight) LUFFY_GATHER(1, 8); else LUFFY_GATHER(1, 4); }
        else { if (eight) LUFFY_GATHER(2, 8); else LUFFY_GATHER(2, 4); }
#undef LUFFY_GATHER
      } else if (k == 1) {
        launch("hist_gather", hist_gather_kernel<1>, blocks, 256, 0, s, offsets, E, ws.bm_off, ws.err, rin,
               ws.colinfo, ws.rb_hi, ws.rb_lo);
      } else {
        launch("hist_gather", hist_gather_kernel<2>, blocks, 256, 0, s, offsets, E, ws.bm_off, ws.err, rin,
               ws.colinfo, ws.rb_hi, ws.rb_lo);
      }
    }
    if (hc->out)
      launch("hist_header", hist_header_kernel, std::max(1, std::min(1024, (S + 255) / 256)), 256, 0, s,
             hc->slot_pos, T, k, offsets, E, max_bucket, ws.bm_off, ws.err, rout);
    HistParams hp;
    hp.h = threshold;
    hp.S1 = hc->S1;
    hp.S2 = hc->S2;
    hp.out_hi = hc->out ? rout.hi : nullptr;
    hp.out_lo = hc->out ? rout.lo : nullptr;
    hp.rb_hi = hc->in ? ws.rb_hi : nullptr;
    hp.rb_lo = hc->in ? ws.rb_lo : nullptr;
    hp.stats = stats;
    hp.queue = ws.queue;
    const bool hin = hc->in != nullptr, hout = hc->out != nullptr;
#define LUFFY_GH_ARGS d, perm_token, offsets, E, inv_norm_use, hp, ws.tile_off, ws.bm_off, ws.err, ws.bitmask, ws.deg
#define LUFFY_GHB_ARGS LUFFY_GH_ARGS, ws.list, ws.list_count
    if (bf16) {
      const uint16_t* xb = static_cast<const uint16_t*>(x);
      const int g = persistent_grid();
      const int th = GramGemm::THREADS;
      if (screen) {
        const ScreenArgs sa{ws.x8, ws.rowq, xb, inv_norm_use, d, dp, da, T, threshold, ws.list, ws.list_count};
        launch("gram", gram_hist_screen_kernel, g, th, 0, s, sa, hp, perm_token, offsets, E, ws.tile_off, ws.bm_off,
               ws.err, ws.bitmask, ws.deg);
        if (hin) launch("gram_recheck", gram_hist_kernel_bf16<true, true, true>, g, th, 0, s, xb, LUFFY_GHB_ARGS);
        else launch("gram_recheck", gram_hist_kernel_bf16<false, true, true>, g, th, 0, s, xb, LUFFY_GHB_ARGS);
      } else if (hin && hout) launch("gram", gram_hist_kernel_bf16<true, true>, g, th, 0, s, xb, LUFFY_GHB_ARGS);
      else if (hin) launch("gram", gram_hist_kernel_bf16<true, false>, g, th, 0, s, xb, LUFFY_GHB_ARGS);
      else if (hout) launch("gram", gram_hist_kernel_bf16<false, true>, g, th, 0, s, xb, LUFFY_GHB_ARGS);
      else launch("gram", gram_hist_kernel_bf16<false, false>, g, th, 0, s, xb, LUFFY_GHB_ARGS);
    } else {
      const float* xf = static_cast<const float*>(x);
      const int g = kGramF32Blocks * persistent_grid();
      if (hin && hout) launch("gram", gram_kernel_f32<true, true, true>, g, 256, 0, s, xf, LUFFY_GH_ARGS);
      else if (hin) launch("gram", gram_kernel_f32<true, true, false>, g, 256, 0, s, xf, LUFFY_GH_ARGS);
      else if (hout) launch("gram", gram_kernel_f32<true, false, true>, g, 256, 0, s, xf, LUFFY_GH_ARGS);
      else launch("gram", gram_kernel_f32<true, false, false>, g, 256, 0, s, xf, LUFFY_GH_ARGS);
    }
#undef LUFFY_GHB_ARGS
#undef LUFFY_GH_ARGS
  }
  const int wave_blocks = (S + 3) / 4;
  const int visit_blocks = (S + kVisitPerBlock - 1) / kVisitPerBlock;
  launch("greedy_round", greedy_round_kernel, visit_blocks, 256, 0, s, offsets, E, ws.bm_off, ws.err, ws.bitmask,
         ws.deg, ws.state, ws.claim, degree);
  if (S <= kSmallSlots) {   // see greedy_small_kernel
#define LUFFY_SMALL_ARGS offsets, E, ws.bm_off, ws.err, ws.bitmask, ws.deg, ws.state, ws.claim, ws.left, perm_token, \
                         rep_of_pos, rep_row, rep_token, rep_offsets
    const int share = small_share(std::min(S, max_bucket));
    if (share == 1) launch("greedy_finish", greedy_small_kernel<false>, E, 1024, 0, s, LUFFY_SMALL_ARGS);
    else launch("greedy_finish", greedy_small_kernel<true>, dim3(E, share), 1024, 0, s, LUFFY_SMALL_ARGS);
#undef LUFFY_SMALL_ARGS
  } else {
    launch("greedy_more", greedy_more_kernel, std::min(visit_blocks, persistent_grid()), 256, 0, s, offsets, E,
           ws.bm_off, ws.err, ws.bitmask, ws.deg, ws.state, ws.claim, ws.left);
    launch("greedy_finish", greedy_finish_kernel, E, 1024, 0, s, offsets, E, ws.bm_off, ws.err, ws.bitmask, ws.deg,
           ws.state, ws.claim, ws.left);
    const int pos_blocks = (S + 1023) / 1024;
    launch("rep_local", rep_local_kernel, pos_blocks, 1024, 0, s, offsets, E, ws.err, ws.state, ws.claim, rep_of_pos,
           ws.local, ws.bsum, S);
    launch("rep_finalize", rep_finalize_kernel, pos_blocks, 1024, (pos_blocks + 1) * sizeof(int), s, offsets, E,
           rep_of_pos, perm_token, ws.local, ws.bsum, rep_row, rep_token, rep_offsets, S);
  }
  if (x_rep) {
    launch("gather", gather_kernel, wave_blocks, 256, 0, s, static_cast<const uint8_t*>(x),
           static_cast<size_t>(d) * elem_bytes(dtype), rep_offsets, E, rep_token, static_cast<uint8_t*>(x_rep));
  }
}

}  // namespace

extern "C" size_t luffy_condense_workspace_size(int T, int d, int E, int k, int max_bucket) {
  if (T <= 0 || E <= 0 || k <= 0 || max_bucket < 0) return 0;
  Carver c(nullptr);
  carve_condense(c, T, d, E, k, max_bucket);
  return c.size();
}

extern "C" int luffy_condense(const void* x, int T, int d, int dtype,
                              const int32_t* perm_token, const int32_t* offsets,
                              int E, int k, int max_bucket, float threshold,
                              int32_t* rep_of_pos, int32_t* rep_row,
                              int32_t* rep_offsets, int32_t* rep_token,
                              void* x_rep, int32_t* degree, const float* inv_norm,
                              void* workspace, size_t workspace_bytes, void* stream) {
  const int st = condense_check("luffy_condense", x, T, d, dtype, perm_token, offsets, E, k, max_bucket, threshold,
                                rep_of_pos, rep_row, rep_offsets, rep_token);
  if (st != LUFFY_OK) return st;
  const size_t need = luffy_condense_workspace_size(T, d, E, k, max_bucket);
  if (workspace_bytes < need || !workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return fail(LUFFY_E_WORKSPACE, "luffy_condense: workspace needs %zu bytes, 256-aligned", need);
  Carver c(workspace);
  const CondenseWs ws = carve_condense(c, T, d, E, k, max_bucket);
  condense_enqueue(x, T, d, dtype, perm_token, offsets, E, k, max_bucket, threshold, rep_of_pos, rep_row,
                   rep_offsets, rep_token, x_rep, degree, inv_norm, ws, nullptr, static_cast<hipStream_t>(stream));
  return check_launch("luffy_condense");
}

extern "C" int luffy_set_similarity_screen(int on) { return g_gram_screen.exchange(on ? 1 : 0); }

extern "C" int luffy_similarity_screen_applies(int T, int d, int E, int k, int dtype) {
  return dtype == LUFFY_BF16 && T > 0 && E > 0 && k > 0 && gram_screen_shape(T, d, E, k) &&
         g_gram_screen.load(std::memory_order_relaxed);
}

extern "C" size_t luffy_history_size(int T, int E, int k, int max_bucket) {
  if (T <= 0 || E <= 0 || k <= 0 || max_bucket < 0) return 0;
  Carver c(nullptr);
  carve_hist(c, T, E, k, max_bucket);
  return c.size();
}

extern "C" size_t luffy_condense_history_workspace_size(int T, int d, int E, int k, int max_bucket) {
  if (T <= 0 || E <= 0 || k <= 0 || max_bucket < 0) return 0;
  Carver c(nullptr);
  carve_condense(c, T, d, E, k, max_bucket, true);
  return c.size();
}

extern "C" int luffy_condense_history(const void* x, int T, int d, int dtype,
                                      const int32_t* perm_token, const int32_t* offsets,
                                      const int32_t* slot_pos, int E, int k, int max_bucket,
                                      float threshold, const void* hist_in, void* hist_out,
                                      float S1, float S2,
                                      int32_t* rep_of_pos, int32_t* rep_row,
                                      int32_t* rep_offsets, int32_t* rep_token,
                                      void* x_rep, int32_t* degree, const float* inv_norm,
                                      unsigned long long* stats,
                                      void* workspace, size_t workspace_bytes, void* stream) {
  const char* fn = "luffy_condense_history";
  const int st = condense_check(fn, x, T, d, dtype, perm_token, offsets, E, k, max_bucket, threshold, rep_of_pos,
                                rep_row, rep_offsets, rep_token);
  if (st != LUFFY_OK) return st;
  if (hist_out && !slot_pos) return fail(LUFFY_E_INVALID, "%s: hist_out needs slot_pos", fn);
  if (S1 != S1 || S2 != S2) return fail(LUFFY_E_INVALID, "%s: S1 or S2 is NaN", fn);
  if (hist_in && hist_in == hist_out) return fail(LUFFY_E_INVALID, "%s: hist_in and hist_out alias", fn);
  if ((reinterpret_cast<uintptr_t>(hist_in) & 255u) || (reinterpret_cast<uintptr_t>(hist_out) & 255u))
    return fail(LUFFY_E_INVALID, "%s: records must be 256-byte aligned", fn);
  const size_t need = luffy_condense_history_workspace_size(T, d, E, k, max_bucket);
  if (workspace_bytes < need || !workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return fail(LUFFY_E_WORKSPACE, "%s: workspace needs %zu bytes, 256-aligned", fn, need);
  Carver c(workspace);
  const CondenseWs ws = carve_condense(c, T, d, E, k, max_bucket, true);
  HistCall hc{slot_pos, hist_in, hist_out, S1, S2, stats};
  condense_enqueue(x, T, d, dtype, perm_token, offsets, E, k, max_bucket, threshold, rep_of_pos, rep_row,
                   rep_offsets, rep_token, x_rep, degree, inv_norm, ws, &hc, static_cast<hipStream_t>(stream));
  return check_launch(fn);
}
