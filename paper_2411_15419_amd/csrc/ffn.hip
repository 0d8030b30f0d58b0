// luffy_expert_ffn: grouped FFN over the representatives of every expert,
//   H = act(X_rep W1_e^T)   (rounded to the element type)
//   Y = H W2_e^T
// Row counts per expert live on the device: the kernels are persistent (bf16:
// one block per CU, float32: three) and find their tiles from rep_offsets.
//
// bf16: MFMA tiles of 256 weight rows by 256 or 320 token rows.  The weight
// rows are the P operand and the token rows the Q operand, so each lane
// ends with groups of four consecutive output columns of one row and stores
// each as one 8-byte word.  The last row tile of an expert usually holds
// fewer rows; its waves skip the MFMAs of the missing rows.
// float32: 64 x 64 or 32 x 32 tiles of float32 MFMA.
#include <type_traits>

#include "gemm_core.h"
#include "luffy_common.h"

namespace luffy {
namespace {

// Activations of the float32 path: exact erf-GELU and SiLU from the device
// math library.
template <int ACT>
__device__ __forceinline__ float act_fn(float z) {
  if constexpr (ACT == LUFFY_ACT_GELU) {
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
  } else {
    return z / (1.0f + expf(-z));
  }
}

// Activations of the bf16 path, whose results are rounded to bf16 (relative
// step 2^-8): a dozen VALU operations instead of the library erf, which
// dominated the epilogue of the first product.
//   GELU: erf from Abramowitz & Stegun 7.1.26 (Hastings' rational
//   approximation), erf(u) = 1 - q(u), q(u) = t (a1 + t (a2 + ... + t a5))
//   e^{-u^2}, t = 1 / (1 + p u), u >= 0, |error| <= 1.5e-7.  With
//   u = |z| / sqrt(2): GELU(z) = z (1 - q/2) for z >= 0 and z q/2 for z < 0,
//   evaluated as |z| (1 - q) / 2 + z / 2.
//   SiLU: z / (1 + 2^{-z log2 e}).
// The hardware exp2 and reciprocal are accurate to about 1 ulp.
// Activation code of a plain product (no activation), used by the backward.
constexpr int kActNone = 2;

template <int ACT>
__device__ __forceinline__ float act_fast(float z) {
  if constexpr (ACT == kActNone) {
    return z;
  } else if constexpr (ACT == LUFFY_ACT_GELU) {
    // Hastings' erf(u) = 1 - t (a1 + a2 t + ... + a5 t^4) e^{-u^2},
    // t = 1 / (1 + p u), u = |z| / sqrt(2), with the a_i halved here so
    // that w = 1/2 - t e P(t) = erf(u) / 2.  Then z Phi(z) = |z| w + z / 2
    // for either sign of z (Phi(z) = 1/2 + sign(z) erf(u) / 2): 10 vector
    // operations and two transcendentals per element.
    constexpr float kPs = 0.3275911f * 0.70710678118654752f;   // p / sqrt(2)
    constexpr float kB1 = 0.5f * 0.254829592f, kB2 = 0.5f * -0.284496736f, kB3 = 0.5f * 1.421413741f;
    constexpr float kB4 = 0.5f * -1.453152027f, kB5 = 0.5f * 1.061405429f;
    constexpr float kHalfLog2e = -0.72134752044448170f;   // -log2(e) / 2
    const float a = fabsf(z);
    const float t = __builtin_amdgcn_rcpf(fmaf(kPs, a, 1.0f));
    const float pt = fmaf(t, fmaf(t, fmaf(t, fmaf(t, kB5, kB4), kB3), kB2), kB1);
    const float e = __builtin_amdgcn_exp2f(z * z * kHalfLog2e);   // e^{-u^2}
    const float w = fmaf(-(t * e), pt, 0.5f);
    return fmaf(a, w, 0.5f * z);
  } else {
    constexpr float kNegLog2e = -1.44269504088896341f;
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z * kNegLog2e));
  }
}

// Derivative of the activation, with the approximations of act_fast (the
// result is rounded to bf16): GELU'(z) = Phi(z) + z phi(z), Phi from the
// same Hastings erf (Phi(z) = 1 - q/2 for z >= 0, q/2 below), phi(z) =
// e^{-z^2/2} / sqrt(2 pi) from the same exp2; SiLU'(z) = s (1 + z (1 - s)).
template <int ACT>
__device__ __forceinline__ float act_grad(float z) {
  if constexpr (ACT == LUFFY_ACT_GELU) {
    constexpr float kP = 0.3275911f;
    constexpr float kA1 = 0.254829592f, kA2 = -0.284496736f, kA3 = 1.421413741f;
    constexpr float kA4 = -1.453152027f, kA5 = 1.061405429f;
    constexpr float kInvSqrt2 = 0.70710678118654752f, kInvSqrt2Pi = 0.39894228040143268f;
    constexpr float kHalfLog2e = -0.72134752044448170f;   // -log2(e) / 2
    const float u = fabsf(z) * kInvSqrt2;
    const float t = __builtin_amdgcn_rcpf(fmaf(kP, u, 1.0f));
    const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, kA5, kA4), kA3), kA2), kA1);
    const float e = __builtin_amdgcn_exp2f(z * z * kHalfLog2e);   // e^{-z^2/2}
    const float hq = 0.5f * poly * e;
    return (z >= 0.f ? 1.0f - hq : hq) + z * kInvSqrt2Pi * e;
  } else {
    constexpr float kNegLog2e = -1.44269504088896341f;
    const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z * kNegLog2e));
    return sg * (1.0f + z * (1.0f - sg));
  }
}

// Epilogue codes of the backward's dA product: multiply by act'(Z) read
// from a second buffer (dZ = dA * act'(Z)).
constexpr int kActDzGelu = 3, kActDzSilu = 4;
// Epilogue codes of the backward's Z product: store Z to the output and
// act(Z), taken on the rounded Z, to the second buffer.
constexpr int kActZaGelu = 5, kActZaSilu = 6;

// Tile shapes of the bf16 products: 256 output columns (weight rows, the P
// operand) by up to 256 token rows (FfnGemm), or by up to 320 token rows
// (FfnGemmWide).  A tile streams its 256 weight rows once per token tile, so
// an expert whose row count lies in (256, 320] (or (512, 640], ...) needs one
// weight pass fewer with the wide shape; every other expert keeps the
// narrow shape, whose main loop runs a few percent faster (fewer registers,
// smaller stages).  Both shapes share the block size, the LDS buffer and the
// split-K slots.
using FfnGemm = GemmRagged64;
using FfnGemmWide = GemmCore<256, 320, 4, 2, true, false>;
// An expert with at most 128 rows (one token tile of 128) streams its weight
// panels from HBM for little MFMA work, so its tiles are bound by how much
// of the stream one CU has in flight: the 256 x 128 shape takes a ring of
// three 64-wide stages in the same LDS (two in flight while one is
// multiplied, against one for the 256 x 256 shape).
using FfnGemmSmall = GemmCore<256, 128, 4, 2, true, false, 64, 3>;
// The backward's row products read the weights transposed: P K-major.
using FfnGemmT = GemmCore<256, 256, 4, 2, true, false, 64, 2, true, false>;
using FfnGemmWideT = GemmCore<256, 320, 4, 2, true, false, 64, 2, true, false>;
using FfnGemmSmallT = GemmCore<256, 128, 4, 2, true, false, 64, 3, true, false>;
static_assert(FfnGemm::BM == FfnGemmWide::BM && FfnGemm::THREADS == FfnGemmWide::THREADS, "shared tile map");
static_assert(FfnGemm::BM == FfnGemmSmall::BM && FfnGemm::THREADS == FfnGemmSmall::THREADS, "shared tile map");
constexpr int kFfnLds = FfnGemmWide::LDS_BYTES > FfnGemm::LDS_BYTES ? FfnGemmWide::LDS_BYTES : FfnGemm::LDS_BYTES;
static_assert(FfnGemmSmall::LDS_BYTES <= kFfnLds && FfnGemmSmallT::LDS_BYTES <= kFfnLds, "small shape's ring");
// tile shapes of the tile map
constexpr int kShapeNarrow = 0, kShapeWide = 1, kShapeSmall = 2;
// split-K partial tiles: one slot (the accumulators of a tile in register
// layout) per work item, at most kFfnMaxSlots (>= CUs) work items
constexpr int kFfnMaxSlots = 1536;
constexpr size_t kFfnSlotFloats = static_cast<size_t>(FfnGemm::BM) * FfnGemmWide::BN;
// split-K parts cut K at multiples of this (a multiple of both stage widths)
constexpr int kFfnKUnit = 64;
static_assert(kFfnKUnit % FfnGemm::BK == 0 && kFfnKUnit % FfnGemmWide::BK == 0, "K unit");
// Tail counters of the grouped products of one call (forward 2, backward 3).
constexpr int kFfnQueueSets = 3;

// Clears the tail counters of the call's products (a kernel, not a memset,
// so that the call can be captured in a graph).
__global__ __launch_bounds__(64) void ffn_queue_clear_kernel(int* __restrict__ queue, int n) {
  if (static_cast<int>(threadIdx.x) < n) queue[threadIdx.x] = 0;
}

// Tile map of the grouped GEMM (persistent kernels; rep_offsets held one
// expert per lane, E <= 64).  Expert e's rows are cut into tiles of rt_e
// rows (128 for an expert of at most 128 rows, else 256, or 320 where that
// takes fewer tiles); the last one is usually partial.  Tiles are numbered expert by expert; inside an expert,
// output-column tiles come in groups of 4 with the row tiles fastest inside
// a group, so the tiles that share a weight tile run side by side and ~32
// consecutive tiles (one XCD's share of a round, with the XCD-aware block
// numbering) span few weight and token rows.
struct FfnTiles {
  int elo, ehi, rt, mt, incl, NT, tiles;
  __device__ __forceinline__ FfnTiles(const int32_t* __restrict__ rep_offsets, int E, int N) {
    const int lane = threadIdx.x & 63;
    NT = (N + FfnGemm::BM - 1) / FfnGemm::BM;
    elo = ehi = mt = 0;
    rt = FfnGemm::BN;
    if (lane < E) {
      elo = rep_offsets[lane];
      ehi = rep_offsets[lane + 1];
      const int n = ehi - elo;
      constexpr int NB = FfnGemm::BN, WB = FfnGemmWide::BN, SB = FfnGemmSmall::BN;
      rt = n <= SB ? SB : ((n + WB - 1) / WB < (n + NB - 1) / NB ? WB : NB);
      mt = (n + rt - 1) / rt;
    }
    incl = mt * NT;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    tiles = __builtin_amdgcn_readfirstlane(__shfl(incl, 63, 64));
  }
  // Tile t -> expert e, first token row row0, row count, first output n0,
  // and its shape (kShape*).
  __device__ __forceinline__ void decode(int t, int E, int& e, int& row0, int& rows, int& n0, int& shape) const {
    const int lane = threadIdx.x & 63;
    e = __popcll(__ballot(lane < E && incl <= t));
    const int me = __shfl(mt, e, 64);
    const int excl = __shfl(incl, e, 64) - me * NT;
    const int r = t - excl;
    const int ng = (NT + 3) / 4;
    const int g = min(r / (4 * me), ng - 1);
    const int r2 = r - 4 * g * me;
    const int ms = r2 % me, nt = 4 * g + r2 / me;
    // shuffles return vector registers: made scalar again so that the
    // buffer resources built from them stay in scalar registers
    const int rte = __builtin_amdgcn_readfirstlane(__shfl(rt, e, 64));
    row0 = __builtin_amdgcn_readfirstlane(__shfl(elo, e, 64) + ms * rte);
    rows = __builtin_amdgcn_readfirstlane(min(rte, __shfl(ehi, e, 64) - row0));
    n0 = __builtin_amdgcn_readfirstlane(nt * FfnGemm::BM);
    shape = rte == FfnGemmWide::BN ? kShapeWide : (rte == FfnGemmSmall::BN ? kShapeSmall : kShapeNarrow);
  }
  // Split-K parts per tile (second product only).  Only a product with
  // fewer tiles than blocks splits (with more, every CU already has a tile
  // and the partial tiles' round trip costs more than the balance gains:
  // measured on 424 tiles of K = 8192).  It takes the split s in 2..4 (each
  // part at least 4 K-units, every part's partial tile within the slots)
  // with the fewest rounds times part length, ceil(tiles*s/grid)/s in units
  // of a whole tile; ties keep the smaller split.  The per-CU operand
  // stream, not HBM, bounds these products, so rounds of shorter parts on
  // more CUs win even when a round is not full: 140 tiles of K = 4096 take
  // 2 rounds of thirds instead of 2 rounds of halves.
  __device__ __forceinline__ int parts(int grid, int nk) const {
    if (tiles <= 0 || tiles >= grid) return 1;
    int best = 1;
    long long best_cost = 12ll * ((tiles + grid - 1) / grid);
    for (int sp = 2; sp <= 4; ++sp) {
      if (nk / sp < 4 || static_cast<long long>(tiles) * sp > kFfnMaxSlots) break;
      const long long cost = (12 / sp) * ((static_cast<long long>(tiles) * sp + grid - 1) / grid);
      if (cost < best_cost) {
        best_cost = cost;
        best = sp;
      }
    }
    return best;
  }
  // Split plan of the second product: tiles [0, full) run whole, the `tail`
  // tiles after them run as S parts each (items full + u, u < tail * S, are
  // part u % S of tile full + u / S; partial slot u).  With fewer tiles than
  // blocks every tile is a tail tile and S comes from parts().  With more,
  // the whole rounds stay whole and only the tiles left over for the last,
  // partial round are split, into the most parts (at most 4, at least 4
  // K-units each) that one and a half rounds of blocks take: their parts
  // then fill the CUs that finish their whole tiles first instead of
  // leaving them idle (376 tiles of K = 8192 on 256 CUs: the 120 left over
  // in thirds, second product + reduction 358 -> 345 us; halves 350,
  // quarters 346).
  __device__ __forceinline__ void split_plan(int grid, int nk, int& full, int& tail, int& S) const {
    if (tiles < grid) {
      full = 0;
      tail = tiles;
      S = parts(grid, nk);
      return;
    }
    full = tiles / grid * grid;
    tail = tiles - full;
    S = 1;
    for (int sp = 2; sp <= 4; ++sp)
      if (tail > 0 && 2 * tail * sp <= 3 * grid && nk / sp >= 4 && tail * sp <= kFfnMaxSlots) S = sp;
  }
};

// Multiplies with only the first nq of the wave's Q blocks (wave-uniform
// nq in 0..FN), so the MFMAs of token rows past a partial tile are skipped.
template <class G, int N>
__device__ __forceinline__ void run_nq(int nq, const uint16_t* pbase, const uint32_t (&poff)[G::LP],
                                       const uint16_t* qbase, const uint32_t (&qoff)[G::LQ], int K, int pvalid,
                                       int qvalid, uint8_t* lds, typename G::Acc& acc, int pld) {
  if constexpr (N == 0) {
    G::template run<0>(pbase, poff, qbase, qoff, K, pvalid, qvalid, lds, acc, pld);
  } else {
    if (nq >= N) G::template run<N>(pbase, poff, qbase, qoff, K, pvalid, qvalid, lds, acc, pld);
    else run_nq<G, N - 1>(nq, pbase, poff, qbase, qoff, K, pvalid, qvalid, lds, acc, pld);
  }
}

// bf16 words pk[g] (columns 8g + 4 hi .. + 3 of a 32-column block of one token
// row) of lanes l and l + 32: after one exchange the low lane stores columns
// 0..15 and the high lane 16..31, two 16-byte stores each (dst: the lane's
// first column).
__device__ __forceinline__ void store_pair_row(const uint32_t (&pk)[4][2], int hi, uint16_t* __restrict__ dst_row) {
  const uint32_t snd[4] = {hi ? pk[0][0] : pk[2][0], hi ? pk[0][1] : pk[2][1], hi ? pk[1][0] : pk[3][0],
                           hi ? pk[1][1] : pk[3][1]};
  uint32_t rcv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) rcv[i] = static_cast<uint32_t>(__shfl_xor(static_cast<int>(snd[i]), 32, 64));
  uint4* dst = reinterpret_cast<uint4*>(dst_row);
  if (hi == 0) {
    dst[0] = make_uint4(pk[0][0], pk[0][1], rcv[0], rcv[1]);
    dst[1] = make_uint4(pk[1][0], pk[1][1], rcv[2], rcv[3]);
  } else {
    dst[0] = make_uint4(rcv[0], rcv[1], pk[2][0], pk[2][1]);
    dst[1] = make_uint4(rcv[2], rcv[3], pk[3][0], pk[3][1]);
  }
}

// One output tile (or one K part of it) of shape G: rows row0.. of A
// (through row_index when given) times the weight rows n0.. of We over K
// range [k0, k1).  Stores bf16 (activation applied when FIRST), or, when
// slot is given, the float32 accumulators in register layout: float4 unit
// ((w*FM + fm)*FN + fn)*4 + g of lane l holds acc[fm][fn][4g..4g+3].
template <class G, int ACT, bool FIRST>
__device__ __forceinline__ void ffn_tile(const uint16_t* __restrict__ A, const int32_t* __restrict__ row_index,
                                         const uint16_t* __restrict__ We, int K, int N, int k0, int k1, int row0,
                                         int rows, int n0, uint16_t* __restrict__ out, float* __restrict__ slot,
                                         uint16_t* __restrict__ aux, uint8_t* lds) {
  static_assert(G::FN <= 5, "ragged dispatch instantiates FN + 1 main loops");
  constexpr bool ZA = ACT == kActZaGelu || ACT == kActZaSilu;
  const int tid = opaque_tid(), lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = G::wave_m(w), wn = G::wave_n(w);
  uint32_t poff[G::LP], qoff[G::LQ];
  // weights [N, K] row-major, or (G::PT) [K, N]: element (k, n) at k * N + n
  if constexpr (G::PT) {
    G::kmajor_offsets(poff, G::SLOTS_P, N, n0, N - n0);
  } else {
#pragma unroll
    for (int j = 0; j < G::LP; ++j) poff[j] = static_cast<uint32_t>(min(n0 + G::load_row(j), N - 1)) * K;
  }
#pragma unroll
  for (int j = 0; j < G::LQ; ++j) {
    const int m = row0 + min(G::load_row(G::LP + j) - G::BM, rows - 1);
    qoff[j] = static_cast<uint32_t>(row_index ? row_index[m] : m) * K;
  }
  const int nq = G::active_q(wn, rows);
  typename G::Acc acc;
  G::zero(acc);
  run_nq<G, G::FN>(__builtin_amdgcn_readfirstlane(nq), We + (G::PT ? static_cast<size_t>(k0) * N : k0), poff,
                   A + k0, qoff, k1 - k0, N - n0, rows, lds, acc, N);
  if constexpr (ACT != kActDzGelu && ACT != kActDzSilu) {
    if (!slot) {
      const int hi = lane >> 5;
#pragma unroll
      for (int fm = 0; fm < G::FM; ++fm) {
#pragma unroll
        for (int fn = 0; fn < G::FN; ++fn) {
          const int ml = G::q_row(wn, fn) + (lane & 31);
          const int nb = n0 + wm * G::WTM + 32 * fm;
          if (ml >= rows || nb >= N) continue;
          uint32_t pk[4][2];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            float z[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              z[q] = acc[fm][fn][4 * g + q];
              if constexpr (FIRST && !ZA) z[q] = act_fast<ACT>(z[q]);
            }
            pk[g][0] = pack_bf16x2(z[0], z[1]);
            pk[g][1] = pack_bf16x2(z[2], z[3]);
          }
          const size_t at = static_cast<size_t>(row0 + ml) * N + nb + 16 * hi;
          store_pair_row(pk, hi, out + at);
          if constexpr (ZA) {
            constexpr int A = ACT == kActZaGelu ? LUFFY_ACT_GELU : LUFFY_ACT_SILU;
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
              for (int q = 0; q < 2; ++q)
                pk[g][q] = pack_bf16x2(act_fast<A>(__uint_as_float(pk[g][q] << 16)),
                                       act_fast<A>(__uint_as_float(pk[g][q] & 0xFFFF0000u)));
            store_pair_row(pk, hi, aux + at);
          }
        }
      }
      return;
    }
  }
#pragma unroll
  for (int fm = 0; fm < G::FM; ++fm) {
#pragma unroll
    for (int fn = 0; fn < G::FN; ++fn) {
      const int ml = G::q_row(wn, fn) + (lane & 31);
      if (ml >= rows) continue;
      uint16_t* orow = out + static_cast<size_t>(row0 + ml) * N;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int nl = wm * G::WTM + 32 * fm + 8 * g + 4 * (lane >> 5);
        const int n = n0 + nl;
        if (n >= N) continue;
        if (slot) {
          // partial tiles keep the accumulator layout: 1 KB per store
          // instruction; the reduction maps it back to rows and columns
          const int u = ((w * G::FM + fm) * G::FN + fn) * 4 + g;
          *reinterpret_cast<float4*>(slot + u * 256 + lane * 4) =
              make_float4(acc[fm][fn][4 * g], acc[fm][fn][4 * g + 1], acc[fm][fn][4 * g + 2],
                          acc[fm][fn][4 * g + 3]);
          continue;
        }
        float z[4];
        if constexpr (ACT == kActDzGelu || ACT == kActDzSilu) {
          // dZ = dA * act'(Z): the four Z values of this store
          const uint2 zw = *reinterpret_cast<const uint2*>(aux + static_cast<size_t>(row0 + ml) * N + n);
          const float zz[4] = {__uint_as_float(zw.x << 16), __uint_as_float(zw.x & 0xFFFF0000u),
                               __uint_as_float(zw.y << 16), __uint_as_float(zw.y & 0xFFFF0000u)};
#pragma unroll
          for (int q = 0; q < 4; ++q)
            z[q] = acc[fm][fn][4 * g + q] * act_grad<ACT == kActDzGelu ? LUFFY_ACT_GELU : LUFFY_ACT_SILU>(zz[q]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            z[q] = acc[fm][fn][4 * g + q];
            if constexpr (FIRST && !ZA) z[q] = act_fast<ACT>(z[q]);
          }
        }
        *reinterpret_cast<uint2*>(orow + n) = make_uint2(pack_bf16x2(z[0], z[1]), pack_bf16x2(z[2], z[3]));
      }
    }
  }
}

// One product of the FFN for every tile of every expert (persistent).  The
// whole rounds of work items are dealt statically (serpentine, XCD-aware
// block order: consecutive items share weight and token rows in an XCD's
// L2); the items left over, the last ones in the order (the smallest
// experts' tiles), go one at a time through a counter (*tail, zero at
// launch) to the blocks that finish first.  The second product (FIRST =
// false) has few output columns (d); with few representatives it can have
// fewer tiles than CUs, and it then splits K (decided on the device from the
// actual tile count): parts store float32 partial tiles and
// ffn_split_reduce_kernel finishes them.
template <int ACT, bool FIRST, bool WT = false>
__global__ __launch_bounds__(FfnGemm::THREADS) void ffn_kernel_bf16(
    const uint16_t* __restrict__ A, const int32_t* __restrict__ row_index,
    const int32_t* __restrict__ rep_offsets, int E, int K, int N,
    const uint16_t* __restrict__ W, uint16_t* __restrict__ out, float* __restrict__ split_slots,
    uint16_t* __restrict__ aux, int* __restrict__ tail) {
  // one LDS array: the operand ring, then the block's current tail item (a
  // second LDS variable would cost the K loop its DMA overlap)
  __shared__ __attribute__((aligned(16))) uint8_t lds[kFfnLds + 16];
  int& item_s = *reinterpret_cast<int*>(lds + kFfnLds);
  const FfnTiles map(rep_offsets, E, N);
  const int nk = K / kFfnKUnit;
  int full = map.tiles, ntail = 0, S = 1;
  if (!FIRST) map.split_plan(gridDim.x, nk, full, ntail, S);
  const int total = full + ntail * S;
  // static rounds: whole tiles only when the tail is split (its parts go
  // to the blocks that finish first), else every whole round of items
  const int g = gridDim.x, rounds = (full > 0 && S > 1) ? full / g : total / g;
  const int vb = xcd_virtual_block();
  for (int round = 0;; ++round) {
    int tt;
    if (round < rounds) {
      tt = serpentine_item(round, vb);
    } else {
      if (rounds * g == total) break;   // no tail
      if (threadIdx.x == 0) item_s = rounds * g + atomicAdd(tail, 1);
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the item is in LDS
      raw_barrier();
      // read before the tile's barriers: thread 0 writes the next item only
      // after every thread has passed them
      tt = item_s;
      if (tt >= total) break;
    }
    // whole tile, or part `part` of S of a tail tile (partial slot u)
    const int u = tt - full;
    const int sp = u < 0 ? 1 : S;
    const int t = u < 0 ? tt : full + u / S, part = u < 0 ? 0 : u - (u / S) * S;
    int e, row0, rows, n0, shape;
    map.decode(t, E, e, row0, rows, n0, shape);
    const uint16_t* We = W + static_cast<size_t>(e) * N * K;
    // K range of this part, in whole 64-wide units
    const int k0 = (part * nk / sp) * kFfnKUnit, k1 = ((part + 1) * nk / sp) * kFfnKUnit;
    float* slot = sp > 1 ? split_slots + static_cast<size_t>(u) * kFfnSlotFloats : nullptr;
    using GN = std::conditional_t<WT, FfnGemmT, FfnGemm>;
    using GW = std::conditional_t<WT, FfnGemmWideT, FfnGemmWide>;
    using GS = std::conditional_t<WT, FfnGemmSmallT, FfnGemmSmall>;
    if (shape == kShapeWide)
      ffn_tile<GW, ACT, FIRST>(A, row_index, We, K, N, k0, k1, row0, rows, n0, out, slot, aux, lds);
    else if (shape == kShapeSmall)
      ffn_tile<GS, ACT, FIRST>(A, row_index, We, K, N, k0, k1, row0, rows, n0, out, slot, aux, lds);
    else
      ffn_tile<GN, ACT, FIRST>(A, row_index, We, K, N, k0, k1, row0, rows, n0, out, slot, aux, lds);
  }
}

// Sums the S split parts of unit q (= (w*FM + fm)*FN + fn) of one output
// tile of shape G, lane l, and stores bf16.  The float4 units g = 0..3 of
// lane l hold columns 8g..8g+3 (l < 32) or 8g+4..8g+7 (l >= 32) of a
// 32-column block of one token row; lanes l and l+32 share the row and swap
// halves so that each stores 16 consecutive bf16 (two 16-byte stores).
template <class G, int S>
__device__ __forceinline__ void reduce_unit(const float* __restrict__ slots, int q, int row0, int rows, int n0,
                                            int N, uint16_t* __restrict__ out) {
  const int l = threadIdx.x & 63, hi = l >> 5;
  const int fn = q % G::FN, fm = (q / G::FN) % G::FM, w = q / (G::FN * G::FM);
  const int ml = G::q_row(G::wave_n(w), fn) + (l & 31);
  const int nb = G::wave_m(w) * G::WTM + 32 * fm;   // first column of the 32-column block
  if (ml >= rows || n0 + nb >= N) return;            // same for lanes l and l+32
  const float* src = slots + static_cast<size_t>(q) * 4 * 256 + l * 4;
  // every part's four float4 units loaded before any is added (S is a
  // template constant, so no load waits behind a branch), then summed in
  // part order
  float4 u[S][4];
#pragma unroll
  for (int p = 0; p < S; ++p)
#pragma unroll
    for (int g = 0; g < 4; ++g) u[p][g] = *reinterpret_cast<const float4*>(src + p * kFfnSlotFloats + g * 256);
  float4 v[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    v[g] = u[0][g];
#pragma unroll
    for (int p = 1; p < S; ++p) {
      v[g].x += u[p][g].x; v[g].y += u[p][g].y; v[g].z += u[p][g].z; v[g].w += u[p][g].w;
    }
  }
  // lane l (< 32) holds columns 8g..8g+3, lane l+32 columns 8g+4..8g+7:
  // the low lane keeps columns 0..15, the high lane 16..31
  float4 send[2] = {hi ? v[0] : v[2], hi ? v[1] : v[3]};
  float4 recv[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    recv[i].x = __shfl_xor(send[i].x, 32, 64);
    recv[i].y = __shfl_xor(send[i].y, 32, 64);
    recv[i].z = __shfl_xor(send[i].z, 32, 64);
    recv[i].w = __shfl_xor(send[i].w, 32, 64);
  }
  const float4 c[4] = {hi ? recv[0] : v[0], hi ? v[2] : recv[0], hi ? recv[1] : v[1], hi ? v[3] : recv[1]};
  uint4* dst = reinterpret_cast<uint4*>(out + static_cast<size_t>(row0 + ml) * N + n0 + nb + 16 * hi);
  dst[0] = make_uint4(pack_bf16x2(c[0].x, c[0].y), pack_bf16x2(c[0].z, c[0].w), pack_bf16x2(c[1].x, c[1].y),
                      pack_bf16x2(c[1].z, c[1].w));
  dst[1] = make_uint4(pack_bf16x2(c[2].x, c[2].y), pack_bf16x2(c[2].z, c[2].w), pack_bf16x2(c[3].x, c[3].y),
                      pack_bf16x2(c[3].z, c[3].w));
}

// Sums the split parts of every split (tail) tile in part order and stores
// bf16.  Recomputes the same tile map and split plan, so it does nothing
// when the product was not split.  One thread per (w, fm, fn, lane) unit of a tile;
// a tile gets the block count of the wide shape (the narrow shape leaves
// its last blocks idle).
constexpr int kReduceUnits = FfnGemmWide::NWAVES * FfnGemmWide::FM * FfnGemmWide::FN * 64;
static_assert(kReduceUnits % 256 == 0 &&
                  FfnGemm::NWAVES * FfnGemm::FM * FfnGemm::FN * 64 <= kReduceUnits, "reduction blocks");

__global__ __launch_bounds__(256) void ffn_split_reduce_kernel(const int32_t* __restrict__ rep_offsets, int E,
                                                               int K, int N, const float* __restrict__ split_slots,
                                                               uint16_t* __restrict__ out, int grid_parts) {
  constexpr int PER_TILE = kReduceUnits / 256;   // blocks per tile
  const FfnTiles map(rep_offsets, E, N);
  int full, ntail, S;
  map.split_plan(grid_parts, K / kFfnKUnit, full, ntail, S);
  if (S == 1) return;
  for (int b = blockIdx.x; b < ntail * PER_TILE; b += gridDim.x) {
    const int tt = b / PER_TILE;                                    // tail tile
    const int q = ((b - tt * PER_TILE) * 256 + threadIdx.x) >> 6;   // (w*FM + fm)*FN + fn
    int e, row0, rows, n0, shape;
    map.decode(full + tt, E, e, row0, rows, n0, shape);
    const float* slots = split_slots + static_cast<size_t>(tt) * S * kFfnSlotFloats;
    const bool narrow_unit = q < FfnGemm::NWAVES * FfnGemm::FM * FfnGemm::FN;
    const bool small_unit = q < FfnGemmSmall::NWAVES * FfnGemmSmall::FM * FfnGemmSmall::FN;
    if (S == 4) {
      if (shape == kShapeWide) reduce_unit<FfnGemmWide, 4>(slots, q, row0, rows, n0, N, out);
      else if (shape == kShapeSmall) { if (small_unit) reduce_unit<FfnGemmSmall, 4>(slots, q, row0, rows, n0, N, out); }
      else if (narrow_unit) reduce_unit<FfnGemm, 4>(slots, q, row0, rows, n0, N, out);
    } else if (S == 3) {
      if (shape == kShapeWide) reduce_unit<FfnGemmWide, 3>(slots, q, row0, rows, n0, N, out);
      else if (shape == kShapeSmall) { if (small_unit) reduce_unit<FfnGemmSmall, 3>(slots, q, row0, rows, n0, N, out); }
      else if (narrow_unit) reduce_unit<FfnGemm, 3>(slots, q, row0, rows, n0, N, out);
    } else {
      if (shape == kShapeWide) reduce_unit<FfnGemmWide, 2>(slots, q, row0, rows, n0, N, out);
      else if (shape == kShapeSmall) { if (small_unit) reduce_unit<FfnGemmSmall, 2>(slots, q, row0, rows, n0, N, out); }
      else if (narrow_unit) reduce_unit<FfnGemm, 2>(slots, q, row0, rows, n0, N, out);
    }
  }
}

// float32 products.  Two tile shapes, chosen on the device from the actual
// row counts (uniform over the grid):
//  * 64 weight rows x 64 token rows on GemmF32 (float32 MFMA, LDS ring shared
//    by four waves) when those tiles give every CU at least two;
//  * else 32 x 32 tiles whose four waves each take a quarter of K, loaded
//    straight into registers in fragment layout (nothing is shared between
//    the waves, so no LDS staging and no barrier in the K loop), and add
//    their partial tiles through LDS in wave order.  A small product is bound
//    by the latency of its K loop, which this divides by four, and the finer
//    tiles fill CUs that 64 x 64 tiles would leave idle.
// GemmF32 reads rows at 32-bit offsets; a 64 x 64 tile of the first product with
// a row of x past them (x itself has no size limit) is taken as four of the
// second shape, whose rows are addressed in full.
// On 8 experts of about 172 rows (512 -> 2048 -> 512) 64 x 64 tiles of vector
// FMA took 98 and 188 us a product, these take 51 (64 x 64) and 70 us
// (32 x 32); on 4 experts of 16 rows (256 -> 1024 -> 256) 21 and 64 us, now
// 11 and 11 us.
constexpr int kF32Blocks = 3;   // blocks a CU (48 KB of LDS each)

struct F32Tiles {
  int elo, ehi, mt, incl, NT, tiles, BT;
  __device__ __forceinline__ F32Tiles(const int32_t* __restrict__ rep_offsets, int E, int N, int cus) {
    const int lane = threadIdx.x & 63;
    elo = lane < E ? rep_offsets[lane] : 0;
    ehi = lane < E ? rep_offsets[lane + 1] : 0;
    layout(64, N);
    if (tiles < 2 * cus) layout(32, N);
  }
  // Tile t -> expert e, first token row, row count, first output column.
  __device__ __forceinline__ void decode(int t, int E, int& e, int& row0, int& rows, int& n0) const {
    const int lane = threadIdx.x & 63;
    e = __popcll(__ballot(lane < E && incl <= t));
    const int me = __shfl(mt, e, 64);
    const int r = t - (__shfl(incl, e, 64) - me * NT);
    row0 = __builtin_amdgcn_readfirstlane(__shfl(elo, e, 64) + r % me * BT);
    rows = __builtin_amdgcn_readfirstlane(min(BT, __shfl(ehi, e, 64) - row0));
    n0 = __builtin_amdgcn_readfirstlane(r / me * BT);
  }

 private:
  // Tiles of bt x bt, expert by expert, the row tiles of one weight tile
  // side by side.
  __device__ __forceinline__ void layout(int bt, int N) {
    const int lane = threadIdx.x & 63;
    BT = bt;
    NT = (N + bt - 1) / bt;
    mt = (ehi - elo + bt - 1) / bt;
    incl = mt * NT;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    tiles = __builtin_amdgcn_readfirstlane(__shfl(incl, 63, 64));
  }
};

// Stores the 32 x 32 block of accumulators (lane l: token row l % 32, value v:
// column 8 (v / 4) + v % 4 + 4 (l / 32)) to rows row0.. and columns n0..
template <int ACT, bool FIRST>
__device__ __forceinline__ void store_block_f32(const f32x16& acc, int row0, int rows, int n0, int N,
                                                float* __restrict__ out) {
  const int lane = threadIdx.x & 63, r = lane & 31;
  if (r >= rows || n0 >= N) return;   // N is a multiple of 64, n0 of 32
  float* dst = out + static_cast<size_t>(row0 + r) * N + n0 + 4 * (lane >> 5);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    float z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      z[q] = acc[4 * g + q];
      if constexpr (FIRST) z[q] = act_fn<ACT>(z[q]);
    }
    *reinterpret_cast<float4*>(dst + 8 * g) = make_float4(z[0], z[1], z[2], z[3]);
  }
}

template <int ACT, bool FIRST>
__global__ __launch_bounds__(GemmF32::THREADS, kF32Blocks) void ffn_kernel_f32(
    const float* __restrict__ A, const int32_t* __restrict__ row_index,
    const int32_t* __restrict__ rep_offsets, int E, int K, int N,
    const float* __restrict__ W, float* __restrict__ out) {
  using G = GemmF32;
  static_assert(G::FM == 1 && G::FN == 1 && G::NWAVES == 4, "one 32 x 32 block a wave");
  static_assert(G::LDS_BYTES >= 4 * 16 * 64 * 4, "partial tiles of the small shape");
  __shared__ __attribute__((aligned(16))) uint8_t lds[G::LDS_BYTES];
  const F32Tiles map(rep_offsets, E, N, gridDim.x / kF32Blocks);
  const int lane = threadIdx.x & 63, w = G::wave();
  for (int t = xcd_virtual_block(); t < map.tiles; t += gridDim.x) {
    int e, row0, rows, n0;
    map.decode(t, E, e, row0, rows, n0);
    const float* We = W + static_cast<size_t>(e) * N * K;
    bool split = map.BT == 32;   // block-uniform: 32 x 32 tiles
    if constexpr (FIRST) {
      if (!split) {
        const int m = row0 + min(lane, rows - 1);
        const long long end = (static_cast<long long>(row_index ? row_index[m] : m) + 1) * K * 4;
        split = __ballot(end > static_cast<long long>(G::kRange)) != 0;
      }
    }
    if (!split) {
      uint32_t poff[G::LP], qoff[G::LQ];
#pragma unroll
      for (int j = 0; j < G::LP; ++j) poff[j] = static_cast<uint32_t>(n0 + G::load_row(j)) * 2u * K;
#pragma unroll
      for (int j = 0; j < G::LQ; ++j) {
        const int m = row0 + min(G::load_row(G::LP + j) - G::BM, rows - 1);
        qoff[j] = static_cast<uint32_t>(row_index ? row_index[m] : m) * 2u * K;
      }
      G::Acc acc;
      G::zero(acc);
      G::run(reinterpret_cast<const uint16_t*>(We), poff, reinterpret_cast<const uint16_t*>(A), qoff, 2 * K, 64, rows,
             lds, acc);
      const int qr = G::q_row(G::wave_n(w), 0);
      store_block_f32<ACT, FIRST>(acc[0][0], row0 + qr, rows - qr, n0 + G::wave_m(w) * 32, N, out);
      continue;
    }
    const int parts = map.BT == 32 ? 1 : 4;
    for (int q4 = 0; q4 < parts; ++q4) {
      const int r0 = row0 + 32 * (q4 & 1), nr = min(32, rows - 32 * (q4 & 1)), col0 = n0 + 32 * (q4 >> 1);
      if (nr <= 0) continue;
      // lane l: weight row col0 + l % 32, token row l % 32, K values 8 s + 4 (l / 32) .. + 3 of step s
      const int m = r0 + min(lane & 31, nr - 1);
      const float* pw = We + static_cast<size_t>(col0 + (lane & 31)) * K + 4 * (lane >> 5);
      const float* pa = A + static_cast<size_t>(row_index ? row_index[m] : m) * K + 4 * (lane >> 5);
      const int nk = K / 32;                                   // 32-value chunks
      const int c0 = w * nk / 4, c1 = (w + 1) * nk / 4;        // this wave's
      constexpr int D = 3;                                     // chunks in flight
      f32x4 fw[D][4], fa[D][4];
      auto load = [&](int c, f32x4 (&w4)[4], f32x4 (&a4)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          w4[u] = *reinterpret_cast<const f32x4*>(pw + 32 * c + 8 * u);
          a4[u] = *reinterpret_cast<const f32x4*>(pa + 32 * c + 8 * u);
        }
      };
      f32x16 acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
      for (int s = 0; s < D; ++s)
        if (c0 + s < c1) load(c0 + s, fw[s], fa[s]);
      // unrolled by D so that the register sets are indexed statically
      for (int c = c0; c < c1; c += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
          if (c + s >= c1) break;
#pragma unroll
          for (int u = 0; u < 4; ++u) acc = mfma32x32x8_f32(fw[s][u], fa[s][u], acc);
          if (c + s + D < c1) load(c + s + D, fw[s], fa[s]);
        }
      }
      // partial tiles: value v of lane l of wave w at [w][v][l]; wave w then adds
      // values 4w..4w+3 (columns 8w + 4 (l / 32) ..) of the four waves in order
      float* part = reinterpret_cast<float*>(lds);
      __syncthreads();   // the previous tile's sums are read
#pragma unroll
      for (int v = 0; v < 16; ++v) part[(w * 16 + v) * 64 + lane] = acc[v];
      __syncthreads();
      if ((lane & 31) < nr) {
        float z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float* p = part + (4 * w + q) * 64 + lane;
          z[q] = ((p[0] + p[16 * 64]) + p[32 * 64]) + p[48 * 64];
          if constexpr (FIRST) z[q] = act_fn<ACT>(z[q]);
        }
        *reinterpret_cast<float4*>(out + static_cast<size_t>(r0 + (lane & 31)) * N + col0 + 8 * w + 4 * (lane >> 5)) =
            make_float4(z[0], z[1], z[2], z[3]);
      }
    }
    if (parts > 1) __syncthreads();   // the sums are read before the next tile's DMA
  }
}

struct FfnWs {
  void* hidden;
  float* split_slots;
  int* queue;   // kFfnQueueSets tail counters
};

FfnWs carve_ffn(Carver& c, int max_rows, int d_ff, int dtype) {
  FfnWs w;
  w.hidden = c.take<uint8_t>(static_cast<size_t>(max_rows) * d_ff * elem_bytes(dtype));
  w.split_slots = nullptr;
  w.queue = nullptr;
  if (dtype == LUFFY_BF16) {
    w.split_slots = c.take<float>(kFfnSlotFloats * kFfnMaxSlots);
    w.queue = c.take<int>(kFfnQueueSets);
  }
  return w;
}


template <int ACT>
void launch_ffn(const void* x, const int32_t* row_index, const int32_t* rep_offsets, int E, int d,
                int d_ff, int dtype, const void* w1, const void* w2, int max_rows, void* y_rep,
                const FfnWs& ws, hipStream_t s) {
  void* hidden = ws.hidden;
  if (dtype == LUFFY_BF16) {
    const int grid = persistent_grid();
    launch("ffn_queue", ffn_queue_clear_kernel, 1, 64, 0, s, ws.queue, 2);
    {
      launch("ffn1", ffn_kernel_bf16<ACT, true>, grid, FfnGemm::THREADS, 0, s, static_cast<const uint16_t*>(x),
             row_index, rep_offsets, E, d, d_ff, static_cast<const uint16_t*>(w1), static_cast<uint16_t*>(hidden),
             ws.split_slots, static_cast<uint16_t*>(nullptr), ws.queue);
    }
    {
      launch("ffn2", ffn_kernel_bf16<ACT, false>, grid, FfnGemm::THREADS, 0, s,
             static_cast<const uint16_t*>(hidden), nullptr, rep_offsets, E, d_ff, d,
             static_cast<const uint16_t*>(w2), static_cast<uint16_t*>(y_rep), ws.split_slots,
             static_cast<uint16_t*>(nullptr), ws.queue + 1);
    }
    {
      launch("ffn2_reduce", ffn_split_reduce_kernel, 8 * grid, 256, 0, s, rep_offsets, E, d_ff, d, ws.split_slots,
             static_cast<uint16_t*>(y_rep), grid);
    }
  } else {
    const int grid = kF32Blocks * persistent_grid();
    launch("ffn1", ffn_kernel_f32<ACT, true>, grid, GemmF32::THREADS, 0, s, static_cast<const float*>(x), row_index,
           rep_offsets, E, d, d_ff, static_cast<const float*>(w1), static_cast<float*>(hidden));
    launch("ffn2", ffn_kernel_f32<ACT, false>, grid, GemmF32::THREADS, 0, s, static_cast<const float*>(hidden), nullptr,
           rep_offsets, E, d_ff, d, static_cast<const float*>(w2), static_cast<float*>(y_rep));
  }
}

// ---------------------------------------------------------------- backward
// Gradients of Y = W2 act(W1 x) on the representatives (bf16):
//   Z = X W1^T (recomputed), dZ = (dY W2) * act'(Z) (in the product's
//   epilogue), dX = dZ W1, dW2 = dY^T act(Z), dW1 = dZ^T X.
// The row products dZ and dX run on the forward's grouped kernel with the
// weights read K-major (no transposed copy: the core's transposing LDS
// reads); the weight gradients contract over an expert's rows, read K-major
// from the row-major activations, with the rows past the expert's read as
// zeros up to the next multiple of 64.

// xg[r] = x[row_index[r]] for the R rows in use (one wave per row).
__global__ __launch_bounds__(256) void gather_rows_kernel(const int32_t* __restrict__ rep_offsets, int E, int d,
                                                          const uint16_t* __restrict__ x,
                                                          const int32_t* __restrict__ row_index,
                                                          uint16_t* __restrict__ xg) {
  const int R = rep_offsets[E];
  const int lane = threadIdx.x & 63;
  for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < R; r += gridDim.x * 4) {
    const uint4* src = reinterpret_cast<const uint4*>(x + static_cast<size_t>(row_index[r]) * d);
    uint4* dst = reinterpret_cast<uint4*>(xg + static_cast<size_t>(r) * d);
    for (int c = lane; c < d / 8; c += 64) dst[c] = src[c];
  }
}

// Weight gradients: out[e][i][j] = sum over the expert's rows r of
// P[r][i] Q[r][j], P [*, M] and Q [*, N] row-major token rows (both read
// K-major: the contraction runs over rows); float32 output [E][M][N]; an
// expert without rows gets zeros.
using WgradGemm = GemmCore<256, 256, 2, 4, false, false, 64, 2, true, true>;

// OUT_BF16: the sums are rounded to bf16 (the weights' own type).
// A tile has few K stages (an expert's rows / 64), so its fixed costs count:
// the operand fragments' addresses are registers and immediates, not
// recomputed per read (gemm_core.h), the stores carry no vector address
// arithmetic and write whole lines, and the tile order lets an XCD share its
// panels.  16 experts of about 250 rows, float32, 1024 x 4096 each: 112 -> 85
// us a gradient; bf16, 2048 x 8192 each, 4095 rows in all: 465 -> 270 us.  Not
// kept: 128 x 128 tiles at two blocks a CU (117 and 385 us; twice the LDS
// traffic a product), the next tile's first stages issued before the stores
// (slower by 1-7%: the loads wait behind the stores either way).
template <bool OUT_BF16>
__global__ __launch_bounds__(WgradGemm::THREADS) void wgrad_kernel(const uint16_t* __restrict__ P,
                                                                   const uint16_t* __restrict__ Q,
                                                                   const int32_t* __restrict__ rep_offsets, int E,
                                                                   int M, int N, void* __restrict__ out) {
  using G = WgradGemm;
  __shared__ __attribute__((aligned(16))) uint8_t lds[G::LDS_BYTES];
  const int mt = (M + G::BM - 1) / G::BM, nt = (N + G::BN - 1) / G::BN;
  const int tpe = mt * nt, total = E * tpe;
  // rows of expert e in lane e (E <= 64): a tile starts without a load
  const int eln = threadIdx.x & 63;
  const int elo = eln < E ? rep_offsets[eln] : 0, ehi = eln < E ? rep_offsets[eln + 1] : 0;
  for (int t = xcd_virtual_block(); t < total; t += gridDim.x) {
    // column tiles in groups of 4, row tiles next, columns fastest: the 32
    // tiles that run together on an XCD share 8 row and 4 column panels
    const int e = t / tpe, r = t - e * tpe, g = r / (4 * mt), r2 = r - g * 4 * mt, wd = min(4, nt - 4 * g);
    const int m0 = r2 / wd * G::BM, n0 = (4 * g + r2 % wd) * G::BN;
    const int lo = __builtin_amdgcn_readlane(elo, e), re = __builtin_amdgcn_readlane(ehi, e) - lo;
    uint32_t poff[G::LP], qoff[G::LQ];
    G::kmajor_offsets(poff, G::SLOTS_P, M, m0, M - m0);
    G::kmajor_offsets(qoff, G::SLOTS_Q, N, n0, N - n0);
    typename G::Acc acc;
    G::zero(acc);
    // an expert without rows has no stage and its sums stay zero
    G::template run<G::FN>(P + static_cast<size_t>(lo) * M, poff, Q + static_cast<size_t>(lo) * N, qoff,
                           (re + 63) / 64 * 64, M - m0, N - n0, lds, acc, M, N, re);
    __builtin_amdgcn_sched_barrier(0);
    // The tile's corner is the base of a buffer resource, a lane's column (and
    // its four-row half) its offset, and a row a scalar offset, so a store
    // costs no vector arithmetic.  M and N are multiples of 64: a wave's 32-row
    // and 64-column blocks are inside the matrix or outside as a whole, and
    // those outside get a resource of no bytes, whose stores are dropped.
    const int lane = opaque_tid() & 63, w = G::wave();
    const int l31 = lane & 31, hi = lane >> 5;
    const int r0 = G::wave_m(w) * G::WTM, c0 = G::q_row(G::wave_n(w), 0);
    constexpr int ES = OUT_BF16 ? 2 : 4;
    uint8_t* corner = static_cast<uint8_t*>(out) + ((static_cast<size_t>(e) * M + m0) * N + n0) * ES;
    static_assert(G::FN == 2, "column blocks are stored in pairs");
#pragma unroll
    for (int fm = 0; fm < G::FM; ++fm) {
      const bool in = n0 + c0 < N && m0 + r0 + 32 * fm < M;
      const __amdgpu_buffer_rsrc_t ors = G::rsrc(corner, in ? G::kRange : 0u);
      if constexpr (OUT_BF16) {
        // a store is four bytes a lane, a whole 128-byte line (64 columns) of
        // two rows: of lanes l and l^1, which hold neighbouring columns of both
        // 32-column blocks, the even one stores the pair of the first block and
        // the odd one that of the second
        const bool odd = lane & 1;
        const uint32_t voff = (static_cast<uint32_t>(4 * hi) * N + c0 + (odd ? 32 : 0) + (l31 & ~1)) * 2u;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float own = odd ? acc[fm][1][v] : acc[fm][0][v], snd = odd ? acc[fm][0][v] : acc[fm][1][v];
          const float rcv = __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
              0, static_cast<int>(__float_as_uint(snd)), 0xB1, 0xF, 0xF, false)));   // quad_perm [1, 0, 3, 2]: lane ^ 1
          const uint32_t word = pack_bf16x2(odd ? rcv : own, odd ? own : rcv);
          __builtin_amdgcn_raw_buffer_store_b32(word, ors, voff, (r0 + 32 * fm + 8 * (v / 4) + v % 4) * N * 2, 0);
        }
      } else {
        const uint32_t voff = (static_cast<uint32_t>(4 * hi) * N + c0 + l31) * 4u;
#pragma unroll
        for (int fn = 0; fn < G::FN; ++fn)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float f = acc[fm][fn][v];
            asm volatile("" : "+v"(f));   // one register out of the tuple at a time
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f), ors, voff + 128 * fn,
                                                  (r0 + 32 * fm + 8 * (v / 4) + v % 4) * N * 4, 0);
          }
      }
    }
  }
}

struct FfnBwdWs {
  uint16_t *z, *a, *dz, *xg;
  float* split_slots;
  int* queue;   // kFfnQueueSets tail counters
};

FfnBwdWs carve_ffn_bwd(Carver& c, int max_rows, int E, int d, int d_ff) {
  (void)E;
  FfnBwdWs w;
  w.z = c.take<uint16_t>(static_cast<size_t>(max_rows) * d_ff);
  w.a = c.take<uint16_t>(static_cast<size_t>(max_rows) * d_ff);
  w.dz = c.take<uint16_t>(static_cast<size_t>(max_rows) * d_ff);
  w.xg = c.take<uint16_t>(static_cast<size_t>(max_rows) * d);
  w.split_slots = c.take<float>(kFfnSlotFloats * kFfnMaxSlots);
  w.queue = c.take<int>(kFfnQueueSets);
  return w;
}

template <int ACT>
void launch_ffn_bwd(const uint16_t* x, const int32_t* row_index, const int32_t* rep_offsets, int E, int d, int d_ff,
                    const uint16_t* w1, const uint16_t* w2, int max_rows, const uint16_t* dy, uint16_t* dx,
                    void* dw1, void* dw2, bool dw_bf16, const FfnBwdWs& ws, hipStream_t s) {
  (void)max_rows;
  const int grid = persistent_grid();
  const int egrid = 4 * grid;
  launch("ffn_queue", ffn_queue_clear_kernel, 1, 64, 0, s, ws.queue, 3);
  // Z = X W1^T and A = act(Z), both from the product's epilogue (a pass of its
  // own that read Z back took 14 us for 4021 rows of 4096)
  constexpr int kZa = ACT == LUFFY_ACT_GELU ? kActZaGelu : kActZaSilu;
  launch("bwd_z", ffn_kernel_bf16<kZa, true>, grid, FfnGemm::THREADS, 0, s, x, row_index, rep_offsets, E, d, d_ff, w1,
         ws.z, ws.split_slots, ws.a, ws.queue);
  // dZ = (dY W2) act'(Z): W2 [E][d][d_ff] read K-major (k = output row o)
  constexpr int kDz = ACT == LUFFY_ACT_GELU ? kActDzGelu : kActDzSilu;
  launch("bwd_da", ffn_kernel_bf16<kDz, true, true>, grid, FfnGemm::THREADS, 0, s, dy, nullptr, rep_offsets, E, d,
         d_ff, w2, ws.dz, ws.split_slots, ws.z, ws.queue + 1);
  // dX = dZ W1: W1 [E][d_ff][d] read K-major, split over K as the forward's second product
  launch("bwd_dx", ffn_kernel_bf16<kActNone, false, true>, grid, FfnGemm::THREADS, 0, s,
         static_cast<const uint16_t*>(ws.dz), nullptr, rep_offsets, E, d_ff, d, w1, dx, ws.split_slots,
         static_cast<uint16_t*>(nullptr), ws.queue + 2);
  launch("bwd_dx_reduce", ffn_split_reduce_kernel, 8 * grid, 256, 0, s, rep_offsets, E, d_ff, d, ws.split_slots, dx,
         grid);
  // dW2 = dY^T A, dW1 = dZ^T X (X's rows gathered first)
  auto* wgrad = dw_bf16 ? wgrad_kernel<true> : wgrad_kernel<false>;
  launch("bwd_dw2", wgrad, grid, WgradGemm::THREADS, 0, s, dy, static_cast<const uint16_t*>(ws.a), rep_offsets, E, d,
         d_ff, dw2);
  const uint16_t* xr = x;
  if (row_index) {
    launch("bwd_gather", gather_rows_kernel, egrid, 256, 0, s, rep_offsets, E, d, x, row_index, ws.xg);
    xr = ws.xg;
  }
  launch("bwd_dw1", wgrad, grid, WgradGemm::THREADS, 0, s, static_cast<const uint16_t*>(ws.dz), xr, rep_offsets, E,
         d_ff, d, dw1);
}

}  // namespace
}  // namespace luffy

using namespace luffy;

extern "C" size_t luffy_expert_ffn_workspace_size(int max_rows, int E, int d_ff, int dtype) {
  (void)E;
  if (max_rows <= 0 || d_ff <= 0) return 0;
  Carver c(nullptr);
  carve_ffn(c, max_rows, d_ff, dtype);
  return c.size();
}

extern "C" int luffy_expert_ffn(const void* x, const int32_t* row_index,
                                const int32_t* rep_offsets, int E, int d, int d_ff,
                                int dtype, const void* w1, const void* w2, int act,
                                int max_rows, void* y_rep,
                                void* workspace, size_t workspace_bytes, void* stream) {
  if (!x || !rep_offsets || !w1 || !w2 || !y_rep)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn: null pointer argument");
  if (E <= 0 || d <= 0 || d_ff <= 0 || max_rows <= 0)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn: E=%d d=%d d_ff=%d max_rows=%d", E, d, d_ff, max_rows);
  if (dtype != LUFFY_F32 && dtype != LUFFY_BF16)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn: unknown dtype %d", dtype);
  if (act != LUFFY_ACT_GELU && act != LUFFY_ACT_SILU)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn: unknown activation %d", act);
  if (E > kMaxExperts) return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn: E=%d > %d", E, kMaxExperts);
  if (d % 64 != 0 || d_ff % 64 != 0)
    return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn: d=%d d_ff=%d must be multiples of 64", d, d_ff);
  if (d > 32768 || d_ff > 32768)
    return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn: d=%d d_ff=%d must be at most 32768", d, d_ff);
  if (static_cast<long long>(max_rows) * d_ff * elem_bytes(dtype) > 0xFFFF0000ll ||
      static_cast<long long>(d) * d_ff * elem_bytes(dtype) > 0xFFFF0000ll)
    return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn: hidden activations or one expert's weights exceed 4 GiB - 64 KiB");
  const size_t need = luffy_expert_ffn_workspace_size(max_rows, E, d_ff, dtype);
  if (workspace_bytes < need || !workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return fail(LUFFY_E_WORKSPACE, "luffy_expert_ffn: workspace needs %zu bytes, 256-aligned", need);
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(workspace);
  const FfnWs ws = carve_ffn(c, max_rows, d_ff, dtype);
  if (act == LUFFY_ACT_GELU)
    launch_ffn<LUFFY_ACT_GELU>(x, row_index, rep_offsets, E, d, d_ff, dtype, w1, w2, max_rows, y_rep, ws, s);
  else
    launch_ffn<LUFFY_ACT_SILU>(x, row_index, rep_offsets, E, d, d_ff, dtype, w1, w2, max_rows, y_rep, ws, s);
  return check_launch("luffy_expert_ffn");
}

extern "C" size_t luffy_expert_ffn_backward_workspace_size(int max_rows, int E, int d, int d_ff, int dtype) {
  if (max_rows <= 0 || E <= 0 || d <= 0 || d_ff <= 0 || dtype != LUFFY_BF16) return 0;
  Carver c(nullptr);
  carve_ffn_bwd(c, max_rows, E, d, d_ff);
  return c.size();
}

extern "C" int luffy_expert_ffn_backward(const void* x, const int32_t* row_index, const int32_t* rep_offsets, int E,
                                         int d, int d_ff, int dtype, const void* w1, const void* w2, int act,
                                         int max_rows, const void* dy_rep, void* dx_rep, void* dw1, void* dw2,
                                         int dw_dtype, void* workspace, size_t workspace_bytes, void* stream) {
  if (!x || !rep_offsets || !w1 || !w2 || !dy_rep || !dx_rep || !dw1 || !dw2)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn_backward: null pointer argument");
  if (E <= 0 || d <= 0 || d_ff <= 0 || max_rows <= 0)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn_backward: E=%d d=%d d_ff=%d max_rows=%d", E, d, d_ff, max_rows);
  if (dtype != LUFFY_F32 && dtype != LUFFY_BF16)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn_backward: unknown dtype %d", dtype);
  if (act != LUFFY_ACT_GELU && act != LUFFY_ACT_SILU)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn_backward: unknown activation %d", act);
  if (dw_dtype != LUFFY_F32 && dw_dtype != LUFFY_BF16)
    return fail(LUFFY_E_INVALID, "luffy_expert_ffn_backward: unknown weight-gradient dtype %d", dw_dtype);
  if (dtype != LUFFY_BF16) return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn_backward: bf16 only");
  if (E > kMaxExperts) return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn_backward: E=%d > %d", E, kMaxExperts);
  if (d % 64 != 0 || d_ff % 64 != 0)
    return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn_backward: d=%d d_ff=%d must be multiples of 64", d, d_ff);
  if (d > 32768 || d_ff > 32768)
    return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn_backward: d=%d d_ff=%d must be at most 32768", d, d_ff);
  // K-major reads of the activations run up to 63 rows past an expert's last
  const long long krows = static_cast<long long>(max_rows) + 64;
  if (static_cast<long long>(max_rows) * d_ff * 2 > 0xFFFF0000ll ||
      static_cast<long long>(d) * d_ff * 2 > 0xFFFF0000ll ||
      krows * (d > d_ff ? d : d_ff) * 2 > 0xFFFF0000ll)
    return fail(LUFFY_E_UNSUPPORTED, "luffy_expert_ffn_backward: an operand exceeds 4 GiB - 64 KiB");
  const size_t need = luffy_expert_ffn_backward_workspace_size(max_rows, E, d, d_ff, dtype);
  if (workspace_bytes < need || !workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return fail(LUFFY_E_WORKSPACE, "luffy_expert_ffn_backward: workspace needs %zu bytes, 256-aligned", need);
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(workspace);
  const FfnBwdWs ws = carve_ffn_bwd(c, max_rows, E, d, d_ff);
  const auto* xb = static_cast<const uint16_t*>(x);
  const auto* w1b = static_cast<const uint16_t*>(w1);
  const auto* w2b = static_cast<const uint16_t*>(w2);
  const auto* dyb = static_cast<const uint16_t*>(dy_rep);
  auto* dxb = static_cast<uint16_t*>(dx_rep);
  if (act == LUFFY_ACT_GELU)
    launch_ffn_bwd<LUFFY_ACT_GELU>(xb, row_index, rep_offsets, E, d, d_ff, w1b, w2b, max_rows, dyb, dxb, dw1, dw2,
                                   dw_dtype == LUFFY_BF16, ws, s);
  else
    launch_ffn_bwd<LUFFY_ACT_SILU>(xb, row_index, rep_offsets, E, d, d_ff, w1b, w2b, max_rows, dyb, dxb, dw1, dw2,
                                   dw_dtype == LUFFY_BF16, ws, s);
  return check_launch("luffy_expert_ffn_backward");
}

