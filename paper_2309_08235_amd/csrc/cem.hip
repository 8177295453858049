// Selection, refit and covariance factorisation of the sampling loop (Alg. 1,
// eqs. (9a)-(9c)) on gfx950: one 512-thread block per problem.
//
//   1. ConstraintEliteSet: the n_proj samples with the lowest residual r,
//      ordered by (r, index) over the order-preserving bit patterns of r
//      (ties keep index order);
//   2. EliteSet: the n_elite lowest c_aug = c1 + r among them, ties kept in
//      the order of step 1.
//   When the ordered set of step 1 is an output, both steps sort packed
//   64-bit keys (order-preserving key bits above the position) with a
//   bitonic network in LDS; otherwise (N <= 2048, n_elite <= 512) they are
//   selects of the boundary keys (histograms of the value range, then of the
//   key range, until at most 32 keys are left) and a ranking of the n_elite
//   survivors by counting, which select and order exactly the same samples.
//   3. weights c_m = exp(-(c_aug_m - delta)/gamma), delta = min c_aug;
//   4. mu' = (1-sigma) mu + sigma sum w xi_bar / sum w,
//      Sigma' = (1-sigma) Sigma + sigma sum w (xi_bar - mu')(xi_bar - mu')^T / sum w;
//   5. L = chol(Sigma' + eps I), eps = cov_jitter tr(Sigma')/D, for the next
//      draw: one wave, a rank-1 MFMA per column.
//
// One block on one CU: bound by chains of LDS round trips, barriers and the
// first fetch of code that a launch runs once.  At N = 1000, 100 elites,
// D = 22 a refit takes 37k cycles (selection 10k, weights 1k, staging and mean
// 6k, covariance 7k, factor 9k; before, 39k to 50k by the number of equal
// keys), at N = 1500, 150 elites, D = 33 60k (15k, 2k, 11k, 12k, 17k; before,
// 85k to 100k).
//
// Every sum runs in a fixed order, so results are bitwise reproducible.
#include "priest_internal.h"
#include "quotient.h"

#include <algorithm>
#include <type_traits>

namespace priest {
namespace {

// Elite rows are summed in chunks of kStageFloats / D rows (which fixes the
// order of every sum).  With up to 2048 samples all rows are staged in LDS at
// once if they fit kRawFloats, and centred kCenRows at a time for the
// covariance; otherwise one chunk is staged at a time.
constexpr int kStageFloats = 4096;
constexpr int kRawFloats = 12288;
constexpr int kCenRows = 64, kCenCols = 48;

__host__ __device__ inline size_t align16(size_t n) { return (n + 15) & ~static_cast<size_t>(15); }

struct CemLayout {
  size_t proj, elite, w, red, mu, pc, A, mu0, cov0, pc0, stage, cen, total;
};

// small: at most 2048 samples.
__host__ __device__ inline CemLayout cem_layout(int D, int n_proj, int n_elite, bool small) {
  CemLayout l{};
  size_t o = 0;
  l.proj = o;  o += align16(sizeof(int) * (n_proj > 0 ? n_proj : 1));
  l.elite = o; o += align16(sizeof(int) * (n_elite > 0 ? n_elite : 1));
  l.w = o;     o += align16(sizeof(float) * (n_elite > 0 ? n_elite : 1));
  l.red = o;   o += align16(sizeof(float) * 64);
  l.mu = o;    o += align16(sizeof(float) * D);
  l.pc = o;    o += align16(sizeof(float) * D);
  l.A = o;     o += align16(sizeof(float) * D * D);
  l.mu0 = o;   o += align16(sizeof(float) * D);
  l.cov0 = o;  o += align16(sizeof(float) * D * D);
  l.pc0 = o;   o += align16(sizeof(float) * D);
  const size_t rows = static_cast<size_t>(n_elite) * D;
  size_t staged = kStageFloats;
  if (small && rows > kStageFloats && rows <= kRawFloats) staged = rows;
  l.stage = o; o += align16(sizeof(float) * staged);
  l.cen = o;   o += small ? sizeof(float) * 2 * kCenRows * kCenCols : 0;
  l.total = o;
  return l;
}

// Order-preserving map float -> uint32 (NaN ranks as +inf, -0 as +0).
__device__ __forceinline__ uint32_t ordered_bits(float v) {
  if (v != v) v = __int_as_float(0x7f800000);
  if (v == 0.0f) v = 0.0f;
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {  // 0 where there is no source lane
  return static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ float dppf(float v) {
  return __uint_as_float(
      static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true)));
}

// The lane's value and that of lane ^ 32 (^ 16), in either order.
struct Two {
  uint32_t a, b;
};
__device__ __forceinline__ Two swap32(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return Two{r[0], r[1]};
}
__device__ __forceinline__ Two swap16(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return Two{r[0], r[1]};
}

// Sum over the wave in every lane: the butterfly over lane ^ 32, 16, 8, 4, 2, 1
// without a trip through LDS.  After the step over 8 the values repeat every 8
// lanes, so that a rotation by 4 within the row of 16 is the exchange over 4.
__device__ __forceinline__ float wave_sum(float v) {
  const Two x = swap32(__float_as_uint(v));
  v = __uint_as_float(x.a) + __uint_as_float(x.b);
  const Two y = swap16(__float_as_uint(v));
  v = __uint_as_float(y.a) + __uint_as_float(y.b);
  v += dppf<0x128>(v);  // row_ror:8
  v += dppf<0x124>(v);  // row_ror:4
  v += dppf<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dppf<0xB1>(v);   // quad_perm [1,0,3,2]
  return v;
}

// Minimum / maximum over the wave, in every lane.
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
  auto op = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
  auto mv = [](uint32_t x, auto ctrl) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_mov_dpp(static_cast<int>(x), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  v = op(v, mv(v, std::integral_constant<int, 0xB1>{}));
  v = op(v, mv(v, std::integral_constant<int, 0x4E>{}));
  v = op(v, mv(v, std::integral_constant<int, 0x124>{}));
  v = op(v, mv(v, std::integral_constant<int, 0x128>{}));
  const Two x = swap16(v);
  v = op(x.a, x.b);
  const Two y = swap32(v);
  return op(y.a, y.b);
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += dpp0<0x111>(v);  // row_shr 1, 2, 4, 8
  v += dpp0<0x112>(v);
  v += dpp0<0x114>(v);
  v += dpp0<0x118>(v);
  v += dpp0<0x142, 0xA>(v);  // lane 15 of rows 0, 2 into rows 1, 3
  v += dpp0<0x143, 0xC>(v);  // lane 31 into rows 2, 3
  return v;
}

__device__ __forceinline__ float bcast(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

using f4 = __attribute__((ext_vector_type(4))) float;

__device__ __forceinline__ f4 mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

using f32 = __attribute__((ext_vector_type(32))) float;

// Lower Cholesky factor L of A + eps I, A the D x D matrix in LDS (the lower
// triangle is read, D <= DM <= 64), by one wave.  A column's update of the rest
// is a rank-1 product: v_mfma_f32_32x32x1 (K = 1: one fused multiply-add per
// entry) applies it to rows 0..31 of columns 0..31 and 32..63 at once, and a
// second one to rows and columns 32..63.  The matrix stays symmetric, so column
// j is row j, which lies in one register of each block, columns across lanes:
// lane n then holds l_nj, which is the operand of the next product as it is.
// The next column's row is read before that product is issued and updated by a
// fused multiply-add of its own, so that the product is not in the chain, which
// per column is two broadcasts and one rsq.  That chain and, in a first pass
// through straight-line code, its fetch bound it: 9.4k cycles at D = 22 and
// 16.9k at D = 33, 7.0k and 12.7k when run again at once.  (With an SGPR
// broadcast per entry and column it took 8.8k and 19.8k; spread over eight
// waves with a barrier per column 10.3k and 17.2k.)  Writes L to LDS (zeros
// above the diagonal).  Returns false if a pivot is not positive and finite (it is
// replaced by 1).
template <int DM>
__device__ __forceinline__ bool cholesky_wave(const float* A, float eps, int D, int lane, float* L) {
  constexpr bool WIDE = DM > 32;  // rows and columns past 31
  const int n = lane & 31, h = lane >> 5;
  // register r of a block: row 8 (r / 4) + 4 h + r % 4, column n (+ 32)
  auto entry = [&](int i, int c) {
    const int hi = max(i, c), lo = min(i, c);
    const float v = A[__mul24(min(hi, D - 1), D) + min(lo, D - 1)];
    return (hi < D ? v : 0.0f) + (i == c ? (i < D ? eps : 1.0f) : 0.0f);
  };
  f32 top;          // registers 0..15: columns 0..31; 16..31: columns 32..63
  f32 low;          // 16..31: rows and columns 32..63
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 8 * (r >> 2) + 4 * h + (r & 3);
    // (rows from DM on are not read)
    top[r] = 8 * (r >> 2) < DM ? entry(i, n) : 0.0f;
    top[16 + r] = WIDE ? entry(i, 32 + n) : 0.0f;
    low[r] = 0.0f;
    low[16 + r] = WIDE && 32 + 8 * (r >> 2) < DM ? entry(32 + i, 32 + n) : 0.0f;
  }
  // row j as it stands in the blocks, columns across lanes
  auto row = [&](int j) {
    const int jr = j & 31, r = 4 * (jr >> 3) + (jr & 3);
    const float lo = j < 32 ? top[r] : low[16 + r], hi = j < 32 ? top[16 + r] : lo;
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(((jr >> 2) & 1) ? x[1] : x[0]);
  };
  bool bad = false;
  float v = row(0);
#pragma unroll
  for (int j = 0; j < DM; ++j) {
    if (j < D) {
      // the next row, without this column's product
      const float next = j + 1 < DM ? row(j + 1) : 0.0f;
      // (scalar: the pivot is positive and below 3e38 in one compare of its bits)
      const float got = bcast(v, j);
      const bool b = __float_as_uint(got) - 1u >= __float_as_uint(3.0e38f) - 1u;
      bad = bad || b;
      const float piv = b ? 1.0f : got;
      // one reciprocal square root per column: l_jj = piv * rsq(piv),
      // l_ij = a_ij * rsq(piv)
      const float inv = __builtin_amdgcn_rsqf(piv);
      const float all = (lane == j ? piv : v) * inv;
      const float l = lane >= j ? all : 0.0f;
      if (lane < D) L[lane * D + j] = l;
      // (finished rows and columns are not read again)
      if (j + 2 < DM) {
        if (j < 30) {
          // both halves: rows 0..31
          const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
          top = __builtin_amdgcn_mfma_f32_32x32x1f32(-__uint_as_float(x[0]), l, top, 0, 0, 0);
        }
        if constexpr (WIDE) low = __builtin_amdgcn_mfma_f32_32x32x1f32(-l, l, low, 0, 0, 0);
      }
      if (j + 1 < DM) v = __fmaf_rn(-bcast(l, j + 1), l, next);
    }
  }
  return !bad;
}

// Ascending sort of n packed keys (key bits << 32 | position) in LDS by a
// bitonic network over the next power of two (padding keys sort last).  The
// positions make every key distinct, so the order is that of a stable sort
// of the key bits.  Every thread of the block calls it; a[] holds at least
// the next power of two >= n entries.
__device__ __forceinline__ void bitonic_sort_keys(unsigned long long* a, int n) {
  const int tid = threadIdx.x;
  int m = 1;
  while (m < n) m <<= 1;
  for (int i = n + tid; i < m; i += kCemThreads) a[i] = ~0ull;
  __syncthreads();
  for (int k = 2; k <= m; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = tid; i < (m >> 1); i += kCemThreads) {
        const int lo = 2 * i - (i & (j - 1)), hi = lo + j;
        const unsigned long long x = a[lo], y = a[hi];
        const bool up = (lo & k) == 0;
        if ((x > y) == up) {
          a[lo] = y;
          a[hi] = x;
        }
      }
      __syncthreads();
    }
  }
}

// ---- selection without a full sort ------------------------------------------
// Used when the ordered constraint-elite set is not asked for: the two
// selections of steps 1 and 2 as selects of the k-th smallest key (select_kth: a
// histogram of the value range, then of the crossing bin's key range, until at most
// 32 keys are left to rank), then the n_elite survivors ranked by counting.  Selects exactly the samples, in exactly the order, of the two
// stable sorts: step 1 keeps the lowest (r key, index), step 2 the lowest
// (c_aug key, r key, index).

constexpr int kFastElite = kCemThreads;  // largest n_elite of the fast selection
static_assert(kCemThreads == 512, "index-order scans assume 8 waves");

// LDS of one select: extremes and counts per wave (two rounds), five histograms
// (zeroed), the list of the last keys (all ones) and its length (zeroed).
struct SelectScratch {
  uint32_t hist[5 * 256];
  uint32_t list[32];
  uint32_t ext[2 * 3 * 8];
  uint32_t len, pad[3];
};

// Inverse of ordered_bits.
__device__ __forceinline__ float ordered_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The k-th smallest (0-based) of the keys with valid[j] set, over the block (k
// below their count): v, with `less` keys below it and `eq` equal to it.  The
// smallest key, often that of r = 0, is tested first (it would fill one bin).
// Then the values from the smallest to the largest finite one are cut into 256
// equal bins (a monotone map, and one that spreads residuals and costs well);
// if the bin of the k-th holds more than 32 keys, its keys' range is cut again
// by a shift until it holds at most 32 keys, or one value.  At most 32 keys are
// ranked by counting.  Every wave reads the histogram and finds the bin on its
// own.
template <int IPT>
__device__ __forceinline__ void select_kth(const uint32_t (&key)[IPT], const bool (&valid)[IPT],
                                           uint32_t k, SelectScratch& sc, uint32_t& v, uint32_t& less,
                                           uint32_t& eq) {
  constexpr uint32_t kInf = 0xff800000u, kFew = 32;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  auto uni = [](uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
  };
  auto lane_of = [](uint32_t x, int l) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), l));
  };
  // smallest and largest of the flagged keys below `top`, and how many equal
  // the smallest
  auto extremes = [&](const bool (&in)[IPT], uint32_t top, uint32_t* e, uint32_t& lo, uint32_t& hi,
                      uint32_t& nlo) {
    uint32_t mn = ~0u, mx = 0u;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      mn = in[j] && key[j] < mn ? key[j] : mn;
      mx = in[j] && key[j] < top && key[j] > mx ? key[j] : mx;
    }
    mn = wave_extreme<false>(mn);
    mx = wave_extreme<true>(mx);
    uint32_t cnt = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      cnt += static_cast<uint32_t>(__builtin_popcountll(__ballot(in[j] && key[j] == mn)));
    if (lane == 0) {
      e[wv] = mn;
      e[8 + wv] = mx;
      e[16 + wv] = cnt;
    }
    __syncthreads();
    // (lane x of a row of 8: wave x)
    const uint32_t m = e[lane & 7], c = e[16 + (lane & 7)];
    lo = uni(wave_extreme<false>(m));
    hi = uni(wave_extreme<true>(e[8 + (lane & 7)]));
    const uint32_t part = wave_scan(lane < 8 && m == lo ? c : 0u);
    nlo = lane_of(part, 63);
  };
  // the bin of h that holds the k-th key: `less` keys before it, eq in it
  auto crossing = [&](const uint32_t* h) {
    const uint4 c = *reinterpret_cast<const uint4*>(h + 4 * lane);
    const uint32_t c2 = c.x + c.y, c3 = c2 + c.z, sum = c3 + c.w;
    const uint32_t before = less + wave_scan(sum) - sum;  // keys below this lane's first bin
    const uint32_t kb = k - before;
    const uint32_t b = (kb >= c.x ? 1u : 0u) + (kb >= c2 ? 1u : 0u) + (kb >= c3 ? 1u : 0u);
    const uint32_t n = before + (b == 0 ? 0u : b == 1 ? c.x : b == 2 ? c2 : c3);
    const uint32_t in = b == 0 ? c.x : b == 1 ? c.y : b == 2 ? c.z : c.w;
    const int l = __builtin_ctzll(__ballot(before <= k && kb < sum));
    less = lane_of(n, l);
    eq = lane_of(in, l);
    return 4u * l + lane_of(b, l);
  };
  uint32_t lo, hi, nlo;
  extremes(valid, kInf, sc.ext, lo, hi, nlo);
  if (k < nlo) {
    v = lo;
    less = 0;
    eq = nlo;
    return;
  }
  less = nlo;
  bool in[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) in[j] = valid[j] && key[j] != lo;
  bool few = false;
  {
    const float x0 = ordered_value(lo), scale = 256.0f / (ordered_value(hi) - x0);
    // (no cut if the range is empty or not finite)
    if (hi > lo && scale > 0.0f && scale < 1.0e30f && x0 > -3.0e38f) {
      uint32_t bin[IPT];
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        const float y = fminf((ordered_value(key[j]) - x0) * scale, 255.0f);
        bin[j] = static_cast<uint32_t>(y);
        if (in[j]) atomicAdd(sc.hist + bin[j], 1u);
      }
      __syncthreads();
      const uint32_t b = crossing(sc.hist);
#pragma unroll
      for (int j = 0; j < IPT; ++j) in[j] = in[j] && bin[j] == b;
      few = eq <= kFew;
    }
  }
  if (!few) {
    uint32_t n0;
    extremes(in, ~0u, sc.ext + 24, lo, hi, n0);
#pragma unroll
    for (int level = 0; level < 4; ++level) {
      // (32 bits of range, then at most 24, 16 and 8)
      const uint32_t range = hi - lo;
      const int shift = range > 255u ? 24 - __builtin_clz(range) : 0;
      uint32_t* h = sc.hist + 256 * (level + 1);
#pragma unroll
      for (int j = 0; j < IPT; ++j)
        if (in[j]) atomicAdd(h + ((key[j] - lo) >> shift), 1u);
      __syncthreads();
      const uint32_t b = crossing(h);
      if (shift == 0) {
        v = lo + b;
        return;
      }
#pragma unroll
      for (int j = 0; j < IPT; ++j) in[j] = in[j] && ((key[j] - lo) >> shift) == b;
      lo += b << shift;
      hi = lo + ((1u << shift) - 1u);
      if (eq <= kFew) break;
    }
  }
  // at most kFew keys left
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if (in[j]) sc.list[atomicAdd(&sc.len, 1u) & (kFew - 1)] = key[j];
  __syncthreads();
  const uint32_t mine = sc.list[lane & (kFew - 1)], kk = k - less;
  uint32_t below = 0, same = 0;
#pragma unroll
  for (uint32_t x = 0; x < kFew; x += 4) {
    if (x >= eq) break;
    const uint4 o = *reinterpret_cast<const uint4*>(sc.list + x);
    below += (o.x < mine ? 1u : 0u) + (o.y < mine ? 1u : 0u) + (o.z < mine ? 1u : 0u) + (o.w < mine ? 1u : 0u);
    same += (o.x == mine ? 1u : 0u) + (o.y == mine ? 1u : 0u) + (o.z == mine ? 1u : 0u) + (o.w == mine ? 1u : 0u);
  }
  const int l = __builtin_ctzll(__ballot(below <= kk && kk < below + same));
  v = lane_of(mine, l);
  less += lane_of(below, l);
  eq = lane_of(same, l);
}

// Exclusive count of the set flags in index order (item j of thread t is
// sample j * 512 + t).  wc: 8 * IPT LDS words.
template <int IPT>
__device__ __forceinline__ void index_scan(const bool (&f)[IPT], uint32_t (&pre)[IPT], uint32_t* wc) {
  static_assert(8 * IPT <= 64, "one count per lane");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const unsigned long long b = __ballot(f[j]);
    pre[j] = static_cast<uint32_t>(__builtin_popcountll(b & lt));
    if (lane == 0) wc[8 * j + wv] = static_cast<uint32_t>(__builtin_popcountll(b));
  }
  __syncthreads();
  const uint32_t c = lane < 8 * IPT ? wc[lane] : 0u;
  const uint32_t before = wave_scan(c) - c;
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    pre[j] += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(before), 8 * j + wv));
}

// LDS of the selection without a sort: two selects' scratch, scan counts, and
// four lists of kFastElite entries (c_aug keys, r keys, indices, ranks).  The
// histograms and lengths, `cnt`, `tie` and the ranks must be zero on entry.
template <int IPT>
struct FastScratch {
  alignas(16) SelectScratch sel[2];
  uint32_t cnt, tie;
  alignas(16) uint32_t lrank[kFastElite];
  alignas(16) uint32_t lk2[kFastElite];
  uint32_t lk1[kFastElite];
  int li[kFastElite];
  uint32_t wc[8 * IPT];
};

// Steps 1 and 2 for N <= 512 * IPT samples: elite[0..n_elite) receives the
// sample indices in rank order.  vr / vc: this thread's r and c1 (sample
// j * 512 + tid); s_r: r of every sample (LDS); gk2: N LDS words of scratch.
template <int IPT>
__device__ __forceinline__ void select_fast(const float (&vr)[IPT], const float (&vc)[IPT], int N,
                                            int n_proj, int n_elite, const float* s_r,
                                            FastScratch<IPT>& ws, uint32_t* gk2, int* elite) {
  const int tid = threadIdx.x;
  bool valid[IPT];
  uint32_t k1[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    valid[j] = tid + j * kCemThreads < N;
    k1[j] = valid[j] ? ordered_bits(vr[j]) : ~0u;
  }
  // step 1: the n_proj lowest (r key, index)
  uint32_t v1, less1, eq1;
  select_kth<IPT>(k1, valid, static_cast<uint32_t>(n_proj - 1), ws.sel[0], v1, less1, eq1);
  const uint32_t t1 = static_cast<uint32_t>(n_proj) - less1;  // members among the keys equal to v1
  bool mem[IPT];
  if (eq1 == t1) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) mem[j] = valid[j] && k1[j] <= v1;
  } else {
    bool tie[IPT];
    uint32_t pre[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) tie[j] = valid[j] && k1[j] == v1;
    index_scan<IPT>(tie, pre, ws.wc);
#pragma unroll
    for (int j = 0; j < IPT; ++j) mem[j] = valid[j] && (k1[j] < v1 || (tie[j] && pre[j] < t1));
  }
  // step 2: the n_elite lowest (c_aug key, r key, index) among them
  uint32_t k2[IPT];
#pragma unroll
  for (int j = 0; j < IPT; ++j) k2[j] = mem[j] ? ordered_bits(vc[j] + vr[j]) : ~0u;
  uint32_t v2, less2, eq2;
  select_kth<IPT>(k2, mem, static_cast<uint32_t>(n_elite - 1), ws.sel[1], v2, less2, eq2);
  const uint32_t t2 = static_cast<uint32_t>(n_elite) - less2;
  bool sel[IPT];
  if (eq2 == t2) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) sel[j] = mem[j] && k2[j] <= v2;
  } else {
    // more c_aug ties at the boundary than places left: rank the tied
    // samples by (r key, index)
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      if (valid[j]) gk2[tid + j * kCemThreads] = k2[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      sel[j] = mem[j] && k2[j] < v2;
      if (mem[j] && k2[j] == v2) {
        const int i = tid + j * kCemThreads;
        uint32_t rank = 0;
        for (int x = 0; x < N; ++x) {
          const uint32_t kx = ordered_bits(s_r[x]);
          rank += static_cast<uint32_t>(gk2[x] == v2) &
                  (static_cast<uint32_t>(kx < k1[j]) | (static_cast<uint32_t>(kx == k1[j]) & static_cast<uint32_t>(x < i)));
        }
        sel[j] = rank < t2;
      }
    }
  }
  // the n_elite survivors, in slots of arbitrary order ...
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    if (sel[j]) {
      const uint32_t slot = atomicAdd(&ws.cnt, 1u);
      if (slot < static_cast<uint32_t>(n_elite)) {
        ws.lk2[slot] = k2[j];
        ws.lk1[slot] = k1[j];
        ws.li[slot] = tid + j * kCemThreads;
      }
    }
  }
  const int n4 = (n_elite + 3) >> 2;
  if (tid >= n_elite && tid < 4 * n4) ws.lk2[tid] = ~0u;  // (above every key)
  __syncthreads();
  // ... ranked by counting: Q threads per survivor, each over a share of the
  // others, four c_aug keys per read.  Survivors with equal c_aug get the same
  // rank, hence the same place in the list, where one of them misses itself:
  // then the ranks are counted again with all three fields.
  const int Q = kCemThreads / n_elite, per = (n4 + Q - 1) / Q;
  const int am = tid % n_elite, q = tid / n_elite;
  if (q < Q) {
    const uint32_t ak = ws.lk2[am];
    uint32_t rk = 0;
#pragma unroll 4
    for (int b = q * per; b < min((q + 1) * per, n4); ++b) {
      const uint4 bk = *reinterpret_cast<const uint4*>(ws.lk2 + 4 * b);
      rk += (bk.x < ak ? 1u : 0u) + (bk.y < ak ? 1u : 0u) + (bk.z < ak ? 1u : 0u) + (bk.w < ak ? 1u : 0u);
    }
    if (Q == 1) ws.lrank[am] = rk;
    else atomicAdd(ws.lrank + am, rk);
  }
  __syncthreads();
  uint32_t place = 0;
  if (tid < n_elite) {
    place = ws.lrank[tid];
    elite[place] = ws.li[tid];
  }
  __syncthreads();
  if (tid < n_elite && elite[place] != ws.li[tid]) ws.tie = 1u;
  __syncthreads();
  if (ws.tie) {
    uint32_t rk = 0;
    if (tid < n_elite) {
      const unsigned long long ak = (static_cast<unsigned long long>(ws.lk2[tid]) << 32) | ws.lk1[tid];
      const int ai = ws.li[tid];
      for (int b = 0; b < n_elite; ++b) {
        const unsigned long long bk = (static_cast<unsigned long long>(ws.lk2[b]) << 32) | ws.lk1[b];
        const int bi = ws.li[b];
        rk += static_cast<uint32_t>(bk < ak) | (static_cast<uint32_t>(bk == ak) & static_cast<uint32_t>(bi < ai));
      }
      elite[rk] = ai;
    }
  }
}

// One block's work: selection, refit and factorisation for problem `prob`
// of `a`.  Shared by the uniform-batch kernel and the descriptor-table kernel.
template <int IPT, int DM>
__device__ __forceinline__ void cem_block(const CemArgs& a, int prob) {
  // packed sort keys of the ordered selection; their low words double as the
  // fast selection's scratch
  __shared__ unsigned long long skv[kCemThreads * IPT];
  uint32_t* skey = reinterpret_cast<uint32_t*>(skv);
  // r and c1 of every sample, read from HBM once (up to 2048 samples; larger
  // problems gather them from HBM)
  constexpr bool kPre = IPT <= 4;
  __shared__ float s_r[kPre ? kCemThreads * IPT : 1], s_c1[kPre ? kCemThreads * IPT : 1];
  struct None {};
  __shared__ std::conditional_t<kPre, FastScratch<kPre ? IPT : 1>, None> s_fast;
  extern __shared__ float4 sm4[];
  char* sm = reinterpret_cast<char*>(sm4);
  const int D = a.D, N = a.N, tid = threadIdx.x;
  constexpr int T = kCemThreads;  // (every launch of the refit uses this block size)
  const CemLayout l = cem_layout(D, a.n_proj, a.n_elite, kPre);
  int* proj = reinterpret_cast<int*>(sm + l.proj);
  int* elite = reinterpret_cast<int*>(sm + l.elite);
  float* w = reinterpret_cast<float*>(sm + l.w);
  float* red = reinterpret_cast<float*>(sm + l.red);
  float* muN = reinterpret_cast<float*>(sm + l.mu);
  float* pcN = reinterpret_cast<float*>(sm + l.pc);
  float* A = reinterpret_cast<float*>(sm + l.A);
  float* mu0 = reinterpret_cast<float*>(sm + l.mu0);
  float* cov0 = reinterpret_cast<float*>(sm + l.cov0);
  float* pc0 = reinterpret_cast<float*>(sm + l.pc0);
  float* mu = a.mu + prob * a.mu_stride;
  float* cov = a.cov + prob * a.cov_stride;
  float* L = a.L + prob * a.L_stride;

  bool best_ok = true;  // the best c_aug is not NaN
  // (the factorisation that starts a plan also starts its status word)
  if (a.chol_only && a.status && tid == 0) a.status[prob] = PRIEST_OK;
  if (!a.chol_only) {
    const float* xb = a.xb + prob * a.xb_stride;
    // everything the refit reads besides the elite rows, loaded in one batch
    // so that the block waits on HBM once: r, c1, mu, Sigma (and the
    // evolution path)
    const float* r = a.resid + prob * a.n_stride;
    const float* c1 = a.c1 + prob * a.n_stride;
    // the ordered constraint-elite set is produced only when asked for;
    // otherwise both selections run without a sort
    const bool fast = kPre && !a.proj_idx && a.n_elite <= kFastElite;
    if constexpr (kPre) {
      if (fast) {  // (while the loads below are on their way)
        for (int i = tid; i < 5 * 256; i += T) s_fast.sel[0].hist[i] = s_fast.sel[1].hist[i] = 0u;
        if (tid < 32) s_fast.sel[0].list[tid] = s_fast.sel[1].list[tid] = ~0u;
        s_fast.lrank[tid] = 0u;
        if (tid == 0) s_fast.sel[0].len = s_fast.sel[1].len = s_fast.cnt = s_fast.tie = 0u;
      }
    }
    constexpr int kCovPer = (DM * DM + kCemThreads - 1) / kCemThreads;
    float vr[IPT], vc[IPT], vcov[kCovPer];
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const int i = tid + k * kCemThreads;
      vr[k] = i < N ? r[i] : 0.0f;
      vc[k] = (kPre && i < N) ? c1[i] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < kCovPer; ++k) {
      const int i = tid + k * kCemThreads;
      vcov[k] = i < D * D ? cov[i] : 0.0f;
    }
    const float vmu = tid < D ? mu[tid] : 0.0f;
    const float vpc = (a.rule == 1 && !a.first && tid < D) ? a.pc[prob * a.pc_stride + tid] : 0.0f;
#pragma unroll
    for (int k = 0; k < kCovPer; ++k) {
      const int i = tid + k * kCemThreads;
      if (i < D * D) cov0[i] = vcov[k];
    }
    if (tid < D) {
      mu0[tid] = vmu;
      pc0[tid] = vpc;
    }
    // 1. lowest residuals
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const int i = tid + k * kCemThreads;
      if (i < N) {
        if constexpr (kPre) {
          s_r[i] = vr[k];
          s_c1[i] = vc[k];
        }
        if (!fast) skv[i] = (static_cast<unsigned long long>(ordered_bits(vr[k])) << 32) | static_cast<uint32_t>(i);
      }
    }
    if constexpr (kPre) {
      r = s_r;
      c1 = s_c1;
    }
    __syncthreads();
    if (fast) {
      if constexpr (kPre) select_fast<IPT>(vr, vc, N, a.n_proj, a.n_elite, s_r, s_fast, skey, elite);
      __syncthreads();
    } else {
      bitonic_sort_keys(skv, N);
      for (int i = tid; i < a.n_proj; i += T) {
        const int s = static_cast<int>(static_cast<uint32_t>(skv[i]));
        proj[i] = s;
        if (a.proj_idx) a.proj_idx[prob * a.n_proj + i] = s;
      }
      __syncthreads();
      // 2. lowest c_aug within them; ties keep the order of step 1
      for (int i = tid; i < a.n_proj; i += T) {
        const int s = proj[i];
        skv[i] = (static_cast<unsigned long long>(ordered_bits(c1[s] + r[s])) << 32) |
                 static_cast<uint32_t>(i);
      }
      __syncthreads();
      bitonic_sort_keys(skv, a.n_proj);
      for (int m = tid; m < a.n_elite; m += T) elite[m] = proj[static_cast<uint32_t>(skv[m])];
      __syncthreads();
    }
    if (a.elite_idx)
      for (int m = tid; m < a.n_elite; m += T) a.elite_idx[prob * a.n_elite + m] = elite[m];
    // 3. weights; fixed-order sum by the first wave
    const int e0 = elite[0];
    const float delta = c1[e0] + r[e0];
    for (int m = tid; m < a.n_elite; m += T) {
      const int s = elite[m];
      w[m] = expf(-((c1[s] + r[s]) - delta) / a.gamma);
    }
    __syncthreads();
    if (tid < 64) {
      float part = 0.0f, part2 = 0.0f;
      for (int m = tid; m < a.n_elite; m += 64) {
        part += w[m];
        part2 = fmaf(w[m], w[m], part2);
      }
      part = wave_sum(part);
      part2 = wave_sum(part2);
      if (tid == 0) {
        red[0] = part;
        red[1] = part2;
      }
    }
    __syncthreads();
    const float inv_sw = 1.0f / red[0];
    // CMA-ES-style rates (rule 1): variance-effective selection mass and the
    // default learning rates for dimension n = D
    float cc = 0.0f, c1r = 0.0f, cmu = 0.0f, mu_eff = 1.0f;
    if (a.rule == 1) {
      const float n = static_cast<float>(D);
      mu_eff = red[0] * red[0] / red[1];
      cc = (4.0f + mu_eff / n) / (n + 4.0f + 2.0f * mu_eff / n);
      c1r = 2.0f / ((n + 1.3f) * (n + 1.3f) + mu_eff);
      cmu = fminf(1.0f - c1r, 2.0f * (mu_eff - 2.0f + 1.0f / mu_eff) / ((n + 2.0f) * (n + 2.0f) + mu_eff));
    }
    // 4. mean and covariance from elite rows staged in LDS, CH rows at a time
    float* stage = reinterpret_cast<float*>(sm + l.stage);
    const int CH = kStageFloats / D;
    const bool one_chunk = a.n_elite <= CH;
    const int wv = tid >> 6, lane = tid & 63;
    // every row is staged (raw) or one chunk of them at a time
    const bool raw = one_chunk || (kPre && a.n_elite * D <= kRawFloats);
    // (16 loads per thread in flight)
    const uint32_t inv_d = inverse_of(static_cast<uint32_t>(D));
    auto stage_rows = [&](int m0, int nm) {
      constexpr int kG = 16;
      const int n = nm * D;
      for (int b = 0; b < n; b += kG * kCemThreads) {
        float v[kG];
#pragma unroll
        for (int u = 0; u < kG; ++u)
          if (b + u * kCemThreads < n) {
            const int i = min(b + u * kCemThreads + tid, n - 1);
            const int m = static_cast<int>(quotient(static_cast<uint32_t>(i), inv_d));
            v[u] = xb[elite[m0 + m] * D + (i - m * D)];
          }
#pragma unroll
        for (int u = 0; u < kG; ++u) {
          const int i = b + u * kCemThreads + tid;
          if (i < n) stage[i] = v[u];
        }
      }
    };
    // mean: coefficient d gets 4 partial sums (elites m = part mod 4 of each
    // chunk), added in a fixed order; the partials live in A until the
    // covariance is written
    float macc = 0.0f;
    const int part = tid / D, md = tid - part * D;
    if (raw) {
      stage_rows(0, a.n_elite);
      __syncthreads();
    }
    for (int m0 = 0; m0 < a.n_elite; m0 += CH) {
      const int nm = min(CH, a.n_elite - m0);
      if (!raw) {
        stage_rows(m0, nm);
        __syncthreads();
      }
      if (part < 4) {
        const float* x = stage + (raw ? m0 * D : 0) + md;
        const float* wm = w + m0;
        int m = part;
        for (; m + 28 < nm; m += 32) {
          float xv[8], wq[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            xv[u] = x[(m + 4 * u) * D];
            wq[u] = wm[m + 4 * u];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) macc = fmaf(wq[u], xv[u], macc);
        }
        for (; m < nm; m += 4) macc = fmaf(wm[m], x[m * D], macc);
      }
      if (!raw) __syncthreads();
    }
    if (part < 4) A[tid] = macc;
    __syncthreads();
    if (tid < D) {
      const float sm4 = (A[tid] + A[D + tid]) + (A[2 * D + tid] + A[3 * D + tid]);
      const float mw = sm4 * inv_sw;
      muN[tid] = (1.0f - a.sigma) * mu0[tid] + a.sigma * mw;
      if (a.rule == 1) {
        pcN[tid] = fmaf(sqrtf(cc * (2.0f - cc) * mu_eff), mw - mu0[tid], (1.0f - cc) * pc0[tid]);
      }
    }
    __syncthreads();
    // covariance about the new mean, sum_m w_m (x_m - mu')(x_m - mu')^T (rule
    // 1: about the current mean), on MFMA 16x16x4: wave v computes
    // lower-triangle tile v of the ceil(D/16)^2 tiles, elites four at a time
    // (two accumulation chains, added at the end)
    const float* cen = (a.rule == 1) ? mu0 : muN;
    const int nt = (D + 15) / 16;
    int ti = 0, tj = 0;
    {
      int v = wv;
      while (ti < nt && v > ti) {
        v -= ti + 1;
        ++ti;
      }
      tj = v;
    }
    const bool owner = ti < nt;
    f4 acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
    if constexpr (kPre) {
      // centred rows, weighted (xw) and not (xc), padded with zeros to whole
      // steps of 32 elites and tiles of 16 columns: the MFMA operands are then
      // plain reads at constant distances
      float* xc = reinterpret_cast<float*>(sm + l.cen);
      float* xw = xc + kCenRows * kCenCols;
      for (int m0 = 0; m0 < a.n_elite; m0 += CH) {
        const int nm = min(CH, a.n_elite - m0);
        if (!raw) {
          stage_rows(m0, nm);
          __syncthreads();
        }
        const float* rows = stage + (raw ? m0 * D : 0);
        for (int b0 = 0; b0 < nm; b0 += kCenRows) {
          const int nb = min(kCenRows, nm - b0), n32 = (nb + 31) & ~31;
          // (wave v takes rows v, v + 8, ..., lane c column c)
          if (lane < kCenCols) {
            const int cc = min(lane, D - 1);
            const float mc = cen[cc];
#pragma unroll
            for (int u = 0; u < kCenRows / 8; ++u) {
              const int m = wv + 8 * u;
              if (m >= n32) break;
              const int mm = b0 + min(m, nb - 1);
              const float d = rows[mm * D + cc] - mc, wd = w[m0 + mm] * d;
              const bool in = m < nb && lane < D;
              xc[m * kCenCols + lane] = in ? d : 0.0f;
              xw[m * kCenCols + lane] = in ? wd : 0.0f;
            }
          }
          __syncthreads();
          if (owner) {
            const float* pa = xw + (lane >> 4) * kCenCols + ti * 16 + (lane & 15);
            const float* pb = xc + (lane >> 4) * kCenCols + tj * 16 + (lane & 15);
            for (int s0 = 0; s0 < n32; s0 += 32) {
              float av[8], bv[8];
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                av[u] = pa[(s0 + 4 * u) * kCenCols];
                bv[u] = pb[(s0 + 4 * u) * kCenCols];
              }
#pragma unroll
              for (int u = 0; u < 8; u += 2) {
                acc0 = mfma(av[u], bv[u], acc0);
                acc1 = mfma(av[u + 1], bv[u + 1], acc1);
              }
            }
          }
          __syncthreads();
        }
      }
    } else {
      for (int m0 = 0; m0 < a.n_elite; m0 += CH) {
        const int nm = min(CH, a.n_elite - m0);
        if (!raw) {
          stage_rows(m0, nm);
          __syncthreads();
        }
        const float* rows = stage + (raw ? m0 * D : 0);
        if (owner) {
          const int ii = ti * 16 + (lane & 15), jj = tj * 16 + (lane & 15);
          const bool iok = ii < D, jok = jj < D;
          const int ic = iok ? ii : 0, jc = jok ? jj : 0;
          const float mi = cen[ic], mj = cen[jc];
          // four groups of eight elites per step: every load of a step is
          // issued before its products.  Positions past the chunk load a
          // clamped, in-range (finite) row and are scaled by zero: a select
          // here lets the compiler move each load under its own branch, one
          // LDS round trip after another.
          constexpr int kU = 4;
          for (int s0 = 0; s0 < nm; s0 += 8 * kU) {
            float av[kU][2], bv[kU][2];
#pragma unroll
            for (int u = 0; u < kU; ++u)
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const int m = s0 + 8 * u + 4 * h + (lane >> 4);
                const bool ok = m < nm;
                const int mc = ok ? m : 0;
                const float wm = w[m0 + mc], xi_ = rows[mc * D + ic], xj_ = rows[mc * D + jc];
                av[u][h] = (wm * (xi_ - mi)) * ((ok && iok) ? 1.0f : 0.0f);
                bv[u][h] = (xj_ - mj) * ((ok && jok) ? 1.0f : 0.0f);
              }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
              acc0 = mfma(av[u][0], bv[u][0], acc0);
              acc1 = mfma(av[u][1], bv[u][1], acc1);
            }
          }
        }
        if (!raw) __syncthreads();
      }
    }
    if (owner) {
      const f4 acc = acc0 + acc1;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = ti * 16 + 4 * (lane >> 4) + r, j = tj * 16 + (lane & 15);
        if (i < D && j < D && i >= j) {
          float v;
          if (a.rule == 1)
            v = fmaf(cmu, acc[r] * inv_sw,
                     fmaf(c1r, pcN[i] * pcN[j], (1.0f - c1r - cmu) * cov0[i * D + j]));
          else
            v = (1.0f - a.sigma) * cov0[i * D + j] + a.sigma * (acc[r] * inv_sw);
          A[i * D + j] = v;
          A[j * D + i] = v;
        }
      }
    }
    __syncthreads();
    // the outputs other than L, written by the other waves while the first
    // one factors
    if (tid >= 64) {
      const int t2 = tid - 64, T2 = T - 64;
      for (int e = t2; e < D * D; e += T2) cov[e] = A[e];
      for (int d = t2; d < D; d += T2) {
        mu[d] = muN[d];
        if (a.rule == 1) a.pc[prob * a.pc_stride + d] = pcN[d];
        // (elite 0's row is still staged when all elites are)
        a.best_xi[prob * a.best_stride + d] = raw ? stage[d] : xb[static_cast<int64_t>(e0) * D + d];
      }
      if (t2 == 0) a.best_cost[prob] = delta;
    }
    best_ok = delta == delta;
  } else {
    for (int e = tid; e < D * D; e += T) A[e] = cov[e];
    __syncthreads();
  }
  // 5. factor Sigma' + eps I (first wave), into the place of the old Sigma
  float* Ls = cov0;
  if (tid < 64) {
    float tr = 0.0f;
    for (int d = tid; d < D; d += 64) tr += A[d * D + d];
    tr = wave_sum(tr);
    const float eps = a.cov_jitter * tr / static_cast<float>(D);
    const bool ok = cholesky_wave<DM>(A, eps, D, tid, Ls);
    if (tid == 0 && a.status && !(ok && best_ok)) a.status[prob] = PRIEST_ERR_NONFINITE;
  }
  __syncthreads();
  for (int e = tid; e < D * D; e += T) L[e] = Ls[e];
}

template <int IPT, int DM>
__global__ __launch_bounds__(kCemThreads) void cem_kernel(CemArgs a) {
  cem_block<IPT, DM>(a, blockIdx.x);
}

// Descriptor table: block t handles task t with its own arguments.
template <int IPT, int DM>
__global__ __launch_bounds__(kCemThreads) void cem_task_kernel(const CemArgs* tasks) {
  cem_block<IPT, DM>(tasks[blockIdx.x], 0);
}

}  // namespace

size_t cem_lds_bytes(int N, int D, int n_elite) {
  return cem_layout(D, N, n_elite, N <= kCemThreads * 4).total;
}

template <int DM>
static void launch_dm(const CemArgs& a, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  if (a.N <= kCemThreads * 2) hipLaunchKernelGGL((cem_kernel<2, DM>), grid, block, lds, s, a);
  else if (a.N <= kCemThreads * 4) hipLaunchKernelGGL((cem_kernel<4, DM>), grid, block, lds, s, a);
  else hipLaunchKernelGGL((cem_kernel<16, DM>), grid, block, lds, s, a);
}

template <int DM>
static void launch_task_dm(const CemTaskLaunch& t, size_t lds, hipStream_t s) {
  const dim3 grid(t.n_tasks), block(kCemThreads);
  if (t.max_N <= kCemThreads * 2) hipLaunchKernelGGL((cem_task_kernel<2, DM>), grid, block, lds, s, t.tasks);
  else if (t.max_N <= kCemThreads * 4) hipLaunchKernelGGL((cem_task_kernel<4, DM>), grid, block, lds, s, t.tasks);
  else hipLaunchKernelGGL((cem_task_kernel<16, DM>), grid, block, lds, s, t.tasks);
}

hipError_t launch_cem_tasks(const CemTaskLaunch& t, hipStream_t s) {
  // the most that any number of elites up to the largest takes: that of the
  // largest, or of the most whose rows are all staged
  const bool small = t.max_N <= kCemThreads * 4;
  const size_t lds = std::max(cem_layout(t.D, t.max_N, t.max_elite, small).total,
                              cem_layout(t.D, t.max_N, std::min(t.max_elite, kRawFloats / t.D), small).total);
  if (t.D <= 24) launch_task_dm<24>(t, lds, s);
  else if (t.D <= 36) launch_task_dm<36>(t, lds, s);
  else launch_task_dm<48>(t, lds, s);
  return hipGetLastError();
}

// D-PRIEST pick: the group with the lowest final cost (NaN ranks last, ties
// go to the lower group index) and a copy of its best trajectory.
__global__ void pick_best_kernel(int G, int D, const float* xi, const float* cost, float* best_xi,
                                 float* best_cost, int32_t* best_group) {
  __shared__ int sb;
  if (threadIdx.x == 0) {
    int b = 0;
    float bc = cost[0];
    if (bc != bc) bc = INFINITY;
    for (int g = 1; g < G; ++g) {
      float c = cost[g];
      if (c != c) c = INFINITY;
      if (c < bc) {
        bc = c;
        b = g;
      }
    }
    sb = b;
    best_cost[0] = cost[b];
    best_group[0] = b;
  }
  __syncthreads();
  for (int d = threadIdx.x; d < D; d += blockDim.x) best_xi[d] = xi[static_cast<int64_t>(sb) * D + d];
}

hipError_t launch_pick_best(int G, int D, const float* xi, const float* cost, float* best_xi,
                            float* best_cost, int32_t* best_group, hipStream_t s) {
  hipLaunchKernelGGL(pick_best_kernel, dim3(1), dim3(64), 0, s, G, D, xi, cost, best_xi, best_cost,
                     best_group);
  return hipGetLastError();
}

hipError_t launch_cem(const CemArgs& a, int n_problems, hipStream_t s) {
  const size_t lds = cem_layout(a.D, a.n_proj, a.n_elite, a.N <= kCemThreads * 4).total;
  const dim3 grid(n_problems), block(kCemThreads);
  // covariance factor rows padded to 24 / 36 / 48 (identity padding)
  if (a.D <= 24) launch_dm<24>(a, grid, block, lds, s);
  else if (a.D <= 36) launch_dm<36>(a, grid, block, lds, s);
  else launch_dm<48>(a, grid, block, lds, s);
  return hipGetLastError();
}

}  // namespace priest
