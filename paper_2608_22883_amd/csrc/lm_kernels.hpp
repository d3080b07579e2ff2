// Draft candidates from the corrected state: logits z = W_LM h_hat over the vocabulary
// and the top-k tokens of every node (paper, Eq. hidden_correction's z_n and Algorithm 1's
// tree expansion, which adds each node's K_c most likely tokens; K_c = 6 in the
// experimental setup).
//
// Two kernels:
//  * lm_kernel / lm_pp_kernel: the logit GEMM (the cores of gemm.hpp: for bf16 the tile that
//    best_bf_tile picks, 64- or 128-row tiles for few rows or a small vocabulary and the
//    ping-pong core's 256-column tiles for the rest; 64-, 128- and 256-row tiles for fp32)
//    with an epilogue that keeps, for
//    every row of the tile, its k largest logits and writes them as candidates
//    [row][column tile][k] - the logits themselves never reach memory;
//  * lm_merge_kernel: one block per row merges the row's candidates into its top k.
// A candidate is one 64-bit key: the logit mapped to an order-preserving unsigned
// integer in the high word and the complemented token id in the low word, so that one
// unsigned comparison orders by logit and then by ascending id.  A NaN logit and an
// empty slot are key 0, below every real logit (-inf included); key 0 decodes to id -1.
// Tile order (LmMap): XCD x owns the x-th eighth of the column tiles, so each weight
// row is pulled into one L2 only; inside its slice an XCD walks groups of up to eight
// row tiles with the row fastest, so the blocks in flight on it cover a patch of about
// 8 x 4 tiles that share their h rows and weight rows through the L2, and a head too
// large for the Infinity Cache (Qwen's 1.09 GB) is read from HBM once per eight row
// tiles rather than once per row tile (measured: 6% on 768 rows of that head).
// Selection (lm_select_quad): four lanes of a wave share a row of the staged tile, a
// quarter of its columns each.  The k-th largest of the row's 32 chunk maxima (8 chunks a
// lane, sorted by a network and merged over the four lanes) bounds the row's k-th largest
// logit from below, so the few logits that reach it (about 7 for k = 6) are all that is
// ranked.  About 8 VALU operations per logit; a sorting network over every logit took
// about 37 (a 256 x 256 tile: 28 us of epilogue after 66 us of products; now 5 us).
#pragma once

#include <cfloat>

#include "common.hpp"
#include "gemm.hpp"

namespace fovea {

template <typename T, int BM>
using LmCfg = GemmCfg<T, BM, BM == 256 ? 3 : 4>;  // three 48 KB stages fit the 256-row tile

constexpr int kLmMaxK = 16;
constexpr int kLmMaxVocab = 1 << 24;
constexpr int kLmMaxRows = 1 << 20;

struct LmMap {
  int rb, cb;  // row and column tiles
  int rc;      // column tiles per XCD
  int gr;      // row tiles per group
  __device__ __forceinline__ bool map(int& tr, int& tc) const {
    const int x = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int g = slot / (gr * rc);
    const int r0 = g * gr;
    if (r0 >= rb) return false;
    const int gs = min(gr, rb - r0);
    const int loc = slot - g * gr * rc;
    tr = r0 + loc % gs;
    const int lc = loc / gs;
    tc = x * rc + lc;
    return lc < rc && tc < cb;
  }
};

inline LmMap make_lm_map(int rb, int cb) {
  LmMap m;
  m.rb = rb;
  m.cb = cb;
  m.rc = (cb + 7) / 8;
  m.gr = rb < 8 ? rb : 8;
  return m;
}

inline int lm_grid(const LmMap& m) { return 8 * m.rb * m.rc; }

// ---- candidate keys -------------------------------------------------------------

// order-preserving image of a logit (-0 taken as +0, so equal logits tie on the id);
// 0 for NaN, which is below the image of -inf
__device__ __forceinline__ uint32_t lm_ord(float v) {
  const uint32_t u = __float_as_uint(v + 0.0f);
  const uint32_t o = u ^ (static_cast<uint32_t>(static_cast<int32_t>(u) >> 31) | 0x80000000u);
  return v == v ? o : 0u;
}

// the logit whose image is o (o != 0)
__device__ __forceinline__ float lm_ord_val(uint32_t o) {
  return __uint_as_float((o >> 31) ? (o ^ 0x80000000u) : ~o);
}

__device__ __forceinline__ uint64_t lm_key_of(uint32_t o, int id) {
  return o == 0u ? 0ull : (static_cast<uint64_t>(o) << 32) | static_cast<uint32_t>(~id);
}

__device__ __forceinline__ uint64_t lm_key(float v, int id) { return lm_key_of(lm_ord(v), id); }

__device__ __forceinline__ int lm_key_id(uint64_t key) {
  return static_cast<int>(~static_cast<uint32_t>(key));
}

__device__ __forceinline__ float lm_key_val(uint64_t key) {
  if (key == 0ull) return -INFINITY;
  return lm_ord_val(static_cast<uint32_t>(key >> 32));
}

// Orders the LDS accesses of one wave (they execute in issue order; this keeps the compiler
// from moving them across the point).
__device__ __forceinline__ void lm_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint64_t umax64(uint64_t a, uint64_t b) { return a > b ? a : b; }

// a and b in descending order (larger first); for 32-bit keys these are v_max / v_min,
// which need no compare result (a 64-bit compare goes through VCC, and reading VCC right
// after writing it costs wait states on this chip)
template <typename K>
__device__ __forceinline__ void cas_desc(K& a, K& b) {
  const K hi = a > b ? a : b, lo = a > b ? b : a;
  a = hi;
  b = lo;
}

__device__ __forceinline__ uint32_t dpp_perm_k(uint32_t v, int sel) { return dpp_perm(v, sel); }

__device__ __forceinline__ uint64_t dpp_perm_k(uint64_t v, int sel) {
  const uint64_t lo = dpp_perm(static_cast<uint32_t>(v), sel);
  const uint64_t hi = dpp_perm(static_cast<uint32_t>(v >> 32), sel);
  return lo | (hi << 32);
}

// Batcher's odd-even merge sort of the first 8 keys, descending (19 comparators,
// depth 6).
template <int N, typename K>
__device__ __forceinline__ void sort8_desc(K (&a)[N]) {
  static_assert(N >= 8, "list length");
  cas_desc(a[0], a[1]); cas_desc(a[2], a[3]); cas_desc(a[4], a[5]); cas_desc(a[6], a[7]);
  cas_desc(a[0], a[2]); cas_desc(a[1], a[3]); cas_desc(a[4], a[6]); cas_desc(a[5], a[7]);
  cas_desc(a[1], a[2]); cas_desc(a[5], a[6]);
  cas_desc(a[0], a[4]); cas_desc(a[1], a[5]); cas_desc(a[2], a[6]); cas_desc(a[3], a[7]);
  cas_desc(a[2], a[4]); cas_desc(a[3], a[5]);
  cas_desc(a[1], a[2]); cas_desc(a[3], a[4]); cas_desc(a[5], a[6]);
}

// Sorts a bitonic sequence of N keys (N a power of two) into descending order.
template <int N, typename K>
__device__ __forceinline__ void bitonic_desc(K (&a)[N]) {
#pragma unroll
  for (int dd = N / 2; dd >= 1; dd >>= 1)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i & dd) == 0) cas_desc(a[i], a[i + dd]);
}

// One butterfly step: the N largest of this lane's sorted list and its DPP partner's
// (partner `sel` of dpp_perm), sorted.  Both partners end with the same list.
template <int N, typename K>
__device__ __forceinline__ void merge_step(K (&a)[N], int sel) {
  K p[N];
#pragma unroll
  for (int i = 0; i < N; ++i) p[i] = dpp_perm_k(a[N - 1 - i], sel);
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = a[i] > p[i] ? a[i] : p[i];
  bitonic_desc<N>(a);
}

// Largest key over each 16-lane row (all 16 lanes active), in all 16 lanes.
__device__ __forceinline__ uint64_t row16_max64(uint64_t v) {
#pragma unroll
  for (int sel = 0; sel < 4; ++sel) v = umax64(v, dpp_perm_k(v, sel));
  return v;
}

// Largest key over the whole (fully active) wave, uniform.
__device__ __forceinline__ uint64_t wave_max64(uint64_t v) {
  v = row16_max64(v);
  uint64_t m = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 16 * r));
    const uint64_t hi =
        static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), 16 * r));
    m = umax64(m, lo | (hi << 32));
  }
  return m;
}

__device__ __forceinline__ float max3_f32(float a, float b, float c) {
  float r;  // a NaN operand is ignored
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;

// For x0 .. x3 in turn, m = 2 m + (x >= t): the compare's carry goes straight into the shift
// (left to itself the compiler keeps every compare in a scalar pair of its own and spills
// them).  A vector instruction may read a scalar pair (VCC too) only two wait states after
// another has written it, and the compiler does not look in here: the four compares stand
// before the four shifts, so that three instructions lie between each write and its read.
__device__ __forceinline__ void push4_ge_f32(uint32_t& m, float x0, float x1, float x2, float x3, float t) {
  uint64_t c0, c1, c2, c3;
  asm("v_cmp_ge_f32_e64 %1, %5, %9\n\tv_cmp_ge_f32_e64 %2, %6, %9\n\t"
      "v_cmp_ge_f32_e64 %3, %7, %9\n\tv_cmp_ge_f32_e64 %4, %8, %9\n\t"
      "v_addc_co_u32_e64 %0, vcc, %0, %0, %1\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\t"
      "v_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %4"
      : "+v"(m), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
      : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(t)
      : "vcc");
}

__device__ __forceinline__ void push4_eq_f32(uint32_t& m, float x0, float x1, float x2, float x3, float t) {
  uint64_t c0, c1, c2, c3;
  asm("v_cmp_eq_f32_e64 %1, %5, %9\n\tv_cmp_eq_f32_e64 %2, %6, %9\n\t"
      "v_cmp_eq_f32_e64 %3, %7, %9\n\tv_cmp_eq_f32_e64 %4, %8, %9\n\t"
      "v_addc_co_u32_e64 %0, vcc, %0, %0, %1\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\t"
      "v_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %4"
      : "+v"(m), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
      : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "v"(t)
      : "vcc");
}

// The value of the lane 16 (32) away: with both operands equal, a row swap leaves this
// lane's value in one result and the partner's in the other.
__device__ __forceinline__ uint32_t xor16_u32(uint32_t v, int lane) {
  const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return (lane & 16) ? static_cast<uint32_t>(p[0]) : static_cast<uint32_t>(p[1]);
}

__device__ __forceinline__ uint32_t xor32_u32(uint32_t v, int lane) {
  const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (lane & 32) ? static_cast<uint32_t>(p[0]) : static_cast<uint32_t>(p[1]);
}

// The LL largest of this lane's sorted list and its partner's, sorted.
template <int LL>
__device__ __forceinline__ void merge_rows(uint32_t (&a)[LL], int lane, bool far) {
  uint32_t p[LL];
#pragma unroll
  for (int i = 0; i < LL; ++i) p[i] = far ? xor32_u32(a[LL - 1 - i], lane) : xor16_u32(a[LL - 1 - i], lane);
#pragma unroll
  for (int i = 0; i < LL; ++i) a[i] = max(a[i], p[i]);
  bitonic_desc<LL>(a);
}

// The k (<= LL) largest logits of 16 staged rows of a tile of 4 NV columns, by one wave:
// lane 16 q + r holds columns q NV .. + NV - 1 of row r (16 consecutive lanes read 16 rows
// 4 banks apart, without conflicts).  so: the wave's first row (rows ld floats apart, ld a
// multiple of 4 with ld % 64 == 4); row0: its index; n0: the tile's first column.  Writes
// candidate t of (row, tile) to cand[(row n_tiles + tile) k + t], in descending order, 0
// where the tile holds fewer than k.  Columns past the vocabulary become NaN, which
// neither reaches a maximum nor compares.
template <int NV, int LL>
__device__ __forceinline__ void lm_select_quad(float* so, int ld, int row0, int n0, int vocab, int k, int n,
                                               uint64_t* __restrict__ cand, int n_tiles, int tile) {
  constexpr int CH = NV / 8;   // columns per chunk
  constexpr int HMAX = LL;            // logits a lane may contribute to the row's list
  constexpr int CAP = 2 * NV - 2;     // keys that fit the row, four of them padding
  static_assert(NV % 32 == 0, "hit words");
  const int lane = threadIdx.x & 63, q = lane >> 4;
  float* row_s = so + (lane & 15) * ld;
  const float* mine = row_s + q * NV;
  const int col0 = n0 + q * NV;
  if (n0 + 4 * NV > vocab) {
    for (int e = max(0, vocab - col0); e < NV; ++e) row_s[q * NV + e] = __builtin_nanf("");
    lm_wave_sync();
  }
  float v[NV];
#pragma unroll
  for (int e = 0; e < NV; e += 4) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(mine + e);
    v[e] = x[0]; v[e + 1] = x[1]; v[e + 2] = x[2]; v[e + 3] = x[3];
  }
  uint32_t L[LL];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float m = -INFINITY;
#pragma unroll
    for (int e = 0; e < CH; e += 2) m = max3_f32(m, v[j * CH + e], v[j * CH + e + 1]);
    L[j] = lm_ord(m);
  }
#pragma unroll
  for (int j = 8; j < LL; ++j) L[j] = 0u;
  sort8_desc(L);
  merge_rows<LL>(L, lane, false);
  merge_rows<LL>(L, lane, true);
  uint32_t th = L[0];
#pragma unroll
  for (int j = 1; j < LL; ++j)
    if (j < k) th = L[j];
  float t0 = lm_ord_val(th);
  // the lane's columns that reach the bound, first column in the highest bit
  uint32_t hit[NV / 32];
  auto find_hits = [&](float t) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < NV / 32; ++w) {
      uint32_t m = 0;
#pragma unroll
      for (int e = 32 * w; e < 32 * w + 32; e += 4) push4_ge_f32(m, v[e], v[e + 1], v[e + 2], v[e + 3], t);
      hit[w] = m;
      c += __popc(m);
    }
    return c;
  };
  int cnt = find_hits(t0);
  auto pair_sums = [&](int x, int& x1, int& x2) {  // counts of lanes q ^ 1 and of the other pair
    x1 = static_cast<int>(xor16_u32(static_cast<uint32_t>(x), lane));
    x2 = static_cast<int>(xor32_u32(static_cast<uint32_t>(x + x1), lane));
    return x + x1 + x2;
  };
  int c1, c2;
  int c = pair_sums(cnt, c1, c2);
  const int row = row0 + (lane & 15);
  uint64_t* dst = cand + (static_cast<int64_t>(row) * n_tiles + tile) * k;
  // whether the hits of the lane's row fit the list: at most HMAX a lane, CAP - 4 a row
  auto row_fits = [&](int mine_cnt, int row_cnt) {
    int o1, o2;
    return pair_sums(mine_cnt > HMAX ? 1 : 0, o1, o2) == 0 && row_cnt <= CAP - 4;
  };
  bool fits = row_fits(cnt, c);
  if (__ballot(!fits) != 0ull) {
    // too many for the list (a tile with few valid columns, logits in one lane, equal
    // logits): search a closer bound, between this one and the maximum, that k logits still
    // reach and the list holds (all rows of the wave together), or the k-th largest logit
    // itself; of that, take the logits above it and of those equal to it the lowest ids that
    // the k slots leave
    uint32_t lo = th, hi = fits ? th : L[0];
    while (__ballot(lo < hi) != 0ull) {
      const uint32_t mid = lo + ((hi - lo + 1) >> 1);
      const int m = find_hits(lm_ord_val(mid));
      const int got = pair_sums(m, c1, c2);
      const bool ok = row_fits(m, got);
      if (lo < hi) {
        if (got >= k) lo = mid;
        if (got < k) hi = mid - 1;
        if (got >= k && ok) hi = lo;
      }
    }
    t0 = lm_ord_val(lo);
    cnt = find_hits(t0);
    c = pair_sums(cnt, c1, c2);
    fits = row_fits(cnt, c);
    if (__ballot(!fits) != 0ull) {
      uint32_t eq[NV / 32];
      int ngt = 0, neq = 0;
#pragma unroll
      for (int w = 0; w < NV / 32; ++w) {
        uint32_t m = 0;
#pragma unroll
        for (int e = 32 * w; e < 32 * w + 32; e += 4) push4_eq_f32(m, v[e], v[e + 1], v[e + 2], v[e + 3], t0);
        eq[w] = fits ? 0u : m;
        hit[w] &= ~eq[w];
        neq += __popc(eq[w]);
        ngt += __popc(hit[w]);
      }
      int e1, e2;
      pair_sums(ngt, e1, e2);
      const int need = k - (ngt + e1 + e2);
      pair_sums(neq, e1, e2);
      int take = min(max(need - (((q & 1) ? e1 : 0) + ((q & 2) ? e2 : 0)), 0), neq);
      cnt = ngt + take;
#pragma unroll
      for (int w = 0; w < NV / 32; ++w)
        for (; take > 0 && eq[w] != 0u; --take) {
          const uint32_t top = 0x80000000u >> __clz(eq[w]);
          hit[w] |= top;
          eq[w] &= ~top;
        }
      c = pair_sums(cnt, c1, c2);
    }
  }
  int pos = ((q & 1) ? c1 : 0) + ((q & 2) ? c2 : 0);
  uint64_t key[HMAX];
#pragma unroll
  for (int t = 0; t < HMAX; ++t) {
    int e = __clz(hit[0]);
    if (hit[0] != 0u) {
      hit[0] &= ~(0x80000000u >> e);
    } else if constexpr (NV == 64) {
      const int e1 = __clz(hit[1]);
      e = 32 + e1;
      if (hit[1] != 0u) hit[1] &= ~(0x80000000u >> e1);
    }
    e = min(e, NV - 1);
    key[t] = lm_key(mine[e], col0 + e);
  }
  lm_wave_sync();  // every value is read before the list overwrites the row
  uint64_t* list = reinterpret_cast<uint64_t*>(row_s);
#pragma unroll
  for (int t = 0; t < HMAX; ++t)
    if (t < cnt) list[pos + t] = key[t];
  list[c + q] = 0ull;  // the ranking reads four at a time
  lm_wave_sync();
  // every lane ranks its own hits, four at a time while some lane has that many
#pragma unroll
  for (int t0 = 0; t0 < HMAX; t0 += 4) {
    if (__ballot(cnt > t0) == 0ull) break;
    int rk[4] = {0, 0, 0, 0};
    for (int u = 0; u < c; u += 4) {
      const u64x2 y0 = *reinterpret_cast<const u64x2*>(list + u);
      const u64x2 y1 = *reinterpret_cast<const u64x2*>(list + u + 2);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        rk[t] += (y0[0] > key[t0 + t] ? 1 : 0) + (y0[1] > key[t0 + t] ? 1 : 0) +
                 (y1[0] > key[t0 + t] ? 1 : 0) + (y1[1] > key[t0 + t] ? 1 : 0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t0 + t < cnt && rk[t] < k && row < n) dst[rk[t]] = key[t0 + t];
  }
  for (int t = c + q; t < k; t += 4)
    if (row < n) dst[t] = 0ull;
}

// ---- logits GEMM + per-tile candidates --------------------------------------------

template <typename T, int BM>
__global__ __launch_bounds__(256) void lm_kernel(LmMap tm, int n, const T* __restrict__ h, int d,
                                                 const T* __restrict__ W, int vocab, int k,
                                                 uint64_t* __restrict__ cand) {
  using C = LmCfg<T, BM>;
  // the pipeline's stages, then the whole tile of fp32 logits
  constexpr int kTileBytes = C::BM * C::SLD * 4;
  constexpr int kSmem = C::SMEM_BYTES > kTileBytes ? C::SMEM_BYTES : kTileBytes;
  static_assert(kSmem <= 160 * 1024, "LDS");
  __shared__ __align__(16) unsigned char smem[kSmem];
  int tr, tc;
  if (!tm.map(tr, tc)) return;
  const int m0 = tr * C::BM, n0 = tc * C::BN;
  f32x4 acc[C::TM][C::TN];
  gemm_mainloop<C>(acc, h, d, n, W, d, vocab, d, m0, n0, smem);

  // stage the whole tile in LDS (the accumulators are then dead), then select, 16 rows a wave
  float* so = reinterpret_cast<float*>(smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        so[(wm * C::SROWS + i * 16 + 4 * (lane >> 4) + v) * C::SLD + wn * C::TN * 16 + j * 16 +
           (lane & 15)] = acc[i][j][v];
  __syncthreads();
  for (int r0 = 16 * wave; r0 < C::BM; r0 += 64) {
    if (k <= 8)
      lm_select_quad<32, 8>(so + r0 * C::SLD, C::SLD, m0 + r0, n0, vocab, k, n, cand, tm.cb, tc);
    else
      lm_select_quad<32, 16>(so + r0 * C::SLD, C::SLD, m0 + r0, n0, vocab, k, n, cand, tm.cb, tc);
  }
}

// The same in the ping-pong core's tiles (64 QM rows x 256 columns, bf16), one row half of
// the tile staged at a time; k candidates per row and 256 columns.
template <int QM>
__global__ __launch_bounds__(512, 2) void lm_pp_kernel(LmMap tm, int n, const bf16_t* __restrict__ h, int d,
                                                       const bf16_t* __restrict__ W, int vocab, int k,
                                                       uint64_t* __restrict__ cand) {
  using C = PpCfg<QM>;
  __shared__ __align__(16) unsigned char smem[C::SMEM_BYTES];
  int tr, tc;
  if (!tm.map(tr, tc)) return;
  const int m0 = tr * C::BM, n0 = tc * C::BN;
  typename C::Acc acc;
  pp_mainloop<C>(acc, h, d, n, W, d, vocab, d, m0, n0, smem);
  float* so = reinterpret_cast<float*>(smem);
  const int r0 = 16 * static_cast<int>(threadIdx.x >> 6);  // AH <= 128: at most 16 rows a wave
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    pp_stage<C>(acc, a, so);
    __syncthreads();
    const int m1 = m0 + a * C::AH + r0;
    if (r0 < C::AH && m1 < n) {  // uniform over the wave
      if (k <= 8)
        lm_select_quad<64, 8>(so + r0 * C::SLD, C::SLD, m1, n0, vocab, k, n, cand, tm.cb, tc);
      else
        lm_select_quad<64, 16>(so + r0 * C::SLD, C::SLD, m1, n0, vocab, k, n, cand, tm.cb, tc);
    }
    __syncthreads();
  }
}

// ---- merge of a row's candidates --------------------------------------------------

// One block per row.  Every thread keeps the KM largest of the keys it reads (a sorted
// register list, updated by compare-and-swap down the list; its loads are issued eight
// at a time so that their latencies overlap).  For k <= 8 (KM = 8) the lists are then
// merged by the butterfly of the logits kernel: within each 16-lane row, then the
// sixteen row winners of the block in wave 0.  For larger k every wave extracts its
// k largest in k rounds and wave 0 ranks the 4 k survivors by counting.
template <int KM>
__global__ __launch_bounds__(256) void lm_merge_kernel(int n_cand, int k,
                                                       const uint64_t* __restrict__ cand,
                                                       int32_t* __restrict__ idx_out,
                                                       float* __restrict__ logit_out) {
  __shared__ uint64_t sk[16 * KM];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = blockIdx.x;
  uint64_t l[KM];
#pragma unroll
  for (int j = 0; j < KM; ++j) l[j] = 0ull;
  const uint64_t* cr = cand + row * n_cand;
  constexpr int U = 8;
  for (int t0 = 0; t0 < n_cand; t0 += 256 * U) {
    uint64_t c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * 256 + static_cast<int>(threadIdx.x);
      c[u] = t < n_cand ? cr[t] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint64_t x = c[u];
#pragma unroll
      for (int j = 0; j < KM; ++j) {
        const uint64_t t = l[j];
        l[j] = umax64(t, x);
        x = t > x ? x : t;
      }
    }
  }
  if constexpr (KM == 8) {
#pragma unroll
    for (int sel = 0; sel < 4; ++sel) merge_step<8>(l, sel);
    if ((lane & 15) == 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) sk[(wave * 4 + (lane >> 4)) * 8 + j] = l[j];
    }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) l[j] = lane < 16 ? sk[lane * 8 + j] : 0ull;
#pragma unroll
    for (int sel = 0; sel < 4; ++sel) merge_step<8>(l, sel);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < k) {
          idx_out[row * k + q] = lm_key_id(l[q]);
          if (logit_out != nullptr) logit_out[row * k + q] = lm_key_val(l[q]);
        }
    }
  } else {
    for (int q = 0; q < k; ++q) {
      const uint64_t b = wave_max64(l[0]);
      if (lane == 0) sk[wave * KM + q] = b;
      if (l[0] == b) {
#pragma unroll
        for (int j = 0; j + 1 < KM; ++j) l[j] = l[j + 1];
        l[KM - 1] = 0ull;
      }
    }
    __syncthreads();
    if (wave != 0 || lane >= 4 * k) return;
    // rank among the 4 k survivors; equal keys (only 0) rank by position
    const uint64_t x = sk[(lane / k) * KM + lane % k];
    int rank = 0;
    for (int j = 0; j < 4 * k; ++j) {
      const uint64_t y = sk[(j / k) * KM + j % k];
      rank += (y > x) | ((y == x) & (j < lane));
    }
    if (rank < k) {
      idx_out[row * k + rank] = lm_key_id(x);
      if (logit_out != nullptr) logit_out[row * k + rank] = lm_key_val(x);
    }
  }
}

}  // namespace fovea
