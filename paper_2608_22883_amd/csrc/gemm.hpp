// MFMA GEMM for gfx950: acc[m, n] = sum_k A[m, k] * B[n, k], with an LDS-staged epilogue.
//
// A is a row-major activation [rows, K] (K contiguous); B is a row-major weight [N, K]
// (the nn.Linear layout).  Block tile BM x 128 run by 2 x 2 wave64s; each wave owns a
// TM x TN grid of 16x16 MFMA accumulators.  Rows past M and columns past N are clamped
// on load; the epilogue hands them to the caller's functor, which drops them.
//
// bf16 mainloop: global -> LDS by direct-to-LDS loads (no register staging), NST LDS
// stages, k-tile kt + NST - 1 in flight while the matrix cores work on tile kt, one
// barrier per k-step.  A k-tile row is 64 bf16 = 128 B = 8 chunks of 16 B, stored with
// chunk c of row r at slot c ^ ((r >> 1) & 7): the 16 rows read by one fragment load
// then fall on distinct bank groups.  A direct-to-LDS load writes lane L's 16 bytes at
// LDS base + 16 L, so the swizzle is applied by choosing which global chunk each lane
// fetches.  The wait before each barrier counts this thread's outstanding loads
// exactly (loads retire in issue order), so tiles further ahead stay in flight.
//
// fp32 mainloop: register-staged copy into a double-buffered, padded LDS tile
// (MFMA 16x16x4 f32).
//
// Epilogue: the accumulators go through LDS (fp32, one wave-row of the tile per pass),
// and each thread then owns 8 consecutive columns of a row, so stores and the loads of
// epilogue operands are 16-byte, row-contiguous.  The 16 threads of a row are 16
// consecutive lanes; a per-row value returned by the functor is summed over them.
//
// Tiles are mapped to XCDs (blocks are dispatched round-robin over the 8 XCDs): the
// tile grid is cut into an xr x xc grid of regions and region x runs on XCD x, so the
// blocks sharing an XCD's L2 share A rows and B columns.
#pragma once

#include <type_traits>
#include <utility>

#include "common.hpp"

namespace fovea {

typedef __attribute__((address_space(3))) void* lds_void_ptr;

template <typename T, int BM_, int NST_ = 4>
struct GemmCfg {
  static constexpr int BM = BM_, BN = 128, WM = 2, WN = 2;
  static constexpr int NT = WM * WN * kWave;
  static constexpr int TM = BM / WM / 16;
  static constexpr int TN = BN / WN / 16;
  static constexpr int VEC = Elem<T>::kPer16B;  // elements per 16-byte chunk
  static constexpr int BK = 8 * VEC;            // k-tile: 64 bf16 or 32 fp32
  static constexpr bool DMA = VEC == 8;         // bf16: direct-to-LDS pipeline
  static constexpr int NST = DMA ? NST_ : 2;
  // bf16 rows are 128 B (swizzled), fp32 rows padded by one chunk
  static constexpr int LDK = DMA ? BK : BK + VEC;
  static constexpr int STAGE_BYTES = (BM + BN) * LDK * static_cast<int>(sizeof(T));
  // direct-to-LDS loads per wave per k-tile (one load moves 8 rows)
  static constexpr int A_DMA = BM / 8 / 4;
  static constexpr int B_DMA = BN / 8 / 4;
  // fp32 register staging: 16-byte chunks per thread per k-tile
  static constexpr int A_CHUNKS = BM * 8 / NT;
  static constexpr int B_CHUNKS = BN * 8 / NT;
  // epilogue staging: one wave-row (TM * 16 rows) of fp32 with a 4-float pad
  static constexpr int SROWS = TM * 16;
  static constexpr int SLD = BN + 4;
  static constexpr int OUT_BYTES = SROWS * SLD * 4;
  static constexpr int PIPE_BYTES = NST * STAGE_BYTES;
  static constexpr int SMEM_BYTES = PIPE_BYTES > OUT_BYTES ? PIPE_BYTES : OUT_BYTES;
  static_assert(BM == 64 || BM == 128 || BM == 256, "block rows");
  static_assert(NST >= 2 && NST <= 5, "pipeline depth");
  static_assert(SMEM_BYTES <= 160 * 1024, "LDS");
};

// Position of a block's tile in the (row-block, column-block) grid; false for padding.
struct TileMap {
  int rb, cb;  // tiles along M and N
  int xr, xc;  // XCD regions along M and N (xr * xc == 8)
  __device__ __forceinline__ bool map(int& tr, int& tc) const {
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int rr = (rb + xr - 1) / xr, rc = (cb + xc - 1) / xc;
    const int lr = slot / rc, lc = slot % rc;
    tr = (xcd / xc) * rr + lr;
    tc = (xcd % xc) * rc + lc;
    return lr < rr && tr < rb && tc < cb;
  }
};

inline TileMap make_tile_map(int rb, int cb, double a_bytes, double b_bytes) {
  // region grid minimising the bytes pulled into the 8 L2s: xc copies of A, xr of B
  TileMap m{rb, cb, 8, 1};
  double best = -1.0;
  for (int xr = 1; xr <= 8; xr *= 2) {
    const int xc = 8 / xr;
    const double cost = xc * a_bytes + xr * b_bytes;
    if (best < 0.0 || cost < best) {
      best = cost;
      m.xr = xr;
      m.xc = xc;
    }
  }
  return m;
}

__host__ __device__ inline int tile_grid(const TileMap& m) {
  return 8 * ((m.rb + m.xr - 1) / m.xr) * ((m.cb + m.xc - 1) / m.xc);
}

// s_waitcnt on the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and
// 15:14, expcnt and lgkmcnt fields at their maxima, i.e. not waited on).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Wait until at most `ahead` k-tiles of direct-to-LDS loads (NI loads each) are still
// outstanding; ahead is clamped to MAXA (the pipeline's steady-state lead).
template <int NI, int MAXA>
__device__ __forceinline__ void wait_tiles(int ahead) {
  if constexpr (MAXA <= 0) {
    wait_vmcnt<0>();
  } else {
    if (ahead >= MAXA)
      wait_vmcnt<MAXA * NI>();
    else
      wait_tiles<NI, MAXA - 1>(ahead);
  }
}

// Workgroup barrier without a memory fence: a fence would also wait for the
// direct-to-LDS loads still in flight.  The compiler barriers keep LDS accesses on
// their side of it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <class C>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[C::TM][C::TN]) {
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// bf16 mainloop (direct-to-LDS pipeline).  A: [M, K] row-major with leading dim lda.
template <class C>
__device__ __forceinline__ void gemm_mainloop_dma(f32x4 (&acc)[C::TM][C::TN],
                                                  const bf16_t* __restrict__ A, int64_t lda, int M,
                                                  const bf16_t* __restrict__ Bw, int64_t ldb, int N,
                                                  int K, int m0, int n0, unsigned char* smem) {
  constexpr int TM = C::TM, TN = C::TN, NST = C::NST;
  constexpr int NI = C::A_DMA + C::B_DMA;
  constexpr int NH = TM + TN;  // fragments per 32-wide k half
  const int lane = threadIdx.x & 63;
  // the wave index is uniform: derived addresses (the direct-to-LDS destinations above
  // all) stay in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  zero_acc<C>(acc);

  // sources and LDS row offsets of this thread's direct-to-LDS loads
  const bf16_t* ga[C::A_DMA];
  const bf16_t* gb[C::B_DMA];
  int da[C::A_DMA], db[C::B_DMA];
#pragma unroll
  for (int j = 0; j < C::A_DMA; ++j) {
    const int r0 = (wave * C::A_DMA + j) * 8;
    const int row = r0 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    ga[j] = A + static_cast<int64_t>(min(m0 + row, M - 1)) * lda + c * 8;
    da[j] = r0 * 128;
  }
#pragma unroll
  for (int j = 0; j < C::B_DMA; ++j) {
    const int r0 = (wave * C::B_DMA + j) * 8;
    const int row = r0 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    gb[j] = Bw + static_cast<int64_t>(min(n0 + row, N - 1)) * ldb + c * 8;
    db[j] = (C::BM + r0) * 128;
  }
  // fragment byte offsets (within a stage) for the two 32-wide k halves of a tile:
  // lane reads chunk 4 h + lane / 16 of row (.. + lane % 16); the swizzle term is the
  // same for all 16-row blocks of the lane
  const int arow = wm * TM * 16 + (lane & 15);
  const int brow = C::BM + wn * TN * 16 + (lane & 15);
  int fa[2], fb[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    fa[h] = arow * 128 + (((4 * h + (lane >> 4)) ^ ((arow >> 1) & 7)) << 4);
    fb[h] = brow * 128 + (((4 * h + (lane >> 4)) ^ ((brow >> 1) & 7)) << 4);
  }
  const int nk = K / C::BK;
  // fragment r (0 .. NH - 1) of half h of the tile in stage st, in the order the i-major
  // MFMAs first use them: A0, B0 .. B(TN-1), A1 .. A(TM-1)
  auto read_frag = [&](const unsigned char* st, int h, int r, bf16x8 (&af)[TM], bf16x8 (&bf)[TN]) {
    if (r == 0)
      af[0] = *reinterpret_cast<const bf16x8*>(st + fa[h]);
    else if (r <= TN)
      bf[r - 1] = *reinterpret_cast<const bf16x8*>(st + fb[h] + (r - 1) * 16 * 128);
    else
      af[r - TN] = *reinterpret_cast<const bf16x8*>(st + fa[h] + (r - TN) * 16 * 128);
  };
  // load q (0 .. NI - 1) of tile kt into its stage
  auto issue_one = [&](int kt, int q) {
    unsigned char* sn = smem + (kt % NST) * C::STAGE_BYTES;
    const int k0 = kt * C::BK;
    if (q < C::A_DMA)
      __builtin_amdgcn_global_load_lds(ga[q] + k0, (lds_void_ptr)(sn + da[q]), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds(gb[q - C::A_DMA] + k0, (lds_void_ptr)(sn + db[q - C::A_DMA]), 16, 0, 0);
  };
  // Step kt, with the first k half of tile kt already in registers (set P):
  //   1. its MFMAs, each followed by one read of the tile's second half and then by one
  //      load of tile kt + NST - 1 (into the stage tile kt - 1 used);
  //   2. this wave's reads done, its loads of tile kt + 1 done, then the barrier: tile
  //      kt + 1 is visible and every wave has finished reading stage kt;
  //   3. the second half's MFMAs, each followed by one read of tile kt + 1's first half
  //      (set 1 - P), so that read latency hides behind matrix work.
  // Loads are issued for every step (past the last tile the last tile is loaded again
  // into a stage nobody reads), so the wait is a fixed count of this thread's loads
  // (they retire in issue order).  After the last step the reads of step 3 touch a stage
  // whose contents are not used.  The compiler barriers keep each access in its slot.
  bf16x8 af0[2][TM], bf0[2][TN], af1[TM], bf1[TN];
  auto step = [&](int kt, auto P) {
    constexpr int p = decltype(P)::value;
    const unsigned char* st = smem + (kt % NST) * C::STAGE_BYTES;
    const unsigned char* sn = smem + ((kt + 1) % NST) * C::STAGE_BYTES;
    const int knext = min(kt + NST - 1, nk - 1);
#pragma unroll
    for (int m = 0; m < TM * TN; ++m) {
      mfma_bf16_16x16x32_acc(acc[m / TN][m % TN], af0[p][m / TN], bf0[p][m % TN]);
      if (m < NH)
        read_frag(st, 1, m, af1, bf1);
      else if (m - NH < NI)
        issue_one(knext, m - NH);
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int q = TM * TN - NH; q < NI; ++q) issue_one(knext, q);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of the stage done
    wait_vmcnt<(NST - 2) * NI>();
    lds_barrier();
#pragma unroll
    for (int m = 0; m < TM * TN; ++m) {
      mfma_bf16_16x16x32_acc(acc[m / TN][m % TN], af1[m / TN], bf1[m % TN]);
      if (m < NH) read_frag(sn, 0, m, af0[1 - p], bf0[1 - p]);
      asm volatile("" ::: "memory");
    }
  };
  // prologue: tiles 0 .. NST - 2, each tile's loads together (in issue order)
#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
#pragma unroll
    for (int q = 0; q < NI; ++q) issue_one(min(s, nk - 1), q);
  wait_vmcnt<(NST - 2) * NI>();
  lds_barrier();
#pragma unroll
  for (int r = 0; r < NH; ++r) read_frag(smem, 0, r, af0[0], bf0[0]);
  asm volatile("" ::: "memory");
  mfma_accumulators_ready(acc);
  int kt = 0;
  for (; kt + 1 < nk; kt += 2) {
    step(kt, std::integral_constant<int, 0>());
    step(kt + 1, std::integral_constant<int, 1>());
  }
  if (kt < nk) {
    mfma_accumulators_ready(acc);
    step(kt, std::integral_constant<int, 0>());
  }
  // the extra loads of the last steps land before the LDS is reused
  wait_vmcnt<0>();
  mfma_results_ready();
  lds_barrier();
}

// fp32 mainloop: register-staged, double-buffered LDS.
template <class C>
__device__ __forceinline__ void gemm_mainloop_f32(f32x4 (&acc)[C::TM][C::TN],
                                                  const float* __restrict__ A, int64_t lda, int M,
                                                  const float* __restrict__ Bw, int64_t ldb, int N,
                                                  int K, int m0, int n0, unsigned char* smem_raw) {
  constexpr int TM = C::TM, TN = C::TN;
  float* smem = reinterpret_cast<float*>(smem_raw);
  constexpr int STAGE = (C::BM + C::BN) * C::LDK;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
  zero_acc<C>(acc);
  const float* ga[C::A_CHUNKS];
  const float* gb[C::B_CHUNKS];
  int la[C::A_CHUNKS], lb[C::B_CHUNKS];
#pragma unroll
  for (int j = 0; j < C::A_CHUNKS; ++j) {
    const int c = tid + j * C::NT;
    ga[j] = A + static_cast<int64_t>(min(m0 + (c >> 3), M - 1)) * lda + (c & 7) * 4;
    la[j] = (c >> 3) * C::LDK + (c & 7) * 4;
  }
#pragma unroll
  for (int j = 0; j < C::B_CHUNKS; ++j) {
    const int c = tid + j * C::NT;
    gb[j] = Bw + static_cast<int64_t>(min(n0 + (c >> 3), N - 1)) * ldb + (c & 7) * 4;
    lb[j] = (C::BM + (c >> 3)) * C::LDK + (c & 7) * 4;
  }
  const int aoff = (wm * TM * 16 + (lane & 15)) * C::LDK + (lane >> 4);
  const int boff = (C::BM + wn * TN * 16 + (lane & 15)) * C::LDK + (lane >> 4);
  const int nk = K / C::BK;
  u32x4 ra[C::A_CHUNKS], rb[C::B_CHUNKS];
#pragma unroll
  for (int j = 0; j < C::A_CHUNKS; ++j) ra[j] = *reinterpret_cast<const u32x4*>(ga[j]);
#pragma unroll
  for (int j = 0; j < C::B_CHUNKS; ++j) rb[j] = *reinterpret_cast<const u32x4*>(gb[j]);
  for (int kt = 0; kt < nk; ++kt) {
    float* st = smem + (kt & 1) * STAGE;
#pragma unroll
    for (int j = 0; j < C::A_CHUNKS; ++j) *reinterpret_cast<u32x4*>(st + la[j]) = ra[j];
#pragma unroll
    for (int j = 0; j < C::B_CHUNKS; ++j) *reinterpret_cast<u32x4*>(st + lb[j]) = rb[j];
    const int k1 = min(kt + 1, nk - 1) * C::BK;
#pragma unroll
    for (int j = 0; j < C::A_CHUNKS; ++j) ra[j] = *reinterpret_cast<const u32x4*>(ga[j] + k1);
#pragma unroll
    for (int j = 0; j < C::B_CHUNKS; ++j) rb[j] = *reinterpret_cast<const u32x4*>(gb[j] + k1);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < C::BK; kk += 4) {
      float af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = st[aoff + i * 16 * C::LDK + kk];
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = st[boff + j * 16 * C::LDK + kk];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_f32_16x16x4(af[i], bf[j], acc[i][j]);
    }
  }
  __syncthreads();
}

template <class C, typename T>
__device__ __forceinline__ void gemm_mainloop(f32x4 (&acc)[C::TM][C::TN], const T* A, int64_t lda,
                                              int M, const T* Bw, int64_t ldb, int N, int K, int m0,
                                              int n0, unsigned char* smem) {
  if constexpr (C::DMA)
    gemm_mainloop_dma<C>(acc, A, lda, M, Bw, ldb, N, K, m0, n0, smem);
  else
    gemm_mainloop_f32<C>(acc, A, lda, M, Bw, ldb, N, K, m0, n0, smem);
}

// LDS-staged epilogue.  f(row, col0, v) sees the 8 accumulators of columns
// col0 .. col0 + 7 of `row` (rows and columns past the matrix included: f drops them)
// and returns a per-row contribution; fr(row, sum) receives the sum of the
// contributions over the tile's 128 columns (lane order fixed, so deterministic).
// fix(row, col0, so), if given, may first change 8 columns of a row where they are staged (it
// is called for each group of 8 when some output of the tile is NaN).
// Must be reached by every thread of the block.
struct NoFix {};

template <class C, class F, class FR, class FX = NoFix>
__device__ __forceinline__ void gemm_epilogue(const f32x4 (&acc)[C::TM][C::TN],
                                              unsigned char* smem, int m0, int n0, F&& f,
                                              FR&& fr, FX&& fix = FX()) {
  constexpr bool FIX = !std::is_same<typename std::decay<FX>::type, NoFix>::value;
  int* flag = reinterpret_cast<int*>(smem + C::OUT_BYTES + 1024);  // of the WN staged waves
  static_assert(!FIX || C::SMEM_BYTES >= C::OUT_BYTES + 1024 + 16 && C::WN == 2, "flags");
  float* so = reinterpret_cast<float*>(smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
  constexpr int GROUPS = C::SROWS * (C::BN / 8);
  static_assert(GROUPS % C::NT == 0 && C::BN / 8 == 16, "epilogue mapping");
#pragma unroll
  for (int p = 0; p < C::WM; ++p) {
    if (wm == p) {
      float t[4] = {0.f, 0.f, 0.f, 0.f};  // NaN as soon as one output of the wave is NaN (or infinite)
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            so[(i * 16 + 4 * (lane >> 4) + v) * C::SLD + wn * C::TN * 16 + j * 16 + (lane & 15)] =
                acc[i][j][v];
            if (FIX) t[v] = fmaf(acc[i][j][v], 0.f, t[v]);
          }
      if (FIX) {
        const float sum = (t[0] + t[1]) + (t[2] + t[3]);
        const bool any = __ballot(sum != sum) != 0ull;
        if (lane == 0) flag[wn] = any ? 1 : 0;
      }
    }
    __syncthreads();
    if constexpr (FIX) {
      if (__builtin_expect(flag[0] | flag[1], 0))
#pragma unroll 1
        for (int g = static_cast<int>(threadIdx.x); g < GROUPS; g += C::NT)
          fix(m0 + p * C::SROWS + (g >> 4), n0 + (g & 15) * 8, so + (g >> 4) * C::SLD + (g & 15) * 8);
    }
#pragma unroll
    for (int g0 = 0; g0 < GROUPS; g0 += C::NT) {
      const int g = g0 + static_cast<int>(threadIdx.x);
      const int r = g >> 4, c8 = g & 15;
      const f32x4 lo = *reinterpret_cast<const f32x4*>(so + r * C::SLD + c8 * 8);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(so + r * C::SLD + c8 * 8 + 4);
      const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      const int row = m0 + p * C::SROWS + r;
      float s;
      // functors that take the group index gi (compile-time after unrolling) can hold
      // operands prefetched per group (epilogue_group)
      if constexpr (std::is_invocable_v<F, int, int, const float(&)[8], int>)
        s = f(row, n0 + c8 * 8, v, p * (GROUPS / C::NT) + g0 / C::NT);
      else
        s = f(row, n0 + c8 * 8, v);
      s = sum16(s);
      if ((lane & 15) == 0) fr(row, s);
    }
    __syncthreads();
  }
}

// Row and first column of epilogue group gi of this thread (gemm_epilogue's mapping):
// groups per thread C::WM * C::SROWS * 16 / C::NT.
template <class C>
__device__ __forceinline__ void epilogue_group(int gi, int m0, int n0, int& row, int& col0) {
  constexpr int PER = C::SROWS * 16 / C::NT;
  const int p = gi / PER, g = (gi % PER) * C::NT + static_cast<int>(threadIdx.x);
  row = m0 + p * C::SROWS + (g >> 4);
  col0 = n0 + (g & 15) * 8;
}

// ---------------------------------------------------------------------------------
// Ping-pong GEMM for grids of many tiles (bf16): 8 waves on a (64 QM) x 256 tile.
//
// Eight waves as 2 (rows) x 4 (columns); each owns QM x 2 accumulators of 16x16 in each
// quadrant of the tile (row half x column half).  A k-tile (64 wide, the same swizzled
// 128-byte rows as above) is four half tiles A0, A1, B0, B1; two k-tiles fill the LDS and
// a half is refilled with k-tile + 2 as soon as every wave has read it.  One k-tile takes
// four phases (quadrants 00, 01, 11, 10), each a read slot (fragments from LDS, loads of
// a half tile issued) and a multiply slot, a barrier after each.  Waves w and w + 4 share
// a SIMD and run one slot apart, so that one of them multiplies while the other reads:
// with one wave per SIMD the reads, waits and barriers of the core above are not hidden.
//   Bound by the matrix cores: a k-tile of 256 x 256 asks 2048 MFMA cycles, 64 KB of
// direct-to-LDS loads (about 1400 cycles) and 192 KB of LDS reads (about 1540).  Measured
// (plain fp32 stores, back to back): 4096^3 99.9 us, 1376 TFLOP/s, against 139 us (128 x
// 128, 4 waves) and 117 us (256 x 128, 4 waves).  A k-tile takes 1.18, 1.06, 0.83 us at
// QM = 4, 3, 2: the slots of smaller tiles are bound by their reads and barriers.
// ---------------------------------------------------------------------------------
template <int QM_>
struct PpCfg {
  static constexpr int QM = QM_, QN = 2, WN = 4, NT = 512;
  static constexpr int BM = 64 * QM, BN = 256;
  static constexpr int AH = BM / 2, BH = BN / 2;  // rows of a half tile
  static constexpr int A_BYTES = AH * 128, B_BYTES = BH * 128;
  static constexpr int STAGE_BYTES = 2 * (A_BYTES + B_BYTES);
  // direct-to-LDS loads per wave and half tile (8 rows each; where the rows do not divide,
  // the last load is repeated so that every wave counts the same number)
  static constexpr int NA = (AH / 8 + 7) / 8, NB = BH / 8 / 8;
  // epilogue staging: one row half of the tile in fp32 with a 4-float pad
  static constexpr int SLD = BN + 4;
  static constexpr int OUT_BYTES = AH * SLD * 4;
  static constexpr int PIPE_BYTES = 2 * STAGE_BYTES;
  static constexpr int SMEM_BYTES = PIPE_BYTES > OUT_BYTES ? PIPE_BYTES : OUT_BYTES;
  using Acc = f32x4[2][2][QM][QN];  // [row half][column half][row block][column block]
  static_assert(QM >= 2 && QM <= 4 && SMEM_BYTES <= 160 * 1024, "tile");
  static constexpr int off_a(int s, int h) { return s * STAGE_BYTES + h * A_BYTES; }
  static constexpr int off_b(int s, int h) { return s * STAGE_BYTES + 2 * A_BYTES + h * B_BYTES; }
};

// One direct-to-LDS load: lane L's 16 bytes at src go to dst + 16 L (dst uniform).
__device__ __forceinline__ void load_lds16(const bf16_t* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds(src, (lds_void_ptr)dst, 16, 0, 0);
}

template <int P>
__device__ __forceinline__ void wave_prio() {
  __builtin_amdgcn_s_setprio(P);
}

// Ends a read slot: at most VM loads still out, this wave's LDS reads done, barrier.
template <int VM>
__device__ __forceinline__ void pp_end_read() {
  if constexpr (VM < 63) wait_vmcnt<VM>();
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  lds_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void pp_end_mma() {
  __builtin_amdgcn_sched_barrier(0);
  lds_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

template <class C>
__device__ __forceinline__ void pp_mainloop(typename C::Acc& acc, const bf16_t* __restrict__ A,
                                            int64_t lda, int M, const bf16_t* __restrict__ Bw, int64_t ldb,
                                            int N, int K, int m0, int n0, unsigned char* smem) {
  constexpr int QM = C::QM, QN = C::QN, NA = C::NA, NB = C::NB;
  constexpr int NT1 = 2 * NA + 2 * NB;  // loads of one k-tile per wave
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave & 1, wn = wave >> 1;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < QM; ++i)
#pragma unroll
        for (int j = 0; j < QN; ++j) acc[a][b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bf16_t* ga[2][NA];
  const bf16_t* gb[2][NB];
  int da[NA], db[NB];
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int r0 = min(wave + 8 * u, C::AH / 8 - 1) * 8;
    const int row = r0 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    da[u] = r0 * 128;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      ga[h][u] = A + static_cast<int64_t>(min(m0 + h * C::AH + row, M - 1)) * lda + c * 8;
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int r0 = (wave + 8 * u) * 8;
    const int row = r0 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    db[u] = r0 * 128;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      gb[h][u] = Bw + static_cast<int64_t>(min(n0 + h * C::BH + row, N - 1)) * ldb + c * 8;
  }
  const int nk = K / 64;
  const int arow = wm * QM * 16 + (lane & 15), brow = wn * QN * 16 + (lane & 15);
  int fa[2], fb[2];
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    fa[kh] = arow * 128 + (((4 * kh + (lane >> 4)) ^ ((arow >> 1) & 7)) << 4);
    fb[kh] = brow * 128 + (((4 * kh + (lane >> 4)) ^ ((brow >> 1) & 7)) << 4);
  }
  // loads past the last k-tile repeat it (into a half that nobody reads any more), so that
  // the waits are fixed counts
  auto load_a = [&](int kt, int s, int h) {
    const int k0 = min(kt, nk - 1) * 64;
#pragma unroll
    for (int u = 0; u < NA; ++u)
      load_lds16(ga[h][u] + k0, smem + C::off_a(s, h) + da[u]);
  };
  auto load_b = [&](int kt, int s, int h) {
    const int k0 = min(kt, nk - 1) * 64;
#pragma unroll
    for (int u = 0; u < NB; ++u)
      load_lds16(gb[h][u] + k0, smem + C::off_b(s, h) + db[u]);
  };
  bf16x8 af[2][QM], bf[2][2][QN];  // [k half][row block], [column half][k half][column block]
  auto read_a = [&](int s, int h) {
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int i = 0; i < QM; ++i)
        af[kh][i] = *reinterpret_cast<const bf16x8*>(smem + C::off_a(s, h) + fa[kh] + i * 16 * 128);
  };
  auto read_b = [&](int s, int h) {
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int j = 0; j < QN; ++j)
        bf[h][kh][j] = *reinterpret_cast<const bf16x8*>(smem + C::off_b(s, h) + fb[kh] + j * 16 * 128);
  };
  auto mma = [&](int a, int b) {
    wave_prio<1>();
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int i = 0; i < QM; ++i)
#pragma unroll
        for (int j = 0; j < QN; ++j) mfma_bf16_16x16x32_acc(acc[a][b][i][j], af[kh][i], bf[b][kh][j]);
    wave_prio<0>();
  };
  // k-tile kt from stage s.  A wave waits, one slot or more before the slot that reads a
  // half, until its own loads of that half are done; the barriers between make every
  // wave's share visible.  Loads are issued in the order A0 B0, B1, A1.
  auto tile = [&](int kt, auto S) {
    constexpr int s = decltype(S)::value;
    read_a(s, 0);
    read_b(s, 0);
    pp_end_read<NA + NT1>();  // B1 of kt is here
    mma(0, 0);
    pp_end_mma();
    read_b(s, 1);
    load_a(kt + 2, s, 0);
    load_b(kt + 2, s, 0);
    pp_end_read<NT1 + NA + NB>();  // A1 of kt
    mma(0, 1);
    pp_end_mma();
    read_a(s, 1);
    load_b(kt + 2, s, 1);
    pp_end_read<63>();
    mma(1, 1);
    pp_end_mma();
    load_a(kt + 2, s, 1);
    pp_end_read<NB + NA + NT1>();  // A0 and B0 of kt + 1
    mma(1, 0);
    pp_end_mma();
  };
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    load_a(t, t, 0);
    load_b(t, t, 0);
    load_b(t, t, 1);
    load_a(t, t, 1);
  }
  wait_vmcnt<NB + NA + NT1>();
  lds_barrier();
  if (wave >= 4) lds_barrier();  // the second wave of each SIMD runs one slot behind
  auto ready = [&]() {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) mfma_accumulators_ready(acc[a][b]);
  };
  ready();
  int kt = 0;
  for (; kt + 1 < nk; kt += 2) {
    tile(kt, std::integral_constant<int, 0>());
    tile(kt + 1, std::integral_constant<int, 1>());
  }
  if (kt < nk) {
    ready();
    tile(kt, std::integral_constant<int, 0>());
  }
  if (wave < 4) lds_barrier();
  wait_vmcnt<0>();  // the repeated loads land before the LDS is reused
  mfma_results_ready();
  lds_barrier();
}

// Row half a of the accumulators into the staging area (fp32, rows SLD apart).
template <class C>
__device__ __forceinline__ void pp_stage(const typename C::Acc& acc, int a, float* so) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < C::QM; ++i)
#pragma unroll
      for (int j = 0; j < C::QN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          so[(wm * C::QM * 16 + i * 16 + 4 * (lane >> 4) + v) * C::SLD + b * C::BH + wn * C::QN * 16 +
             j * 16 + (lane & 15)] = acc[a][b][i][j][v];
}

// LDS-staged epilogue: f(row, col0, v) sees 8 consecutive columns of a row, as in
// gemm_epilogue (without row sums); 16 consecutive lanes hold 128 columns of a row.
template <class C, class F>
__device__ __forceinline__ void pp_epilogue(const typename C::Acc& acc, unsigned char* smem,
                                            int m0, int n0, F&& f) {
  float* so = reinterpret_cast<float*>(smem);
  constexpr int GROUPS = C::AH * (C::BN / 8);
  static_assert(GROUPS % C::NT == 0, "epilogue mapping");
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    pp_stage<C>(acc, a, so);
    __syncthreads();
#pragma unroll
    for (int g0 = 0; g0 < GROUPS; g0 += C::NT) {
      const int g = g0 + static_cast<int>(threadIdx.x);
      const int r = g / (C::BN / 8), c8 = g % (C::BN / 8);
      float v[8];
      load8(so + r * C::SLD + c8 * 8, v);
      f(m0 + a * C::AH + r, n0 + c8 * 8, v);
    }
    __syncthreads();
  }
}

// bf16 tiles of a product that has no split along K: the core above with 4 waves (128 columns)
// or the ping-pong core (256).  cost: a k-tile of 64, in 10 ns, measured on memory builds and
// LM heads of 126 + 269 sizes (300 to 65536 rows; 40 to 1920 rows over vocabularies of 1000 to
// 152064), where the tile with the smallest rounds x cost is 1% from the fastest on average.
// A round is 32 tiles on the XCD that has most: 36 x 7 tiles in regions of 5 x 7 take two
// rounds, although they are fewer than 256 (4608 x 1792 x 3584: 104 us, 70 in 192-row tiles),
// and a few wide tiles leave compute units idle (200 x 8192 x 4096: 63 us, 32 in 64-row tiles).
struct BfTile {
  int rows, cols, cost;
};
constexpr BfTile kBfTiles[] = {{64, 128, 33}, {128, 128, 48}, {128, 256, 80}, {192, 256, 96}, {256, 256, 108}};

// The best of kBfTiles; per_xcd(rows, cols): tiles on the XCD that has most of them.
template <class F>
inline BfTile best_bf_tile(F&& per_xcd) {
  BfTile best = kBfTiles[0];
  int64_t best_cost = -1;
  for (const BfTile& t : kBfTiles) {
    const int64_t c = (static_cast<int64_t>(per_xcd(t.rows, t.cols)) + 31) / 32 * t.cost;
    if (best_cost < 0 || c < best_cost) {
      best_cost = c;
      best = t;
    }
  }
  return best;
}

// ---------------------------------------------------------------------------------
// GEMM over fp32 operands on the bf16 matrix cores.
//
// x = x0 + x1 (+ x2) with x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1).  Two
// planes leave 2^-16 |x| and take three products (00, 10, 01); three planes hold all 24
// bits of an operand of at least 2^-110 (below that the lower planes run into bf16's
// subnormals, and an operand keeps its bits down to 2^-133) and take the six products of
// weight 2^-16 or more (00, 01, 10, 11, 02, 20): what is left out is below fp32's own
// rounding, and the matrix cores round once per 32 products, so the sum is closer to 64 bits
// than fp32 MFMA's (1920 x 2048 x 4096: 1.0e-6 against 1.2e-6).
//   B comes as planes, [row][K / 32][plane][32]: 64 P bytes hold 32 k of a row in every
// plane, one LDS row of a k-tile, so that a loaded tile serves all products (three copies
// of K in one ordinary GEMM load and read half as much again).  A comes as planes too, or
// as fp32 rows whose fragments each wave splits in registers between the products, which
// costs neither a pass over A nor room for its planes.
//   128 (or 64) x 128 tiles, 2 x 2 waves.  Step kt multiplies the fragments of k-tile kt,
// all in registers, and between the products reads those of kt + 1 and loads k-tile
// kt + NST into the stage that kt left; one barrier per step.  Bound by the matrix cores:
// three planes 1920 x 2048 x 4096 147 us (1314 TFLOP/s of bf16 products) against 292 us
// on fp32 MFMA; two planes 87 us.
// ---------------------------------------------------------------------------------
template <int P_, int BM_, bool AF32_>
struct SplitCfg {
  static constexpr int P = P_, BM = BM_, BN = 128, WM = 2, WN = 2;
  static constexpr bool AF32 = AF32_;
  static constexpr int NT = WM * WN * kWave;
  static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static constexpr int CHA = AF32 ? 8 : 4 * P, CHB = 4 * P;  // 16-byte chunks of an LDS row (32 k)
  static constexpr int NST = BM == 128 && P == 3 ? 3 : 4;
  static constexpr int A_BYTES = BM * CHA * 16;
  static constexpr int STAGE_BYTES = A_BYTES + BN * CHB * 16;
  static constexpr int LA = BM * CHA / 64, LB = BN * CHB / 64;  // direct-to-LDS loads of a k-tile
  static constexpr int NI = (LA + LB) / 4;                      // per wave
  static constexpr int SROWS = TM * 16, SLD = BN + 4, OUT_BYTES = SROWS * SLD * 4;
  static constexpr int PIPE_BYTES = NST * STAGE_BYTES;
  static constexpr int SMEM_BYTES = PIPE_BYTES > OUT_BYTES ? PIPE_BYTES : OUT_BYTES;
  static_assert((P == 2 || P == 3) && (BM == 64 || BM == 128), "planes, rows");
  static_assert((LA + LB) % 4 == 0 && SMEM_BYTES <= 160 * 1024, "loads, LDS");
  // slot of chunk c in row r of CH chunks: 16 rows' reads of one chunk fall on distinct banks
  template <int CH>
  __device__ static int slot(int c, int r) {
    if constexpr (CH == 8) return c ^ ((r >> 1) & 7);
    const int s = c + ((r >> 2) & 3);
    return s >= CH ? s - CH : s;
  }
  template <int CH>
  __device__ static int chunk(int s, int r) {  // the chunk held by slot s of row r
    if constexpr (CH == 8) return s ^ ((r >> 1) & 7);
    const int c = s - ((r >> 2) & 3);
    return c < 0 ? c + CH : c;
  }
};

// Element offset of column k in a row of planes (plane 0; plane p is 32 p further).
template <int P>
__host__ __device__ __forceinline__ int64_t plane_col(int64_t k) {
  return (k >> 5) * (32 * P) + (k & 31);
}

// Two values into P packed planes.  The first plane saturates at the largest bf16, so that
// a finite value never becomes infinite.  An infinite one is (largest, infinity, NaN), whose
// products are NaN; the forward computes those again (plain_dot).
template <int P>
__device__ __forceinline__ void split_pair(float x, float y, uint32_t (&out)[P]) {
  constexpr float kBig = 3.3895313892515355e38f;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t w = p == 0 ? pack_bf16x2(__builtin_amdgcn_fmed3f(x, -kBig, kBig),
                                            __builtin_amdgcn_fmed3f(y, -kBig, kBig))
                              : pack_bf16x2(x, y);
    out[p] = w;
    if (p + 1 < P) {
      x -= __uint_as_float(w << 16);
      y -= __uint_as_float(w & 0xffff0000u);
    }
  }
}

// Eight consecutive columns k .. k + 7 (k a multiple of 8) of a row of planes.
template <int P>
__device__ __forceinline__ void store_planes8(bf16_t* row, int64_t k, const float (&x)[8]) {
  u32x4 w[P];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t o[P];
    split_pair<P>(x[2 * e], x[2 * e + 1], o);
#pragma unroll
    for (int p = 0; p < P; ++p) w[p][e] = o[p];
  }
#pragma unroll
  for (int p = 0; p < P; ++p) *reinterpret_cast<u32x4*>(row + plane_col<P>(k) + 32 * p) = w[p];
}

// f(integral_constant 0), .., f(integral_constant N - 1)
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}

template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>());
}

// acc = A B^T over the k-tiles [kt0, kt1) of 32 columns.  A: fp32 rows lda apart, or planes;
// B: planes, rows ldb elements apart.
template <class C, typename TA>
__device__ __forceinline__ void split_mainloop(f32x4 (&acc)[C::TM][C::TN], const TA* __restrict__ A,
                                               int64_t lda, int M, const bf16_t* __restrict__ Bw,
                                               int64_t ldb, int N, int kt0, int kt1, int m0, int n0,
                                               unsigned char* smem) {
  static_assert(std::is_same<TA, float>::value == C::AF32, "operand A");
  constexpr int P = C::P, TM = C::TM, TN = C::TN, NST = C::NST, NI = C::NI;
  constexpr int RA = C::AF32 ? 2 * TM : P * TM;        // LDS reads of A per step
  constexpr int NR = RA + P * TN;
  constexpr int NP = P == 2 ? 3 : 6;                   // products
  constexpr int PA[6] = {0, P == 2 ? 1 : 0, P == 2 ? 0 : 1, 1, 0, 2};
  constexpr int PB[6] = {0, P == 2 ? 0 : 1, P == 2 ? 1 : 0, 1, 2, 0};
  constexpr int NM = NP * TM * TN;                     // MFMAs per step
  constexpr int NO = NR + NI, OP = NO / NI;            // reads and loads of a step, one load in OP
  constexpr int SPREAD = NM - NM / 4;
  constexpr int NC = C::AF32 ? 4 * TM : 0;             // pairs per lane to split
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  zero_acc<C>(acc);
  const int nk = kt1 - kt0;
  constexpr int SA = C::AF32 ? 128 : 64 * P, SB = 64 * P;  // bytes of a row per k-tile
  const char* gp[NI];
  int dp[NI];
#pragma unroll
  for (int u = 0; u < NI; ++u) {
    const int j = wave * NI + u;  // uniform: the first LA loads are A's
    if (j < C::LA) {
      const int l = j * 64 + lane, row = l / C::CHA;
      const int c = C::template chunk<C::CHA>(l % C::CHA, row);
      gp[u] = reinterpret_cast<const char*>(A + static_cast<int64_t>(min(m0 + row, M - 1)) * lda) +
              static_cast<int64_t>(kt0) * SA + c * 16;
      dp[u] = j * 1024;
    } else {
      const int l = (j - C::LA) * 64 + lane, row = l / C::CHB;
      const int c = C::template chunk<C::CHB>(l % C::CHB, row);
      gp[u] = reinterpret_cast<const char*>(Bw + static_cast<int64_t>(min(n0 + row, N - 1)) * ldb) +
              static_cast<int64_t>(kt0) * SB + c * 16;
      dp[u] = j * 1024;
    }
  }
  static_assert(C::LA * 1024 == C::A_BYTES, "B follows A");
  int fa[C::AF32 ? 2 : P], fb[P];
  const int r = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int p = 0; p < (C::AF32 ? 2 : P); ++p) {
    const int c = C::AF32 ? 2 * kg + p : 4 * p + kg;
    fa[p] = ((wm * TM * 16 + r) * C::CHA + C::template slot<C::CHA>(c, r)) * 16;
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    fb[p] = C::A_BYTES + ((wn * TN * 16 + r) * C::CHB + C::template slot<C::CHB>(4 * p + kg, r)) * 16;
  auto issue = [&](int kt, int st, int u) {
    const int64_t step = (C::AF32 && wave * NI + u < C::LA) ? SA : SB;
    load_lds16(reinterpret_cast<const bf16_t*>(gp[u] + min(kt, nk - 1) * step), smem + st * C::STAGE_BYTES + dp[u]);
  };
  bf16x8 af[2][P][TM], bf[2][P][TN];
  f32x4 raw[C::AF32 ? TM : 1][2];
  // read f of a step: A's first, then B's plane by plane
  auto read_frag = [&](const unsigned char* sp, int f, bf16x8 (&a)[P][TM], bf16x8 (&b)[P][TN]) {
    if (f < RA) {
      if constexpr (C::AF32)
        raw[f / 2][f % 2] = *reinterpret_cast<const f32x4*>(sp + fa[f % 2] + (f / 2) * 16 * C::CHA * 16);
      else
        a[f / TM][f % TM] = *reinterpret_cast<const bf16x8*>(sp + fa[f / TM] + (f % TM) * 16 * C::CHA * 16);
    } else {
      const int g = f - RA;
      b[g / TN][g % TN] = *reinterpret_cast<const bf16x8*>(sp + fb[g / TN] + (g % TN) * 16 * C::CHB * 16);
    }
  };
  // pair c of the next k-tile's A fragments into planes
  auto split_frag = [&](int c, bf16x8 (&a)[P][TM]) {
    if constexpr (C::AF32) {
      const int i = c / 4, e = c % 4;
      uint32_t o[P];
      split_pair<P>(raw[i][e / 2][2 * (e % 2)], raw[i][e / 2][2 * (e % 2) + 1], o);
#pragma unroll
      for (int p = 0; p < P; ++p) {
        u32x4 t = __builtin_bit_cast(u32x4, a[p][i]);
        t[e] = o[p];
        a[p][i] = __builtin_bit_cast(bf16x8, t);
      }
    }
  };
  // the splits run in the second half of a step, when the reads of A have returned
  constexpr int C0 = NM / 2, CSTEP = NC > 0 ? (NM - C0) / NC : 1;
  int st = 0;  // stage of the k-tile being multiplied
  auto step = [&](int kt, auto S) {
    constexpr int set = decltype(S)::value;
    const int sn = st + 1 == NST ? 0 : st + 1;
    const unsigned char* sp = smem + sn * C::STAGE_BYTES;
    static_for<NM>([&](auto M_) {
      constexpr int m = decltype(M_)::value;
      constexpr int pr = m / (TM * TN), i = (m / TN) % TM, j = m % TN;
      mfma_bf16_16x16x32_acc(acc[i][j], af[set][PA[pr]][i], bf[set][PB[pr]][j]);
      // the reads and loads are spread evenly over the first SPREAD products (a read after
      // every product would ask more than the LDS delivers)
      constexpr int o0 = (m * NO + SPREAD - 1) / SPREAD, o1 = ((m + 1) * NO + SPREAD - 1) / SPREAD;
      static_for<(o1 < NO ? o1 : NO) - (o0 < NO ? o0 : NO)>([&](auto O_) {
        constexpr int o = o0 + decltype(O_)::value;
        if constexpr (o % OP == OP - 1 && o / OP < NI)
          issue(kt + NST, st, o / OP);
        else
          read_frag(sp, o - (o / OP < NI ? o / OP : NI), af[1 - set], bf[1 - set]);
      });
      if constexpr (m >= C0 && (m - C0) % CSTEP == 0 && (m - C0) / CSTEP < NC)
        split_frag((m - C0) / CSTEP, af[1 - set]);
      __builtin_amdgcn_sched_barrier(0);
    });
    // this wave has read k-tile kt + 1, and its loads of kt + 2 are done
    __builtin_amdgcn_s_waitcnt(0xC07F);
    wait_vmcnt<(NST - 2) * NI>();
    lds_barrier();
    st = sn;
  };
  // prologue: k-tiles 0 .. NST - 1; the fragments of k-tile 0
#pragma unroll
  for (int t = 0; t < NST; ++t)
#pragma unroll
    for (int u = 0; u < NI; ++u) issue(t, t, u);
  wait_vmcnt<(NST - 1) * NI>();
  lds_barrier();
#pragma unroll
  for (int f = 0; f < NR; ++f) read_frag(smem, f, af[0], bf[0]);
#pragma unroll
  for (int c = 0; c < NC; ++c) split_frag(c, af[0]);
  __builtin_amdgcn_s_waitcnt(0xC07F);
  wait_vmcnt<(NST - 2) * NI>();
  lds_barrier();
  mfma_accumulators_ready(acc);
  int kt = 0;
  for (; kt + 1 < nk; kt += 2) {
    step(kt, std::integral_constant<int, 0>());
    step(kt + 1, std::integral_constant<int, 1>());
  }
  if (kt < nk) {
    mfma_accumulators_ready(acc);
    step(kt, std::integral_constant<int, 0>());
  }
  wait_vmcnt<0>();  // the repeated loads land before the LDS is reused
  mfma_results_ready();
  lds_barrier();
}

struct NoRowSum {
  __device__ __forceinline__ void operator()(int, float) const {}
};

// The forward's GEMM core: bf16 storage on the bf16 core; fp32 storage with A as it is and
// the packed weights B as three bf16 planes (rows 3 K apart).
template <typename T, int BM, int NST>
struct FwdCfg_ {
  using type = SplitCfg<3, BM, true>;
};
template <int BM, int NST>
struct FwdCfg_<bf16_t, BM, NST> {
  using type = GemmCfg<bf16_t, BM, NST>;
};
template <typename T, int BM, int NST = 4>
using FwdCfg = typename FwdCfg_<T, BM, NST>::type;

// acc = A B^T over the columns [k0, k0 + Kc) of K (multiples of 64).
template <class C, typename T>
__device__ __forceinline__ void fwd_mainloop(f32x4 (&acc)[C::TM][C::TN], const T* A, int M,
                                             const bf16_t* Bw, int N, int K, int k0, int Kc, int m0,
                                             int n0, unsigned char* smem) {
  if constexpr (std::is_same<T, bf16_t>::value)
    gemm_mainloop<C>(acc, A + k0, K, M, Bw + k0, K, N, Kc, m0, n0, smem);
  else
    split_mainloop<C>(acc, A, K, M, Bw, 3 * static_cast<int64_t>(K), N, k0 / 32, (k0 + Kc) / 32, m0, n0, smem);
}

// The product of fp32 row a and packed row w over the K-columns k0 .. k0 + Kc in plain fp32: an
// infinite operand, or one whose partial products overflow with both signs, has no sum over
// planes.  Ends at the first NaN, so an output that is NaN by right costs one step.
__device__ __forceinline__ float plain_dot(const float* __restrict__ a, const bf16_t* __restrict__ w, int k0,
                                           int Kc) {
  float s = 0.f;
#pragma unroll 1
  for (int k = k0; s == s && k < k0 + Kc; k += 8) {
    float x[8], w0[8], w1[8], w2[8];
    load8(a + k, x);
    load8(w + plane_col<3>(k), w0);
    load8(w + plane_col<3>(k) + 32, w1);
    load8(w + plane_col<3>(k) + 64, w2);
#pragma unroll
    for (int j = 0; j < 8; ++j)  // (plane 1 of an infinity or a NaN is that value)
      s = fmaf(x[j], fabsf(w1[j]) < INFINITY ? w0[j] + w1[j] + w2[j] : w1[j], s);
  }
  return s;
}

// gemm_epilogue after fwd_mainloop over the same operands and columns of K.
template <class C, typename T, class F, class FR>
__device__ __forceinline__ void fwd_epilogue(const f32x4 (&acc)[C::TM][C::TN], const T* A, int M,
                                             const bf16_t* Bw, int N, int K, int k0, int Kc, int m0,
                                             int n0, unsigned char* smem, F&& f, FR&& fr) {
  if constexpr (std::is_same<T, bf16_t>::value) {
    gemm_epilogue<C>(acc, smem, m0, n0, f, fr);
  } else {
    gemm_epilogue<C>(acc, smem, m0, n0, f, fr, [&](int row, int col0, float* so) {
#pragma unroll 1
      for (int e = 0; e < 8; ++e)
        if (so[e] != so[e] && row < M && col0 < N)
          so[e] = plain_dot(A + static_cast<int64_t>(row) * K, Bw + 3 * static_cast<int64_t>(col0 + e) * K, k0, Kc);
    });
  }
}

// Split-K for GEMMs with too few output tiles to fill the chip: block (tile, y) contracts
// K slice y (Kc = K / ks columns, a multiple of BK) and stores its fp32 partial tile in
// part[y][M][N]; a combine kernel then sums the slices in order and runs the fused
// kernel's epilogue (splitk_combine), so the result does not depend on timing.
template <class C, typename T>
__device__ __forceinline__ void gemm_splitk_partial(const T* A, int M, const bf16_t* Bw, int N, int K,
                                                    int ks, int m0, int n0, float* __restrict__ part,
                                                    unsigned char* smem) {
  const int Kc = K / ks;
  const int k0 = static_cast<int>(blockIdx.y) * Kc;
  f32x4 acc[C::TM][C::TN];
  fwd_mainloop<C>(acc, A, M, Bw, N, K, k0, Kc, m0, n0, smem);
  float* pp = part + static_cast<int64_t>(blockIdx.y) * M * N;
  fwd_epilogue<C>(
      acc, A, M, Bw, N, K, k0, Kc, m0, n0, smem,
      [&](int row, int col0, const float(&v)[8]) -> float {
        if (row < M && col0 < N) store8(pp + static_cast<int64_t>(row) * N + col0, v);
        return 0.f;
      },
      NoRowSum{});
}

// One block per (blockDim / 16 rows, 128-column tile blockIdx.x): thread t owns columns
// 8 (t % 16) .. + 7 of row (blockDim / 16) blockIdx.y + t / 16, sums the ks partials in slice
// order and calls f(row, col0, v) and fr(row, sum over the tile's 128 columns) exactly
// as gemm_epilogue does (rows and columns past the matrix included: f drops them).
template <class F, class FR>
__device__ __forceinline__ void splitk_combine(int M, int N, int ks, const float* __restrict__ part,
                                               F&& f, FR&& fr) {
  const int row = static_cast<int>(blockIdx.y * (blockDim.x >> 4) + (threadIdx.x >> 4));
  const int col0 = static_cast<int>(blockIdx.x) * 128 + static_cast<int>(threadIdx.x & 15) * 8;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (row < M && col0 < N) {
    // eight slices' loads in flight at a time, added in slice order
    for (int y0 = 0; y0 < ks; y0 += 8) {
      float t[8][8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (y0 + u < ks) load8(part + (static_cast<int64_t>(y0 + u) * M + row) * N + col0, t[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (y0 + u < ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += t[u][e];
    }
  }
  float s = f(row, col0, v);
  s = sum16(s);
  if ((threadIdx.x & 15) == 0) fr(row, s);
}

// ---------------------------------------------------------------------------------
// Skinny GEMM for a few rows (bf16, one request's draft tree): a block of NW waves computes a
// (16 RM) x 16 tile over the whole of K, wave w the w-th part of it, fragments straight from
// global memory (no staging, up to U steps of 64 k in flight); the waves' sums are added in
// wave order through LDS.  Bound by latency for short K, which is what it is for; over
// K = 4096 the fragment loads (16 rows a load) run at a quarter of the staged core's rate.
// Inside a step the k are permuted alike in A and B: lane group g takes 16 g .. + 7, then
// 16 g + 8 .. + 15, so that every load touches both halves of its 128-byte lines.
//   f(row, col0, v): 8 consecutive columns of a row as in gemm_epilogue (rows past M
// included); the sum of its results over the tile's 16 columns goes to fr(row, sum).
// Reached by every thread of the block.  K a multiple of 64.
// ---------------------------------------------------------------------------------
template <int RM, int NW, int U, class F, class FR>
__device__ __forceinline__ void skinny_tile(const bf16_t* __restrict__ A, int M, const bf16_t* __restrict__ B,
                                            int K, int m0, int n0, F&& f, FR&& fr) {
  __shared__ __align__(16) float red[NW * RM * 4 * 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int nk = K / 64, per = (nk + NW - 1) / NW;
  const int s0 = wave * per, cnt = max(0, min(per, nk - s0));
  const int r = lane & 15, kofs = s0 * 64 + 16 * (lane >> 4);
  const bf16_t* pa[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) pa[i] = A + static_cast<int64_t>(min(m0 + 16 * i + r, M - 1)) * K + kofs;
  const bf16_t* pb = B + static_cast<int64_t>(n0 + r) * K + kofs;
  f32x4 acc[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int b0 = 0; b0 < cnt; b0 += U) {
    bf16x8 a[U][RM][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (b0 + u < cnt)  // uniform
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          b[u][q] = *reinterpret_cast<const bf16x8*>(pb + (b0 + u) * 64 + 8 * q);
#pragma unroll
          for (int i = 0; i < RM; ++i)
            a[u][i][q] = *reinterpret_cast<const bf16x8*>(pa[i] + (b0 + u) * 64 + 8 * q);
        }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (b0 + u < cnt)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int i = 0; i < RM; ++i) acc[i] = mfma_bf16_16x16x32(a[u][i][q], b[u][q], acc[i]);
  }
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((wave * RM + i) * 4 + v) * 64 + lane] = acc[i][v];
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 32 * RM) {  // whole waves (RM even)
    const int row = t >> 1, c8 = (t & 1) * 8;
    const int e = ((row >> 4) * 4 + (row & 3)) * 64 + 16 * ((row & 15) >> 2) + c8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      float x[8];
      load8(red + w * RM * 256 + e, x);
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] += x[q];
    }
    float sum = f(m0 + row, n0 + c8, v);
    sum += __shfl_xor(sum, 1, kWave);
    if ((t & 1) == 0) fr(m0 + row, sum);
  }
}

// Number of K slices for a GEMM of `tiles` output tiles: powers of two while the grid
// stays within one block per compute unit and every slice keeps >= 2 k-tiles.
inline int splitk_slices(int tiles, int K, int BK) {
  int ks = 1;
  if (tiles >= 128) return 1;
  while (tiles * ks * 2 <= 256 && K % (BK * ks * 2) == 0 && K / (ks * 2) >= 2 * BK) ks *= 2;
  return ks;
}

}  // namespace fovea
