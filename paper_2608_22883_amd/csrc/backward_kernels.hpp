// Backward of one draft step (paper, Method, training objective; appendix, draft model
// training: the module is trained end to end, the selected sets are a discrete choice
// and are held fixed).  Given dL/dh_hat it produces dL/dh, dL/dkeys, dL/dvalues and the
// gradients of every per-step weight, in fp32, from the raw (unfolded) fp32 weights.
//
// Forward quantities are recomputed rather than saved by the forward (the forward
// keeps none of them):  xhat = (h - mu) rstd, xe = xhat g_q + b_q + E_dep[l],
// q = xe W_Q^T, alpha = softmax over I_n of q . k_i / sqrt(d_m), r = sum alpha_i u_i,
// y = [h; r], z = y [W_c1; W_g1]^T + [b_c1; b_g1], a = SiLU(z), c = a_c W_c2^T + b_c2,
// g = sigmoid(a_g . w_g2 + b_g2), h' = h + g c.  Then, in order:
//   RMSNorm and gate (per node)      dh' , dc = g dh', dlogit = (dh' . c) g (1 - g),
//                                    dz_g = dlogit w_g2 SiLU'(z_g)
//   layer 2 (GEMM)                   dz_c = (dc W_c2) SiLU'(z_c)
//   layer 1 (GEMM)                   [dh | dr] += dz [W_c1; W_g1]
//   readout and scores (per node)    da_i = dr . u_i, ds_i = alpha_i (da_i - alpha . da),
//                                    dq = sum ds_i k_i / sqrt(d_m),
//                                    du_i += alpha_i dr, dk_i += ds_i q / sqrt(d_m)
//   query (GEMM) and LayerNorm       dxe = dq W_Q, dh += LN backward of dxe g_q
//   weight gradients (GEMMs over the node axis of transposed activations) and
//   bias / gain / E_dep gradients (column sums, deterministic two-stage).
// The memory gradients are accumulated per request in a fixed order (dense rows of
// alpha and ds over the request's memory, then one pass over the request's nodes per
// tile of memory rows), so every output is deterministic.
#pragma once

#include "common.hpp"
#include "correct_kernels.hpp"
#include "gemm.hpp"
#include "retrieve_kernels.hpp"

namespace fovea {

constexpr uint32_t kErrSelection = 0x10u;  // K or an index outside the request's memory
constexpr int kColChunks = 64;             // row chunks of the column sums
constexpr int kColGroups = 8;              // groups (depths) per column-sum pass

__device__ __forceinline__ float dsilu_f(float z) {
  const float s = sigmoid_f(z);
  return s * (1.0f + z * (1.0f - s));
}

// sum over the 256 threads of a block, in every thread (red: 4 floats of LDS)
__device__ __forceinline__ float block_sum256(float v, float* red) {
  v = wave_sum_f32(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// sum_{i < K} w[i] * rows[(m0 + ix[i]) * ld + j + c] for the four columns c < 4 (16-byte loads;
// ld and j multiples of 4), the row loads issued eight at a time so that their latencies overlap
__device__ __forceinline__ f32x4 weighted_rows4(const float* __restrict__ w, const int32_t* __restrict__ ix,
                                                int K, const float* __restrict__ rows, int64_t m0,
                                                int64_t ld, int j) {
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < K; i0 += 8) {
    f32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = i0 + u < K ? *reinterpret_cast<const f32x4*>(rows + (m0 + ix[i0 + u]) * ld + j)
                        : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + u < K) {
        const float wu = w[i0 + u];
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(wu, v[u][c], acc[c]);
      }
  }
  return acc;
}

// out[i] = scale * (x . rows[m0 + ix[i]]) for the entries i = wave, wave + 4, ... < K of
// a 4-wave block (x in LDS, d_m wide): four entries at a time, each lane's loads of all
// four issued together (512 columns per pass).
__device__ __forceinline__ void wave_row_dots(const float* x, const int32_t* __restrict__ ix, int K,
                                              const float* __restrict__ rows, int64_t m0, int d_m,
                                              float scale, float* out, int wave, int lane) {
  for (int i0 = wave; i0 < K; i0 += 16) {
    const float* rp[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) rp[u] = rows + (m0 + ix[min(i0 + 4 * u, K - 1)]) * d_m;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < d_m; j0 += 512) {
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int j = j0 + lane + 64 * t;
          v[u][t] = j < d_m ? rp[u][j] : 0.f;
        }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int j = j0 + lane + 64 * t;
        const float xj = j < d_m ? x[j] : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = fmaf(xj, v[u][t], acc[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float sdot = wave_sum_f32(acc[u]);
      if (lane == 0 && i0 + 4 * u < K) out[i0 + 4 * u] = sdot * scale;
    }
  }
}

__global__ __launch_bounds__(256) void fill_f32_kernel(int64_t count, float* __restrict__ p, float v) {
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < count; i += static_cast<int64_t>(gridDim.x) * 256)
    p[i] = v;
}

// Four consecutive floats, 16-byte aligned only if vec.
__device__ __forceinline__ f32x4 load4(const float* p, bool vec) {
  if (vec) return *reinterpret_cast<const f32x4*>(p);
  return f32x4{p[0], p[1], p[2], p[3]};
}

// Planes of the recomputed forward's two net layers (z and c): three, as exact as fp32, since
// dL/db_g2 is one sum of both signs over every node of what c's error leaves; every other
// product takes two.
constexpr int kFwdPlanes = 3;

// Four consecutive columns k .. k + 3 (k a multiple of 4) of a row of P planes.
template <int P>
__device__ __forceinline__ void store_planes4(bf16_t* row, int64_t k, const f32x4& x) {
  uint32_t a[P], b[P];
  split_pair<P>(x[0], x[1], a);
  split_pair<P>(x[2], x[3], b);
#pragma unroll
  for (int p = 0; p < P; ++p)
    *reinterpret_cast<uint2*>(row + plane_col<P>(k) + 32 * p) = make_uint2(a[p], b[p]);
}

// Rows of an fp32 matrix as a GEMM operand sees them: as they are, or with a LayerNorm
// applied on the way ((x - mu) rstd g + b, plus the depth's row of E if given), so that the
// normalised rows need not be stored.  Rows with ok < 0 (if given) are zero.
struct RowSrc {
  const float* x;
  int64_t ld;
  const float2* stats;    // nullable
  const float* g;         // with stats
  const float* b;
  const float* E;         // nullable
  const int32_t* depth;   // with E
  int n_depth;
  const int32_t* ok;      // nullable
  bool vec;               // x, g, b and E 16-byte aligned, ld a multiple of 4
  __device__ __forceinline__ f32x4 load(int r, int c, int cols) const {
    if (ok != nullptr && ok[r] < 0) return f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 v = load4(x + static_cast<int64_t>(r) * ld + c, vec);
    if (stats != nullptr) {
      const float2 st = stats[r];
      const f32x4 gv = load4(g + c, vec);
      f32x4 bv = load4(b + c, vec);
      if (E != nullptr)
        bv += load4(E + static_cast<int64_t>(min(max(depth[r], 0), n_depth - 1)) * cols + c, vec);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaf((v[e] - st.x) * st.y, gv[e], bv[e]);
    }
    return v;
  }
};

// Per node: the planes of xe = LN(h) + E_dep[l] and of h as the left part of y = [h; r]
// (rows of kFwdPlanes (d + d_m)), four columns per thread and step.  Nodes that failed validation
// are zeros.
__global__ __launch_bounds__(256) void bwd_prep_kernel(int n, int d, int d_m, RowSrc xe, RowSrc h,
                                                       bf16_t* __restrict__ xe_p,
                                                       bf16_t* __restrict__ y_p) {
  const int row = blockIdx.x;
  if (row >= n) return;
#pragma unroll 4
  for (int j = 4 * threadIdx.x; j < d; j += 1024) {
    store_planes4<2>(xe_p + static_cast<int64_t>(row) * 2 * d, j, xe.load(row, j, d));
    store_planes4<kFwdPlanes>(y_p + static_cast<int64_t>(row) * kFwdPlanes * (d + d_m), j, h.load(row, j, d));
  }
}

// Per node (one block): validates its K and indices, then recomputes the renormalised
// softmax over the selected entries (alpha [n, k_max]) and the readout r [n, d_m], also as
// the right part of y's planes.  ok[n] = 0 marks a node that failed validation (here or in the statistics
// kernel); it contributes nothing to any gradient and its dh row becomes NaN.
__global__ __launch_bounds__(256) void bwd_sel_fwd_kernel(int n, int d, int d_m, int k_max,
                                                          const NodeInfo* __restrict__ info,
                                                          const int32_t* __restrict__ K_in,
                                                          const int32_t* __restrict__ idx,
                                                          const float* __restrict__ q,
                                                          const float* __restrict__ keys,
                                                          const float* __restrict__ values,
                                                          float scale, float* __restrict__ alpha,
                                                          float* __restrict__ r_out,
                                                          bf16_t* __restrict__ y_p,
                                                          int32_t* __restrict__ ok_out,
                                                          uint32_t* err) {
  extern __shared__ float smem_f[];
  float* sq = smem_f;             // q_n [d_m]
  float* sa = smem_f + d_m;       // scores, then alpha [k_max]
  __shared__ float red[4];
  __shared__ int sbad;
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (row >= n) return;
  const NodeInfo ni = info[row];
  int K = K_in[row];
  if (tid == 0) sbad = 0;
  __syncthreads();
  bool ok = ni.M >= 0;
  if (ok && (K < 0 || K > min(k_max, ni.M))) {
    ok = false;
    if (tid == 0) atomicOr(err, kErrSelection);
  }
  if (ok) {
    for (int i = tid; i < K; i += 256) {
      const int ix = idx[static_cast<int64_t>(row) * k_max + i];
      if (ix < 0 || ix >= ni.M) sbad = 1;
    }
  }
  __syncthreads();
  if (ok && sbad) {
    ok = false;
    if (tid == 0) atomicOr(err, kErrSelection);
  }
  if (tid == 0) ok_out[row] = ok ? 1 : 0;
  if (!ok) K = 0;
  #pragma unroll 8
  for (int j = tid; j < d_m; j += 256) sq[j] = q[static_cast<int64_t>(row) * d_m + j];
  __syncthreads();
  // scores of the selected entries
  wave_row_dots(sq, idx + static_cast<int64_t>(row) * k_max, K, keys, ni.m0, d_m, scale, sa, wave, lane);
  __syncthreads();
  float mx = -INFINITY;
  for (int i = tid; i < K; i += 256) mx = fmaxf(mx, sa[i]);
  mx = wave_max(mx);
  __syncthreads();
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float z = 0.f;
  for (int i = tid; i < K; i += 256) z += expf(sa[i] - mx);
  z = block_sum256(z, red);
  for (int i = tid; i < K; i += 256) {
    const float a = expf(sa[i] - mx) / z;
    sa[i] = a;
    alpha[static_cast<int64_t>(row) * k_max + i] = a;
  }
  __syncthreads();
  // r = sum alpha_i u_i, columns over the threads
  const int32_t* ixr = idx + static_cast<int64_t>(row) * k_max;
  for (int j = 4 * tid; j < d_m; j += 1024) {
    const f32x4 v = weighted_rows4(sa, ixr, K, values, ni.m0, d_m, j);
    *reinterpret_cast<f32x4*>(r_out + static_cast<int64_t>(row) * d_m + j) = v;
    store_planes4<kFwdPlanes>(y_p + static_cast<int64_t>(row) * kFwdPlanes * (d + d_m), d + j, v);
  }
}

// Per node: gate, h' = h + g c, RMSNorm backward, the residual split and the gate's
// backward.  Writes dh (= dh'), dc = g dh' (also as planes), hn = h' rho (for dL/drms_w),
// dlogit[row] and dz[:, d_c:] = dlogit w_g2 SiLU'(z_g) (also as planes).  Nodes with ok = 0
// get zero gradients.  A row of up to 1024 R columns stays in registers between the sums and
// the outputs (1920 rows of 4096: 51.7 us reading it twice, 8 bytes a load).
template <int R>
__global__ __launch_bounds__(256) void bwd_rms_gate_kernel(int n, int d, int d_c,
                                                           const float* __restrict__ h,
                                                           const float* __restrict__ c,
                                                           const float* __restrict__ z,
                                                           const float* __restrict__ a,
                                                           const float* __restrict__ w_g2, float b_g2,
                                                           const float* __restrict__ rms_w, float eps,
                                                           const float* __restrict__ dh_hat,
                                                           const int32_t* __restrict__ ok_in,
                                                           float* __restrict__ dh,
                                                           float* __restrict__ dc,
                                                           bf16_t* __restrict__ dc_p,
                                                           float* __restrict__ hn,
                                                           float* __restrict__ dlogit,
                                                           float* __restrict__ dz,
                                                           bf16_t* __restrict__ dz_p) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  if (row >= n) return;
  const bool ok = ok_in[row] != 0;
  const int64_t ro = static_cast<int64_t>(row) * d;
  const int64_t zo = static_cast<int64_t>(row) * 2 * d_c;
  constexpr f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 hv[R], cv[R], gv[R];  // h then h', c, dh_hat
  auto load = [&](int u, int j) {
    hv[u] = *reinterpret_cast<const f32x4*>(h + ro + j);
    cv[u] = *reinterpret_cast<const f32x4*>(c + ro + j);
    gv[u] = *reinterpret_cast<const f32x4*>(dh_hat + ro + j);
  };
  const bool held = d <= 1024 * R;
  if (held)
#pragma unroll
    for (int u = 0; u < R; ++u) {
      hv[u] = cv[u] = gv[u] = zero;
      if (4 * tid + 1024 * u < d) load(u, 4 * tid + 1024 * u);
    }
  float t = 0.f;
#pragma unroll 8
  for (int j = tid; j < d_c; j += 256) t = fmaf(a[zo + d_c + j], w_g2[j], t);
  const float g = sigmoid_f(block_sum256(t, red) + b_g2);
  float rho = 1.f, tw = 0.f;
  if (rms_w != nullptr) {
    float ss = 0.f, sw = 0.f;
    auto sums = [&](int u, int j) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(rms_w + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float hp = fmaf(g, cv[u][e], hv[u][e]);
        ss = fmaf(hp, hp, ss);
        sw = fmaf(w[e] * gv[u][e], hp, sw);
      }
    };
    if (held) {
#pragma unroll
      for (int u = 0; u < R; ++u)
        if (4 * tid + 1024 * u < d) sums(u, 4 * tid + 1024 * u);
    } else {
      for (int j = 4 * tid; j < d; j += 1024) {
        load(0, j);
        sums(0, j);
      }
    }
    ss = block_sum256(ss, red);
    tw = block_sum256(sw, red);
    rho = 1.0f / sqrtf(ss / static_cast<float>(d) + eps);
  }
  const float k3 = rho * rho * rho * tw / static_cast<float>(d);
  float sdg = 0.f;
  auto finish = [&](int u, int j) {
    const f32x4 w = rms_w != nullptr ? *reinterpret_cast<const f32x4*>(rms_w + j) : zero;
    f32x4 dhv, dcv, hnv;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float hp = fmaf(g, cv[u][e], hv[u][e]);
      float dhp = rms_w != nullptr ? rho * w[e] * gv[u][e] - k3 * hp : gv[u][e];
      dhp = ok ? dhp : 0.f;
      hnv[e] = ok ? hp * rho : 0.f;
      dhv[e] = dhp;
      dcv[e] = g * dhp;
      sdg = fmaf(dhp, cv[u][e], sdg);
    }
    if (rms_w != nullptr) *reinterpret_cast<f32x4*>(hn + ro + j) = hnv;
    *reinterpret_cast<f32x4*>(dh + ro + j) = dhv;
    *reinterpret_cast<f32x4*>(dc + ro + j) = dcv;
    store_planes4<2>(dc_p + 2 * ro, j, dcv);
  };
  if (held) {
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (4 * tid + 1024 * u < d) finish(u, 4 * tid + 1024 * u);
  } else {
    for (int j = 4 * tid; j < d; j += 1024) {
      load(0, j);
      finish(0, j);
    }
  }
  const float dl = block_sum256(sdg, red) * g * (1.0f - g);
  if (tid == 0) dlogit[row] = dl;
  for (int j = 4 * tid; j < d_c; j += 1024) {
    const f32x4 zv = *reinterpret_cast<const f32x4*>(z + zo + d_c + j);
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = dl * w_g2[j + e] * dsilu_f(zv[e]);
    *reinterpret_cast<f32x4*>(dz + zo + d_c + j) = v;
    store_planes4<2>(dz_p + 2 * zo, d_c + j, v);
  }
}

// Per node: the readout and score backward.  dr [n, d_m]; writes dq [n, d_m] (also as planes) and the
// node's dense rows over its request's memory (m_max wide): wa = alpha_i and
// ws = ds_i / sqrt(d_m) at the selected entries, 0 elsewhere (the selected indices are
// distinct, as the forward produces them).
__global__ __launch_bounds__(256) void bwd_sel_kernel(int n, int d_m, int k_max, int m_max,
                                                      const NodeInfo* __restrict__ info,
                                                      const int32_t* __restrict__ K_in,
                                                      const int32_t* __restrict__ idx,
                                                      const int32_t* __restrict__ ok_in,
                                                      const float* __restrict__ alpha,
                                                      const float* __restrict__ dr,
                                                      const float* __restrict__ keys,
                                                      const float* __restrict__ values,
                                                      float scale, float* __restrict__ dq,
                                                      bf16_t* __restrict__ dq_p,
                                                      float* __restrict__ wa,
                                                      float* __restrict__ ws) {
  extern __shared__ float smem_f[];
  float* sdr = smem_f;        // dr_n [d_m]
  float* sds = smem_f + d_m;  // da, then ds [k_max]
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (row >= n) return;
  const int K = ok_in[row] ? K_in[row] : 0;
  const int64_t m0 = info[row].m0;
  const int32_t* ix = idx + static_cast<int64_t>(row) * k_max;
  const float* al = alpha + static_cast<int64_t>(row) * k_max;
  float* war = wa + static_cast<int64_t>(row) * m_max;
  float* wsr = ws + static_cast<int64_t>(row) * m_max;
  for (int i = tid; i < m_max; i += 256) {
    war[i] = 0.f;
    wsr[i] = 0.f;
  }
  #pragma unroll 8
  for (int j = tid; j < d_m; j += 256) sdr[j] = dr[static_cast<int64_t>(row) * d_m + j];
  __syncthreads();
  wave_row_dots(sdr, ix, K, values, m0, d_m, 1.0f, sds, wave, lane);  // da_i = dr . u_i
  __syncthreads();
  float ad = 0.f;
  for (int i = tid; i < K; i += 256) ad = fmaf(al[i], sds[i], ad);
  ad = block_sum256(ad, red);
  for (int i = tid; i < K; i += 256) {
    const float dsi = al[i] * (sds[i] - ad);
    sds[i] = dsi;
    war[ix[i]] = al[i];  // after the zeroing above (block barrier in block_sum256)
    wsr[ix[i]] = dsi * scale;
  }
  __syncthreads();
  for (int j = 4 * tid; j < d_m; j += 1024) {
    const f32x4 v = weighted_rows4(sds, ix, K, keys, m0, d_m, j);
    const f32x4 o = f32x4{v[0] * scale, v[1] * scale, v[2] * scale, v[3] * scale};
    *reinterpret_cast<f32x4*>(dq + static_cast<int64_t>(row) * d_m + j) = o;
    store_planes4<2>(dq_p + static_cast<int64_t>(row) * 2 * d_m, j, o);
  }
}

// Memory gradients of one request, one tile of 32 memory rows x 256 columns per block:
//   dvalues[m0 + i] = sum over the request's nodes t of wa[t][i] dr[t]
//   dkeys[m0 + i]   = sum over the request's nodes t of ws[t][i] q[t]
// in node order.  Grid: (ceil(d_m / 256), ceil(m_max / 32), B).
constexpr int kMemRows = 32;

// A request whose memory and node ranges are usable (the memory-gradient kernel writes
// every row of such a request, zeros included)
__device__ __forceinline__ bool mem_request_ok(int64_t m0, int64_t m1, int t0, int t1, int m_max,
                                               int t_max, int n, int64_t n_mem) {
  return 0 <= m0 && m0 <= m1 && m1 <= n_mem && m1 - m0 <= m_max && 0 <= t0 && t0 <= t1 &&
         t1 <= n && t1 - t0 <= t_max;
}

// Zero rows of dkeys and dvalues that no usable request covers (run before
// bwd_mem_grad_kernel, which writes all the others).  16 rows per block, 16 threads per
// row.  The covering request is found by binary search over mem_off; where mem_off is
// not sorted the search may miss a cover, and the zeros written are then overwritten.
__global__ __launch_bounds__(256) void bwd_mem_gaps_kernel(int d_m, int m_max, int t_max, int B,
                                                           const int64_t* __restrict__ mem_off,
                                                           const int32_t* __restrict__ node_off,
                                                           int n, int64_t n_mem,
                                                           float* __restrict__ dkeys,
                                                           float* __restrict__ dvalues) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 16 + (threadIdx.x >> 4);
  if (i >= n_mem) return;
  int lo = 0, hi = B;  // the last b < B with mem_off[b] <= i, else 0
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (mem_off[mid] <= i)
      lo = mid;
    else
      hi = mid;
  }
  const int64_t m0 = mem_off[lo], m1 = mem_off[lo + 1];
  if (mem_request_ok(m0, m1, node_off[lo], node_off[lo + 1], m_max, t_max, n, n_mem) && m0 <= i &&
      i < m1)
    return;
  const f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int j = 4 * (threadIdx.x & 15); j < d_m; j += 64) {
    *reinterpret_cast<f32x4*>(dkeys + i * d_m + j) = z;
    *reinterpret_cast<f32x4*>(dvalues + i * d_m + j) = z;
  }
}

__global__ __launch_bounds__(256) void bwd_mem_grad_kernel(int d_m, int m_max, int t_max,
                                                           const int64_t* __restrict__ mem_off,
                                                           const int32_t* __restrict__ node_off,
                                                           int n, int64_t n_mem,
                                                           const float* __restrict__ wa,
                                                           const float* __restrict__ ws,
                                                           const float* __restrict__ dr,
                                                           const float* __restrict__ q,
                                                           float* __restrict__ dkeys,
                                                           float* __restrict__ dvalues) {
  // [t_max][kMemRows] of wa, then of ws, then each wave's list of nodes
  extern __shared__ float smem_f[];
  float* swa = smem_f;
  float* sws = smem_f + t_max * kMemRows;
  uint16_t* slist = reinterpret_cast<uint16_t*>(smem_f + 2 * t_max * kMemRows);
  const int b = blockIdx.z, r0 = blockIdx.y * kMemRows;
  const int64_t m0 = mem_off[b], m1 = mem_off[b + 1];
  const int t0 = node_off[b], t1 = node_off[b + 1];
  // offsets were validated per node; a request whose range is unusable is skipped here
  const bool ok = mem_request_ok(m0, m1, t0, t1, m_max, t_max, n, n_mem);
  const int M = ok ? static_cast<int>(m1 - m0) : 0;
  if (r0 >= M) return;
  const int T = t1 - t0;
  // stage the request's rows of wa / ws (eight loads in flight per thread)
  for (int e0 = 0; e0 < T * kMemRows; e0 += 256 * 4) {
    float va[4], vs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * 256 + static_cast<int>(threadIdx.x);
      const int t = min(e / kMemRows, T - 1), r = e % kMemRows;
      const int64_t src = static_cast<int64_t>(t0 + t) * m_max + min(r0 + r, m_max - 1);
      va[u] = wa[src];
      vs[u] = ws[src];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * 256 + static_cast<int>(threadIdx.x);
      if (e < T * kMemRows) {
        swa[e] = va[u];
        sws[e] = vs[u];
      }
    }
  }
  __syncthreads();
  // wave w owns memory rows r0 + 8 w .. + 7; lane l owns columns j0 .. j0 + 3.  A node selects
  // few entries (16 of 576, say), so most have none of the wave's rows: the wave lists those
  // that have, in node order (their weights may still be 0 or NaN), and walks the list.
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint16_t* list = slist + wv * t_max;
  int nl = 0;
  for (int tb = 0; tb < T; tb += 64) {
    const int t = min(tb + lane, T - 1);
    bool any = false;
#pragma unroll
    for (int r = 0; r < 8; ++r)
      any |= !(swa[t * kMemRows + 8 * wv + r] == 0.f) || !(sws[t * kMemRows + 8 * wv + r] == 0.f);
    const unsigned long long m = __ballot(any && tb + lane < T);
    if (any && tb + lane < T) list[nl + __popcll(m & ((1ull << lane) - 1ull))] = static_cast<uint16_t>(t);
    nl += __popcll(m);
  }
  wave_lds_sync();
  const int j0 = blockIdx.x * 256 + 4 * lane;
  if (j0 >= d_m) return;
  float au[8][4], ak[8][4];
#pragma unroll
  for (int r = 0; r < 8; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      au[r][c] = 0.f;
      ak[r][c] = 0.f;
    }
  // the listed nodes' rows of dr and q come through a 4-deep register prefetch
  constexpr int PF = 4;
  f32x4 drb[PF], qb[PF];
  auto fetch = [&](int u, int i) {
    const int64_t tt = t0 + list[min(i, nl - 1)];
    drb[u] = *reinterpret_cast<const f32x4*>(dr + tt * d_m + j0);
    qb[u] = *reinterpret_cast<const f32x4*>(q + tt * d_m + j0);
  };
  if (nl > 0) {
#pragma unroll
  for (int u = 0; u < PF; ++u) fetch(u, u);
  for (int ib = 0; ib < nl; ib += PF) {
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    if (ib + u >= nl) break;
    const int t = list[ib + u];
    const f32x4 drv = drb[u], qv = qb[u];
    fetch(u, ib + u + PF);
    const f32x4 wa0 = *reinterpret_cast<const f32x4*>(swa + t * kMemRows + 8 * wv);
    const f32x4 wa1 = *reinterpret_cast<const f32x4*>(swa + t * kMemRows + 8 * wv + 4);
    const f32x4 ws0 = *reinterpret_cast<const f32x4*>(sws + t * kMemRows + 8 * wv);
    const f32x4 ws1 = *reinterpret_cast<const f32x4*>(sws + t * kMemRows + 8 * wv + 4);
    const float wa[8] = {wa0[0], wa0[1], wa0[2], wa0[3], wa1[0], wa1[1], wa1[2], wa1[3]};
    const float ws[8] = {ws0[0], ws0[1], ws0[2], ws0[3], ws1[0], ws1[1], ws1[2], ws1[3]};
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        au[r][c] = fmaf(wa[r], drv[c], au[r][c]);
        ak[r][c] = fmaf(ws[r], qv[c], ak[r][c]);
      }
  }
  }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int i = r0 + 8 * wv + r;
    if (i < M) {
      *reinterpret_cast<f32x4*>(dvalues + (m0 + i) * d_m + j0) = f32x4{au[r][0], au[r][1], au[r][2], au[r][3]};
      *reinterpret_cast<f32x4*>(dkeys + (m0 + i) * d_m + j0) = f32x4{ak[r][0], ak[r][1], ak[r][2], ak[r][3]};
    }
  }
}

// Per row: out (+)= LayerNorm backward of dx g, with xhat = (x - mu) rstd from the input
// and its statistics; rows with ok = 0 become NaN (ok_in null: every row is valid).  Rows of
// up to 1024 R columns are read once into registers.
template <int R, bool ADD>
__global__ __launch_bounds__(256) void bwd_ln_kernel(int n, int d, const float* __restrict__ dx,
                                                     const float* __restrict__ x,
                                                     const float* __restrict__ g, bool g_vec,
                                                     const float2* __restrict__ stats,
                                                     const int32_t* __restrict__ ok_in,
                                                     float* __restrict__ out) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  if (row >= n) return;
  const int64_t ro = static_cast<int64_t>(row) * d;
  const float2 st = stats[row];
  f32x4 tv[R], xv[R], ov[R];
  float s1 = 0.f, s2 = 0.f;
  auto load = [&](int u, int j) {
    tv[u] = *reinterpret_cast<const f32x4*>(dx + ro + j) * load4(g + j, g_vec);
    xv[u] = *reinterpret_cast<const f32x4*>(x + ro + j);
    if (ADD) ov[u] = *reinterpret_cast<const f32x4*>(out + ro + j);
  };
  auto sums = [&](int u) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xv[u][e] = (xv[u][e] - st.x) * st.y;
      s1 += tv[u][e];
      s2 = fmaf(tv[u][e], xv[u][e], s2);
    }
  };
  const bool held = d <= 1024 * R;
  if (held) {
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (4 * tid + 1024 * u < d) load(u, 4 * tid + 1024 * u);
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (4 * tid + 1024 * u < d) sums(u);
  } else {
    for (int j = 4 * tid; j < d; j += 1024) {
      load(0, j);
      sums(0);
    }
  }
  const float m1 = block_sum256(s1, red) / static_cast<float>(d);
  const float m2 = block_sum256(s2, red) / static_cast<float>(d);
  const bool ok = ok_in == nullptr || ok_in[row] != 0;
  auto finish = [&](int u, int j) {
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = st.y * (tv[u][e] - m1 - xv[u][e] * m2);
      o[e] = ok ? (ADD ? ov[u][e] + v : v) : __builtin_nanf("");
    }
    *reinterpret_cast<f32x4*>(out + ro + j) = o;
  };
  if (held) {
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (4 * tid + 1024 * u < d) finish(u, 4 * tid + 1024 * u);
  } else {
    for (int j = 4 * tid; j < d; j += 1024) {
      load(0, j);
#pragma unroll
      for (int e = 0; e < 4; ++e) xv[0][e] = (xv[0][e] - st.x) * st.y;
      finish(0, j);
    }
  }
}

// out[j] = sum_i X[j * ldx + i] (* s[i]) over i < len: one wave per row of a transposed
// (node-minor, zero-padded) array.
__global__ __launch_bounds__(256) void rowsum_kernel(int rows, int len, const float* __restrict__ X,
                                                     int64_t ldx, const float* __restrict__ s,
                                                     float* __restrict__ out) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= rows) return;
  const float* xr = X + static_cast<int64_t>(r) * ldx;
  float acc = 0.f;
  for (int i0 = lane; i0 < len; i0 += 64 * 8) {
    float x[8], w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + 64 * u;
      x[u] = i < len ? xr[i] : 0.f;
      w[u] = s != nullptr && i < len ? s[i] : 1.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = fmaf(x[u], w[u], acc);
  }
  acc = wave_sum_f32(acc);
  if (lane == 0) out[r] = acc;
}

// Column sums of several row-major fp32 arrays in one launch.  A job sums over the rows
// i < n of X (16-byte aligned, ldx and cols multiples of 4), each row scaled by rs[i] if
// given, into up to three kinds of outputs:
//   out_x[j]                   = sum_i X[i][j]
//   out_xy[j]                  = sum_i X[i][j] Y[i][j]
//   out_grp[(g0 + g) cols + j] = sum over the rows with grp[i] == g0 + g (g < ng) of X[i][j]
// (a null output is not computed; grp values are clamped to 0 .. n_grp_total - 1).
// Stage 1 writes per-chunk partial sums, stage 2 adds the chunks in a fixed order, so
// every sum is deterministic.
constexpr int kColJobs = 8;
constexpr int kColSlots = 2 + kColGroups;

struct ColJob {
  const float* X;
  int64_t ldx;
  const float* Y;  // nullable (needed for out_xy)
  int64_t ldy;
  const float2* ys;      // nullable: Y[i][j] stands for (Y[i][j] - ys[i].x) ys[i].y, 0 where yok[i] < 0
  const int32_t* yok;    // nullable
  const float* rs;       // nullable
  const int32_t* grp;    // nullable (needed for out_grp)
  float* out_x;          // nullable
  float* out_xy;         // nullable
  float* out_grp;        // nullable
  int g0, ng, n_grp_total;
  int cols;
  int64_t part_off;      // floats: this job's partials, [kColChunks][slots][cols]
};

struct ColJobs {
  ColJob job[kColJobs];
  int n_jobs;
};

__device__ __forceinline__ int col_job_slots(const ColJob& jb) {
  return (jb.out_x != nullptr) + (jb.out_xy != nullptr) + (jb.out_grp != nullptr ? jb.ng : 0);
}

// Stage 1: grid (ceil(max cols / 256), kColChunks, n_jobs); the block's 256 columns are four
// per lane, its chunk of rows is split over the four waves (consecutive quarters, eight rows
// in flight each), whose sums are added in wave order through LDS.  Bound by HBM; with a
// block of 1024 columns per chunk one array of 4096 columns held one block per compute unit
// (two arrays of 4608 x 4096: 58 us).
__global__ __launch_bounds__(256) void colsum_multi_kernel(int n, ColJobs jobs,
                                                           float* __restrict__ part) {
  __shared__ f32x4 red[3][64];
  const ColJob& jb = jobs.job[blockIdx.z];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  if (static_cast<int>(blockIdx.x) * 256 >= jb.cols) return;  // uniform
  const int j = 4 * (blockIdx.x * 64 + lane);
  const int jc = min(j, jb.cols - 4);
  const int per = (n + kColChunks - 1) / kColChunks, sub = (per + 3) / 4;
  const int c0 = blockIdx.y * per, c1 = min(n, c0 + per);
  const int i0 = c0 + wave * sub, i1 = min(c1, i0 + sub);
  const bool want_x = jb.out_x != nullptr, want_xy = jb.out_xy != nullptr,
             want_g = jb.out_grp != nullptr;
  constexpr f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 acc[kColSlots];  // x, x y, then the groups
#pragma unroll
  for (int t = 0; t < kColSlots; ++t) acc[t] = zero;
  for (int ib = i0; ib < i1; ib += 8) {
    f32x4 x[8], y[8];
    float sc[8], mu[8], rs[8];
    int grp[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = min(ib + u, i1 - 1);  // repeated rows are dropped below
      x[u] = *reinterpret_cast<const f32x4*>(jb.X + static_cast<int64_t>(i) * jb.ldx + jc);
      y[u] = want_xy ? *reinterpret_cast<const f32x4*>(jb.Y + static_cast<int64_t>(i) * jb.ldy + jc) : zero;
      sc[u] = jb.rs != nullptr ? jb.rs[i] : 1.f;
      mu[u] = jb.ys != nullptr ? jb.ys[i].x : 0.f;
      rs[u] = jb.ys != nullptr ? jb.ys[i].y : 1.f;
      if (jb.yok != nullptr && jb.yok[i] < 0) rs[u] = -1.f;  // (an rstd is positive or NaN)
      grp[u] = want_g ? min(max(jb.grp[i], 0), jb.n_grp_total - 1) - jb.g0 : 0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (ib + u >= i1) break;  // uniform
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float v = x[u][c] * sc[u];
        const float yv = rs[u] < 0.f ? 0.f : (y[u][c] - mu[u]) * rs[u];
        acc[0][c] += v;
        acc[1][c] = fmaf(v, yv, acc[1][c]);
        if (want_g)
#pragma unroll
          for (int g = 0; g < kColGroups; ++g) acc[2 + g][c] += g == grp[u] ? v : 0.f;
      }
    }
  }
  const int slots = col_job_slots(jb);
  float* pp = part + jb.part_off + static_cast<int64_t>(blockIdx.y) * slots * jb.cols + j;
  int sl = 0;
#pragma unroll
  for (int t = 0; t < kColSlots; ++t) {
    if (t == 0 ? !want_x : t == 1 ? !want_xy : !(want_g && t - 2 < jb.ng)) continue;  // uniform
    __syncthreads();
    if (wave > 0) red[wave - 1][lane] = acc[t];
    __syncthreads();
    if (wave == 0 && j < jb.cols)
      *reinterpret_cast<f32x4*>(pp + static_cast<int64_t>(sl) * jb.cols) =
          ((acc[t] + red[0][lane]) + red[1][lane]) + red[2][lane];
    ++sl;
  }
}

// Stage 2: grid (ceil(max cols / 256), kColSlots, n_jobs); the chunks' partials of one
// slot added in chunk order.
__global__ __launch_bounds__(256) void colsum_multi_final_kernel(ColJobs jobs,
                                                                 const float* __restrict__ part) {
  const ColJob& jb = jobs.job[blockIdx.z];
  const int j = blockIdx.x * 256 + threadIdx.x;
  const int slots = col_job_slots(jb), sl = blockIdx.y;
  if (j >= jb.cols || sl >= slots) return;
  const float* pp = part + jb.part_off + static_cast<int64_t>(sl) * jb.cols + j;
  const int64_t stride = static_cast<int64_t>(slots) * jb.cols;
  float acc = 0.f;
#pragma unroll 16
  for (int ch = 0; ch < kColChunks; ++ch) acc += pp[ch * stride];
  int k = sl;
  float* out;
  if (jb.out_x != nullptr && k == 0) {
    out = jb.out_x;
  } else {
    k -= jb.out_x != nullptr;
    if (jb.out_xy != nullptr && k == 0) {
      out = jb.out_xy;
    } else {
      k -= jb.out_xy != nullptr;
      out = jb.out_grp + static_cast<int64_t>(jb.g0 + k) * jb.cols;
    }
  }
  out[j] = acc;
}

// fp32 rows as P bf16 planes (the split GEMM core's layout), at columns c_off .. of rows
// of W columns: thread i converts 8 consecutive columns (C, W and c_off multiples of 32).
template <int P>
__global__ __launch_bounds__(256) void split_planes_kernel(int R, int C, const float* __restrict__ src,
                                                           int64_t lds, bf16_t* __restrict__ dst, int W,
                                                           int c_off, bool vec) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t r = i / (C / 8);
  const int c = static_cast<int>(i % (C / 8)) * 8;
  if (r >= R) return;
  const f32x4 a = load4(src + r * lds + c, vec), b = load4(src + r * lds + c + 4, vec);
  const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  store_planes8<P>(dst + r * P * W, c_off + c, x);
}

// The planes of src^T: row c of dst (2 W long) holds column c of src [R, C] at columns
// r_off .. r_off + R_pad - 1 (rows R .. R_pad - 1 zero), through 64 x 64 LDS tiles: the
// node-axis operands of the weight-gradient GEMMs and the transposed weights.  Grid:
// (ceil(C / 64), ceil(R_pad / 64)).  Each thread loads four columns of a row and stores
// 16-byte plane pieces (eight source rows): C a multiple of 4, R_pad, W and r_off of 32.
__global__ __launch_bounds__(256) void transpose_planes_kernel(int R, int R_pad, int C, RowSrc src,
                                                               bf16_t* __restrict__ dst, int W,
                                                               int r_off) {
  __shared__ float t[64][65];
  const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  const int tid = threadIdx.x;
  // tile row (tid / 16) + 16 p, columns 4 (tid % 16) .. + 3
  const int q = 4 * (tid & 15);
  f32x4 v[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = r0 + (tid >> 4) + 16 * p, c = c0 + q;
    v[p] = (r < R && c < C) ? src.load(r, c, C) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int e = 0; e < 4; ++e) t[(tid >> 4) + 16 * p][q + e] = v[p][e];
  __syncthreads();
  // tile column (tid / 8) + 32 p (a row of dst), tile rows 8 (tid % 8) .. + 7
  const int g = 8 * (tid & 7);
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int cl = (tid >> 3) + 32 * p, c = c0 + cl, r = r0 + g;
    if (c < C && r < R_pad) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = t[g + e][cl];
      store_planes8<2>(dst + static_cast<int64_t>(c) * 2 * W, r_off + r, x);
    }
  }
}

// GEMM C = A B^T over P-plane operands (A [M, K], B [N, K], K a multiple of 32, N of 8)
// with the epilogues the backward needs.
enum BwdEpi : int {
  kEpiStore = 0,  // out = v (+ bias[col])
  kEpiZ = 1,      // out = v + bias (pre-activation), out2 = SiLU(out), planes of out2[:, :split]
  kEpiDsilu = 2,  // out = v * SiLU'(aux), also as planes
  kEpiSplit = 3,  // col < split: out[col] += v; else out2[col - split] = v
  kEpiRows = 4,   // row < split: out[row] = v; else out2[row - split] = v
};

struct BwdGemm {
  int M, N, K;
  const bf16_t* A;  // planes
  const bf16_t* B;
  float* out;
  int64_t ldo;
  const float* bias;   // nullable
  const float* bias2;  // nullable: the bias of the columns from split on (Store, Z)
  float* out2;
  int64_t ldo2;
  const float* aux;
  int64_t ldaux;
  int split;
  bf16_t* planes;  // Z, Dsilu: rows ldp elements apart
  int64_t ldp;
};

template <int EPI, int BM, int P>
__global__ __launch_bounds__(256) void bwd_gemm_kernel(TileMap tm, BwdGemm g) {
  using C = SplitCfg<P, BM, false>;
  __shared__ __align__(16) unsigned char smem[C::SMEM_BYTES];
  int tr, tc;
  if (!tm.map(tr, tc)) return;
  const int m0 = tr * C::BM, n0 = tc * C::BN;
  f32x4 acc[C::TM][C::TN];
  const int64_t ld = P * static_cast<int64_t>(g.K);
  split_mainloop<C>(acc, g.A, ld, g.M, g.B, ld, g.N, 0, g.K / 32, m0, n0, smem);
  gemm_epilogue<C>(
      acc, smem, m0, n0,
      [&](int row, int col0, const float(&v)[8]) -> float {
        if (row >= g.M || col0 >= g.N) return 0.f;
        float o[8];
        // bias of the column group: bias2 past split when given (8-column groups do not
        // straddle split, a multiple of 8)
        const float* bb = g.bias == nullptr ? nullptr
                          : g.bias2 != nullptr && col0 >= g.split ? g.bias2 + (col0 - g.split)
                                                                   : g.bias + col0;
        if (EPI == kEpiStore || EPI == kEpiZ) {
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = v[e] + (bb != nullptr ? bb[e] : 0.f);
          store8(g.out + static_cast<int64_t>(row) * g.ldo + col0, o);
          if (EPI == kEpiZ) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = silu_f(o[e]);
            store8(g.out2 + static_cast<int64_t>(row) * g.ldo2 + col0, o);
            if (col0 < g.split) store_planes8<kFwdPlanes>(g.planes + static_cast<int64_t>(row) * g.ldp, col0, o);
          }
        } else if (EPI == kEpiDsilu) {
          float zz[8];
          load8(g.aux + static_cast<int64_t>(row) * g.ldaux + col0, zz);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = v[e] * dsilu_f(zz[e]);
          store8(g.out + static_cast<int64_t>(row) * g.ldo + col0, o);
          store_planes8<2>(g.planes + static_cast<int64_t>(row) * g.ldp, col0, o);
        } else if (EPI == kEpiRows) {
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = v[e];
          if (row < g.split)
            store8(g.out + static_cast<int64_t>(row) * g.ldo + col0, o);
          else
            store8(g.out2 + static_cast<int64_t>(row - g.split) * g.ldo2 + col0, o);
        } else {
          if (col0 < g.split) {
            float* p = g.out + static_cast<int64_t>(row) * g.ldo + col0;
            load8(p, o);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += v[e];
            store8(p, o);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = v[e];
            store8(g.out2 + static_cast<int64_t>(row) * g.ldo2 + (col0 - g.split), o);
          }
        }
        return 0.f;
      },
      NoRowSum{});
}

}  // namespace fovea
