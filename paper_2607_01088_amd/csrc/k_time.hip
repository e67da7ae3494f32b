// Time conditioning: flow time tau -> modulation table.
//
// A call needs the modulation vectors only for its distinct flow times
// (tau = k/K over the requests' step counts), so they are computed once per
// distinct tau and looked up per row afterwards.  The weights of this stage
// (two d x d time-MLP matrices and L+1 modulation projections, about 0.23 GB in
// bf16 for the pi0 shape) are streamed once per call for all distinct taus
// together: the kernels are HBM-bound on weight bytes.
#include <algorithm>
#include <cfloat>

#include "rosa_device.h"
#include "rosa_internal.h"

namespace rosa {

// emb[t][i] = sin(1000 tau_t w_i), emb[t][half + i] = cos(1000 tau_t w_i),
// w_i = 10000^(-i/half).  Angles and sin/cos in double (the angle reaches 1000
// radians, where fp32 argument rounding alone would cost ~1e-4 absolute).
__global__ void time_embedding_kernel(const float *__restrict__ taus, int dt, float *__restrict__ emb) {
  const int t = blockIdx.y;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int half = dt / 2;
  if (i >= half) return;
  const double w = pow(10000.0, -(double)i / (double)half);
  const double a = 1000.0 * (double)taus[t] * w;
  emb[(size_t)t * dt + i] = (float)sin(a);
  emb[(size_t)t * dt + half + i] = (float)cos(a);
}

hipError_t launch_time_embedding(const float *taus, int n_tau, int dt, float *emb, hipStream_t s) {
  dim3 grid((dt / 2 + 255) / 256, n_tau);
  hipLaunchKernelGGL(time_embedding_kernel, grid, dim3(256), 0, s, taus, dt, emb);
  return hipGetLastError();
}

// Y[t][col] = act(sum_k X[t][k] W[k][col] + b[col]) for up to 16 rows t per
// pass (fp32 mode).  A thread owns two adjacent columns and uses each weight
// for all rows.  X
// is staged in LDS transposed ([k][t]), so the 16 row values of one k are four
// broadcast 16-byte LDS reads.  The kernel is bound by streaming W once; to
// keep enough bytes in flight each thread issues 16 weight loads at a time
// and K is split over blockIdx.z, the slices' partial sums being added in
// slice order by small_gemv_reduce_kernel (deterministic).
constexpr int kGemvChunk = 128;
constexpr int kGemvRows = 16;
__global__ void __launch_bounds__(256) small_gemv_kernel(const float *__restrict__ X, int n, int K,
                                                         const float *__restrict__ W, int N,
                                                         int k_per_slice, float *__restrict__ P) {
  constexpr int NT = kGemvRows;
  __shared__ __attribute__((aligned(16))) float xs[kGemvChunk][NT];
  const int col = 2 * (blockIdx.x * 256 + threadIdx.x);
  const int kb = blockIdx.z * k_per_slice, ke = min(K, kb + k_per_slice);
  float acc0[NT], acc1[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc0[t] = acc1[t] = 0.f;
  const float *Wp = W + min(col, N - 2);
  for (int k0 = kb; k0 < ke; k0 += kGemvChunk) {
    const int kn = min(kGemvChunk, ke - k0);
    __syncthreads();
    for (int i = threadIdx.x; i < kn * NT; i += 256) {
      const int kk = i / NT, t = i % NT;
      xs[kk][t] = t < n ? X[(size_t)t * K + k0 + kk] : 0.f;
    }
    __syncthreads();
    for (int kk0 = 0; kk0 < kn; kk0 += 16) {
      float w0[16], w1[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int kk = min(kk0 + u, kn - 1);
        const float2 f = *reinterpret_cast<const float2 *>(Wp + (size_t)(k0 + kk) * N);
        w0[u] = f.x;
        w1[u] = f.y;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (kk0 + u < kn) {
          const float4 *xr = reinterpret_cast<const float4 *>(&xs[kk0 + u][0]);
#pragma unroll
          for (int q = 0; q < NT / 4; ++q) {
            const float4 xv = xr[q];
            acc0[4 * q + 0] = fmaf(xv.x, w0[u], acc0[4 * q + 0]); acc1[4 * q + 0] = fmaf(xv.x, w1[u], acc1[4 * q + 0]);
            acc0[4 * q + 1] = fmaf(xv.y, w0[u], acc0[4 * q + 1]); acc1[4 * q + 1] = fmaf(xv.y, w1[u], acc1[4 * q + 1]);
            acc0[4 * q + 2] = fmaf(xv.z, w0[u], acc0[4 * q + 2]); acc1[4 * q + 2] = fmaf(xv.z, w1[u], acc1[4 * q + 2]);
            acc0[4 * q + 3] = fmaf(xv.w, w0[u], acc0[4 * q + 3]); acc1[4 * q + 3] = fmaf(xv.w, w1[u], acc1[4 * q + 3]);
          }
        }
      }
    }
  }
  if (col >= N) return;               // N is even
  float *Pz = P + (size_t)blockIdx.z * n * N;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t < n) {
      Pz[(size_t)t * N + col] = acc0[t];
      Pz[(size_t)t * N + col + 1] = acc1[t];
    }
  }
}

// Y[t][col] = act(sum over slices z in order of P[z][t][col] + b[col]).
__global__ void small_gemv_reduce_kernel(const float *__restrict__ P, int slices, int n, int N,
                                         const float *__restrict__ b, int act, float *__restrict__ Y) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)n * N) return;
  float v = P[i];
  for (int z = 1; z < slices; ++z) v += P[(size_t)z * n * N + i];
  v += b ? b[i % N] : 0.f;
  if (act == 1) v = silu_f(v);
  Y[i] = v;
}

size_t small_gemv_workspace_floats(int N) { return (size_t)kGemvMaxSlices * kGemvRows * N; }

hipError_t launch_small_gemv(const float *X, int n, int K, const float *W, const float *b, int N, int act, float *Y,
                             float *ws, hipStream_t s) {
  if (N % 2) return hipErrorInvalidValue;
  for (int t0 = 0; t0 < n; t0 += kGemvRows) {
    const int nt = std::min(kGemvRows, n - t0);
    const int cols = (N / 2 + 255) / 256;
    // Enough blocks to keep ~1000 in flight, each slice at least one chunk of K.
    const int want = std::max(1, std::min((1024 + cols - 1) / cols, kGemvMaxSlices));
    const int kps = ((K + want - 1) / want + kGemvChunk - 1) / kGemvChunk * kGemvChunk;
    const int slices = (K + kps - 1) / kps;
    dim3 grid(cols, 1, slices);
    hipLaunchKernelGGL(small_gemv_kernel, grid, dim3(256), 0, s, X + (size_t)t0 * K, nt, K, W, N, kps, ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t total = (size_t)nt * N;
    hipLaunchKernelGGL(small_gemv_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, ws, slices,
                       nt, N, b, act, Y + (size_t)t0 * N);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------ bf16 weights
// Y[t][col] = act(sum_k X[t][k] W[k][col] + b[col]) for up to 16 rows t of fp32 X
// and bf16 W (kb32, K padded to 32), on the matrix cores without giving up
// fp32 inputs: X = hi + mid + lo in bf16, each the rounded remainder of
// the ones before (24 bits and more together), so three
// v_mfma_f32_16x16x32_bf16 per weight fragment form the exact products and
// accumulate them in fp32.  Values beyond bf16's range have no such split (inf - inf,
// or 0 times an infinite weight): four outputs among which one comes out infinite or NaN
// are summed again from X itself.  The eight waves split K; a wave keeps its share of X
// (up to 128 of K) in registers and streams weights: CT tiles of 16 columns per
// step, every load of the next step in flight while the waves' partial sums meet in
// LDS and are added in wave order.  Bound by streaming W once: the 0.23 GB
// modulation weights take 54 us (a kernel on the vector units took 79 and a reduction
// launch 5), a 2 MB time-MLP matrix 9 us (28).
constexpr int kTauRows = 16, kTauWaves = 8, kTauSteps = 4;
template <int CT>
__global__ void __launch_bounds__(64 * kTauWaves) tau_gemm_kernel(const float *__restrict__ X, int ldx, size_t x_stride,
                                                                  int n_rows, int K, const bf16 *__restrict__ W,
                                                                  size_t w_stride, int N, const float *__restrict__ b,
                                                                  int act, float *__restrict__ Y, int ldy,
                                                                  size_t y_stride, int vec) {
  constexpr int LDR = 20;                   // floats per staged row of 16 (padded)
  __shared__ __attribute__((aligned(16))) float red[2][kTauWaves][CT][16 * LDR];
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t0 = blockIdx.z * kTauRows, n = min(kTauRows, n_rows - t0);
  X += blockIdx.y * x_stride + (size_t)t0 * ldx;
  W += blockIdx.y * w_stride;
  Y += blockIdx.y * y_stride + (size_t)t0 * ldy;
  const int T = (K + 31) >> 5;              // steps of 32 of K, in chunks of 8 kTauSteps
  const int n_chunks = (T + kTauWaves * kTauSteps - 1) / (kTauWaves * kTauSteps);
  auto share = [&](int c, int &lo, int &cnt) __attribute__((always_inline)) {
    const int s0 = c * kTauWaves * kTauSteps, tc = min(kTauWaves * kTauSteps, T - s0);
    lo = s0 + tc * wave / kTauWaves;
    cnt = s0 + tc * (wave + 1) / kTauWaves - lo;
  };
  // Lane holds row lane % 16, K values 8 (lane / 16) .. + 7 of each step.
  bf16x8 xh[kTauSteps], xm[kTauSteps], xl[kTauSteps];
  auto load_x = [&](int lo, int cnt) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < kTauSteps; ++s) {
      float v[8];
      const int k = (lo + s) * 32 + 8 * q4;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (s < cnt && r16 < n && k + j < K) ? X[(size_t)r16 * ldx + k + j] : 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bf16 h = (bf16)v[j];
        const float r1 = v[j] - (float)h;
        const bf16 m = (bf16)r1;
        xh[s][j] = h;
        xm[s][j] = m;
        xl[s][j] = (bf16)(r1 - (float)m);
      }
    }
  };
  bf16x8 wv[kTauSteps][CT];
  auto load_w = [&](int g, int lo, int cnt) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < kTauSteps; ++s)
#pragma unroll
      for (int c = 0; c < CT; ++c)
        if (s < cnt) {
          const int col = min((g * CT + c) * 16, N - 16) + r16;
          wv[s][c] = *reinterpret_cast<const bf16x8 *>(W + ((size_t)(lo + s) * N + col) * 32 + 8 * q4);
        }
  };
  const int n_groups = (N / 16 + CT - 1) / CT;
  int lo, cnt;
  share(0, lo, cnt);
  int g = blockIdx.x;
  if (g < n_groups) load_w(g, lo, cnt);
  load_x(lo, cnt);
  for (int it = 0; g < n_groups; ++it, g += gridDim.x) {
    f32x4 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int ch = 0; ch < n_chunks; ++ch) {
      if (n_chunks > 1) {                   // the share of X changes with the chunk
        share(ch, lo, cnt);
        load_w(g, lo, cnt);
        load_x(lo, cnt);
      }
#pragma unroll
      for (int s = 0; s < kTauSteps; ++s)
        if (s < cnt) {
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[s][c], xl[s], acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[s][c], xm[s], acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[s][c], xh[s], acc[c], 0, 0, 0);
          }
        }
    }
    if (n_chunks == 1 && g + (int)gridDim.x < n_groups) load_w(g + gridDim.x, lo, cnt);
    // Lane holds row (t) lane % 16, columns 4 (lane / 16) .. + 3 of each tile.  Two
    // staging buffers: a buffer is written again only after the other's barrier.
    float(*rb)[CT][16 * LDR] = red[it & 1];
#pragma unroll
    for (int c = 0; c < CT; ++c) *reinterpret_cast<f32x4 *>(&rb[wave][c][r16 * LDR + 4 * q4]) = acc[c];
    __syncthreads();
    if (tid < CT * 64) {
      const int c = tid >> 6, t = (tid & 63) >> 2, c4 = (tid & 3) * 4, col = (g * CT + c) * 16 + c4;
      f32x4 v = *reinterpret_cast<const f32x4 *>(&rb[0][c][t * LDR + c4]);
#pragma unroll
      for (int w = 1; w < kTauWaves; ++w) {
        const f32x4 p = *reinterpret_cast<const f32x4 *>(&rb[w][c][t * LDR + c4]);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += p[k];
      }
      if (t < n && col < N) {
        const bool finite = fabsf(v[0]) <= FLT_MAX && fabsf(v[1]) <= FLT_MAX && fabsf(v[2]) <= FLT_MAX && fabsf(v[3]) <= FLT_MAX;
        if (__builtin_expect(!finite, 0)) {
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = 0.f;
          for (int i = 0; i < K; ++i) {
            const float x = X[(size_t)t * ldx + i];
#pragma unroll
            for (int k = 0; k < 4; ++k)
              v[k] = fmaf(x, (float)W[((size_t)(i >> 5) * N + col + k) * 32 + (i & 31)], v[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (b) v[k] += b[col + k];
          if (act == 1) v[k] = silu_f(v[k]);
        }
        float *y = Y + (size_t)t * ldy + col;
        if (vec) {
          *reinterpret_cast<f32x4 *>(y) = v;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) y[k] = v[k];
        }
      }
    }
  }
}

hipError_t launch_tau_gemm(const float *X, int ldx, size_t x_stride, int n, int K, const void *W, size_t w_stride, int N,
                           const float *b, int act, float *Y, int ldy, size_t y_stride, int n_mat, hipStream_t s) {
  if (n <= 0 || n_mat <= 0) return hipSuccess;
  if (K < 1 || N < 16 || N % 16) return hipErrorInvalidValue;
  const int vec = ldy % 4 == 0 && y_stride % 4 == 0 && ((uintptr_t)Y & 15) == 0;   // 16-byte stores
  const int chunks = (n + kTauRows - 1) / kTauRows;
  // Wide matrices 64 columns per step over at most 256 persistent blocks (two
  // steps each when many matrices share the launch); narrow ones 16 per block.
  if (N >= 2048) {
    const int groups = (N + 63) / 64;
    const int blocks = n_mat > 1 ? (groups + 1) / 2 : std::min(groups, 256);
    hipLaunchKernelGGL(tau_gemm_kernel<4>, dim3(blocks, n_mat, chunks), dim3(64 * kTauWaves), 0, s, X, ldx, x_stride, n, K,
                       (const bf16 *)W, w_stride, N, b, act, Y, ldy, y_stride, vec);
  } else {
    hipLaunchKernelGGL(tau_gemm_kernel<1>, dim3(N / 16, n_mat, chunks), dim3(64 * kTauWaves), 0, s, X, ldx, x_stride, n, K,
                       (const bf16 *)W, w_stride, N, b, act, Y, ldy, y_stride, vec);
  }
  return hipGetLastError();
}

}  // namespace rosa
