// Inverse of a symmetric positive definite matrix, for the Pade denominator of a
// symmetric operator: q_m(X) = V - U is a polynomial of X without zeros on
// [-theta_m, theta_m], hence positive definite where X is symmetric (its
// eigenvalues lie within ||X||_1 <= theta_m), with a condition number below
// e^theta_13 or so.
//
// Blocked Gauss-Jordan elimination by symmetric sweeps (the sweep operator of
// Beaton 1964, on 64 x 64 blocks): sweeping block k of
//   [ D  B^T ]          [ -D^-1      D^-1 B^T       ]
//   [ B  C   ]   gives  [ B D^-1     C - B D^-1 B^T ]
// and sweeping every block leaves -P^-1.  Each sweep is one symmetric update of
// the whole matrix, so no triangular solve is left and every step has the same
// parallelism; no pivots are needed for a positive definite matrix.  Only the
// lower triangle is kept up.  A sweep is three launches: the block's column
// gathered from both sides of the diagonal beside D^-1 (one workgroup), then
// W = B D^-1, which also replaces the block's row and column, then the update.
// Bound by the update's traffic (8 n^2 bytes a sweep) from n of about 4000 on
// and by the launches and D^-1 (about 20 us) below.
#include "common.h"

namespace dme {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kB = 64;

// Blocks 1..: rows 64 (blockIdx - 1) .. of the panel, P (ld ldp) = A(:, k0 ..
// k0 + 64) of the symmetric A (columns past jb zero).  Block 0: Dinv = inverse
// of the diagonal block (identity past jb) by 64 scalar sweeps; wave w holds
// rows 16 w .. of it in registers, a column per lane.  A step publishes the
// pivot's row through LDS; by symmetry it is the pivot's column too.
__global__ __launch_bounds__(256) void spd_panel_kernel(const double* __restrict__ A, int64_t ld, int n, int k0,
                                                        int jb, double* __restrict__ P, int64_t ldp,
                                                        double* __restrict__ Dinv, int* __restrict__ info) {
  __shared__ double t[kB][kB + 1];
  __shared__ alignas(16) double prow[2][kB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (blockIdx.x > 0) {
    const int i0 = (blockIdx.x - 1) * kB;
    const bool above = i0 < k0;  // (blocks are aligned: all of its rows or none)
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int c = wave + 4 * u;  // lane = the fast index of what is read
      // above: row k0 + lane of A, column i0 + c; else row i0 + lane, column k0 + c,
      // inside the block from the lower triangle
      int r = above ? k0 + lane : i0 + lane, q = above ? i0 + c : k0 + c;
      if (r < q) { const int x = r; r = q; q = x; }
      v[u] = A[min(r, n - 1) + (int64_t)min(q, n - 1) * ld];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) pin(v[u]);
    if (above) {
#pragma unroll
      for (int u = 0; u < 16; ++u) t[lane][wave + 4 * u] = v[u];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = t[wave + 4 * u][lane];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int c = wave + 4 * u;
      if (i0 + lane < n) P[i0 + lane + (int64_t)c * ldp] = c < jb ? v[u] : 0.0;
    }
    return;
  }
  double a[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = 16 * wave + i, hi = max(r, lane), lo = min(r, lane);
    a[i] = A[min(k0 + hi, n - 1) + (int64_t)min(k0 + lo, n - 1) * ld];
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    pin(a[i]);
    const int r = 16 * wave + i;
    if (max(r, lane) >= jb) a[i] = r == lane ? 1.0 : 0.0;
  }
#pragma unroll 1
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int p = 16 * g + q, par = q & 1;
      if (wave == g) prow[par][lane] = a[q];
      __syncthreads();
      const double d = prow[par][p];
      const double dinv = 1.0 / d;
      if (tid == 0 && !(d > 0.0)) atomicCAS(info, 0, k0 + p + 1);
      const bool me = lane == p;
      const double sj = me ? -dinv : prow[par][lane] * dinv;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const double ai = me ? 0.0 : a[i];
        a[i] = fma(-prow[par][16 * wave + i], sj, ai);
      }
      if (wave == g) a[q] = sj;
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) Dinv[16 * wave + i + lane * kB] = -a[i];
}

// W = P Dinv for 64 rows a workgroup (FP64 MFMA, a wave 16 rows), written to W
// and to the block's column (rows below) or row (rows above) of A; the block's
// own rows take -Dinv.
__global__ __launch_bounds__(256) void spd_w_kernel(double* __restrict__ A, int64_t ld, int n, int k0, int jb,
                                                    const double* __restrict__ P, int64_t ldp,
                                                    const double* __restrict__ Dinv, double* __restrict__ W) {
  __shared__ double sP[kB][kB + 1], sD[kB][kB + 1];  // [column][row], symmetric
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.x * kB;
  double v[16], w[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int c = wave + 4 * u;
    v[u] = P[min(i0 + lane, n - 1) + (int64_t)c * ldp];
    w[u] = Dinv[lane + c * kB];
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    sP[wave + 4 * u][lane] = v[u];
    sD[wave + 4 * u][lane] = w[u];
  }
  __syncthreads();
  const int r16 = lane & 15, kq = lane >> 4;
  v4d acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kB; k += 4) {
    const double fp = sP[k + kq][16 * wave + r16];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(sD[k + kq][16 * j + r16], fp, acc[j], 0, 0, 0);
  }
  // lane holds W(m = 16 wave + r16, c = 16 j + 4 x + kq)
  const int m = i0 + 16 * wave + r16;
  if (m >= n) return;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int c = 16 * j + 4 * x + kq;
      const double o = acc[j][x];
      W[m + (int64_t)c * ldp] = o;
      if (c >= jb) continue;
      if (m >= k0 + jb) A[m + (int64_t)(k0 + c) * ld] = o;
      else if (m < k0) A[k0 + c + (int64_t)m * ld] = o;
      else if (m >= k0 + c) A[m + (int64_t)(k0 + c) * ld] = -sD[c][m - k0];
    }
}

// out = -S of the symmetric S held in its lower triangle
__global__ __launch_bounds__(256) void spd_unfold_kernel(const double* __restrict__ S, int64_t ld, int n,
                                                         double* __restrict__ out, int64_t ldo) {
  __shared__ double t[32][33];
  const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
  if (c0 > r0) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int j = ty; j < 32; j += 8) {
    const int r = r0 + tx, c = c0 + j;
    const double v = (r < n && c < n && r >= c) ? -S[r + (int64_t)c * ld] : 0.0;
    if (r < n && c < n && r >= c) out[r + (int64_t)c * ldo] = v;
    t[j][tx] = v;
  }
  __syncthreads();
  for (int j = ty; j < 32; j += 8) {
    const int r = c0 + tx, c = r0 + j;  // the mirror image, above the diagonal
    if (r < n && c < n && r < c) out[r + (int64_t)c * ldo] = t[tx][j];
  }
}

int64_t panel_ld(int64_t n) { return n + (n & 1); }

}  // namespace

size_t spd_inverse_workspace(int64_t n) {
  return 2 * ((size_t)panel_ld(n) * kB * sizeof(double) + 256) + kB * kB * sizeof(double) + 256 +
         gemm_sym_workspace(n, kB);
}

void spd_inverse_f64(hipStream_t s, int64_t n, double* A, int64_t ld, double* out, int64_t ldo, Arena& ws,
                     int* info_dev) {
  if (n <= 0) return;
  DME_REQUIRE(n < (1ll << 30), DME_EINVAL, "symmetric inverse: dimension too large");
  const size_t mark = ws.used;
  const int64_t ldp = panel_ld(n);
  double* P = ws.get<double>((size_t)ldp * kB);
  double* W = ws.get<double>((size_t)ldp * kB);
  double* Dinv = ws.get<double>(kB * kB);
  const unsigned nb = (unsigned)cdiv(n, kB);
  for (int64_t k0 = 0; k0 < n; k0 += kB) {
    const int jb = (int)std::min<int64_t>(kB, n - k0);
    hipLaunchKernelGGL(spd_panel_kernel, dim3(nb + 1), dim3(256), 0, s, A, ld, (int)n, (int)k0, jb, P, ldp, Dinv,
                       info_dev);
    DME_HIP(hipGetLastError());
    hipLaunchKernelGGL(spd_w_kernel, dim3(nb), dim3(256), 0, s, A, ld, (int)n, (int)k0, jb, P, ldp, Dinv, W);
    DME_HIP(hipGetLastError());
    if (n > kB) gemm_sym_f64(s, 'T', n, kB, -1.0, W, ldp, P, ldp, 1.0, A, ld, false, ws, k0, k0 + jb);
  }
  const unsigned nt = (unsigned)cdiv(n, 32);
  hipLaunchKernelGGL(spd_unfold_kernel, dim3(nt, nt), dim3(256), 0, s, A, ld, (int)n, out, ldo);
  DME_HIP(hipGetLastError());
  ws.used = mark;
}

}  // namespace dme
