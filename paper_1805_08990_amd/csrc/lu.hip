// Dense LU with row exchanges and the multi-right-hand-side solve used for the
// Pade denominator of the matrix exponential, (V - U) F = V + U, and for the mass
// matrix.  Pivots are chosen a panel at a time by a tournament (communication
// avoiding LU, Grigori, Demmel and Xiang 2011); in one level that is partial
// pivoting, in more its bound on the growth of the entries is weaker.
//
// Blocked right-looking factorisation, 64 columns a block, applied to the
// right-hand sides as it goes (they are further columns of the trailing
// matrix), so that L is not needed afterwards and the only substitution left
// is the backward one with U.  A block is two 32-column panels:
//   select : the panel's 32 pivot rows by a tournament.  A wave holds up to 192
//            rows of the panel in registers, eliminates with partial pivoting
//            (largest |a|, first row on ties) and names its 32 pivot rows; the
//            rows named by all waves play the next level until one wave is
//            left, whose elimination is the factor of the diagonal block.  Up to
//            192 rows are one level, which is plain partial pivoting.
//   rows   : L21 = A21 inv(U11) for the rows below, the rows that gave way to
//            pivots moved to the places those left, and for the first panel the
//            update of the second one's columns.
//   cols   : the remaining columns and the right-hand sides: both panels' row
//            moves and U12 = inv(L11) A12.
//   A22    : A22 - L21 U12 and the same of the right-hand sides (FP64 MFMA).
// The kept form rounds every entry as the method's first implementation did with
// the same pivots (a division per multiplier, block triangles applied through
// their inverses by products), for callers whose results depend on the last bit
// (Solver::kept).
// What bounds it: up to n of a few thousand the chain of panels (a launch pair
// per column takes 18 us a column; at n = 4096 a 64-column block of this takes
// 180 us and the whole solve 17 ms instead of 95); beyond that the trailing
// update's traffic.
#include "common.h"

#include <type_traits>

namespace dme {
namespace {

constexpr int kPW = 32;          // panel width
constexpr int kNB = 2 * kPW;     // block width
constexpr int kLeaf = 192;       // rows a wave of the tournament holds at most

// Row moves of one panel (positions are global rows): pivot t's row was at
// piv[t]; the rows src[q] of the panel's top that are not pivots go to the
// places dst[q] below it that pivots left (dst[q] = -1: no more).
struct Moves {
  int piv[kPW];
  int dst[kPW];
  int src[kPW];
};

// Several systems of one size at a time: system blockIdx.y has its arrays that
// many entries after those of the first.  The chain of panels is bound by its
// latency up to n of a few thousand, so more systems take little more time.
struct Systems {
  int64_t a = 0, q = 0;          // matrix, right-hand sides
  int64_t blk = 0;               // diagonal blocks (and their inverses)
  int64_t tmp = 0;               // moved block rows
  int list = 0, mv = 0, lbuf = 0;
};

// value of lane S of each aligned group of four
template <int S>
__device__ inline double quad_bcast_f64(double v) {
  return dpp_mov_f64<S * 0x55>(v);
}

// Forward substitution with a triangular block, a vector of 4 NJ entries per
// quad of lanes: lane q of the quad holds entries 4 j + q in x[j].  Step c
// takes entry c as it stands (times sR[c] where SCALE), p, and subtracts
// sM[c][i] p from the entries i > c; sM (rows of 4 NJ, 4 NJ more readable behind
// the last one) holds zeros for i <= c in c's group of four.  Every fourth step
// hands the four finished entries to put(k, value) and shifts the vector down,
// so the loop body is short and has no register indexed by the step (the
// straight-line form ran at the rate its instructions could be fetched).
// Entries shifted in past the end are never used.  4 * groups steps.
// DIVIDE: sR holds the divisors themselves (0: the entry becomes 0).
template <int NJ, bool SCALE, bool DIVIDE = false, class Put>
__device__ inline void quad_substitute(double (&x)[NJ], int groups, const double* sM, const double* sR, int q, Put put) {
#pragma unroll 1
  for (int k = 0; k < groups; ++k) {
    const double* mk = sM + 4 * k * (4 * NJ) + 4 * k + q;
    auto step = [&](auto sc) {
      constexpr int S = decltype(sc)::value;
      double p = quad_bcast_f64<S>(x[0]);
      if (SCALE) {
        if (DIVIDE) p = sR[4 * k + S] != 0.0 ? p / sR[4 * k + S] : 0.0;
        else p *= sR[4 * k + S];
        if (q == S) x[0] = p;
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) x[j] = fma(-mk[S * 4 * NJ + 4 * j], p, x[j]);
    };
    step(std::integral_constant<int, 0>());
    step(std::integral_constant<int, 1>());
    step(std::integral_constant<int, 2>());
    step(std::integral_constant<int, 3>());
    put(k, x[0]);
#pragma unroll
    for (int j = 0; j + 1 < NJ; ++j) x[j] = x[j + 1];
  }
}

// largest value of the wave, in every lane
__device__ inline uint32_t wave_max_u32(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor1, 0xF, 0xF, true));
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor2, 0xF, 0xF, true));
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppHalfMirror, 0xF, 0xF, true));
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppMirror, 0xF, 0xF, true));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = max(b[0], b[1]);
#endif
  return v;
}
// v of lane l (uniform), as a scalar
__device__ inline double readlane_f64(double v, int l) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// The first lane with the largest v >= 0 (v < 0: not playing), -1 if none
// plays: by the upper words, and by the lower ones only where those tie.
__device__ inline int wave_argmax(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t hi = v >= 0.0 ? (uint32_t)(b >> 32) + 1u : 0u;
  const uint32_t mh = __builtin_amdgcn_readfirstlane(wave_max_u32(hi));
  if (mh == 0) return -1;
  unsigned long long who = __ballot(hi == mh);
  if (__popcll(who) > 1) {
    const uint32_t lo = hi == mh ? (uint32_t)b : 0u;
    const uint32_t ml = __builtin_amdgcn_readfirstlane(wave_max_u32(lo));
    who = __ballot(hi == mh && lo == ml);
  }
  return __ffsll(who) - 1;
}

// One level of the tournament for panel columns [c0, c0 + jb).  The players are
// rows r0, r0 + 1, ... < n (cand == nullptr) or cand[0 .. ncand) (-1: none); a
// workgroup is one wave and takes the 64 R players from 64 R blockIdx on, R
// rows a lane.  The step is a latency chain, so it has no barrier and no LDS
// round trip in it: the wave finds the pivot by lane moves, reads the pivot row
// from its lane into scalar registers and eliminates with those as operands
// (four waves that exchanged candidate rows through LDS took 1.0 us a step for
// 256 rows; this takes 0.7 us for 192, 28 us a launch).  A lane keeps its rows shifted so that the pivot
// column is always entry 0 (no register is indexed by the step): a step writes
// entry i from entry i + 1, so a row that becomes pivot t holds columns t .. 31
// and zeros; the multipliers go to lbuf.
// fin == 0: the pivot rows go to out[32 b ...).  fin != 0 (one workgroup): the
// factor of the diagonal block goes to blk + o (1 + kNB) (ld kNB, o the
// panel's offset in its block), the row moves to mv, and
//   o == 0: U12 of the block's second panel (columns c0 + 32 .. c0 + 32 + jb2)
//   o > 0 : the pivot rows' multipliers of the first panel
// to the rest of the panel's rows of blk.
template <int R>
__global__ __launch_bounds__(64) void lu_select_kernel(const double* __restrict__ A, int64_t lda, int n, int r0,
                                                       int c0, int jb, const int* __restrict__ cand, int ncand,
                                                       int* __restrict__ out, int fin, int o, int jb2,
                                                       double* __restrict__ blk, Moves* __restrict__ mv,
                                                       double* lbuf, int* __restrict__ info, Systems sys) {
  A += blockIdx.y * sys.a;
  if (cand) cand += blockIdx.y * sys.list;
  out += blockIdx.y * sys.list;
  blk += blockIdx.y * sys.blk;
  mv += blockIdx.y * sys.mv;
  lbuf += blockIdx.y * sys.lbuf;
  __shared__ alignas(16) double srow[kPW][kPW + 2];  // the pivot rows, shifted
  __shared__ double sM[kPW * kPW + kPW];
  __shared__ int spiv[kPW], swho[kPW];
  const int lane = threadIdx.x;
  int row[R];
  double a[R][kPW];
  const int q0 = (blockIdx.x * 64 + lane) * R;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    row[u] = -1;
    if (cand) row[u] = q0 + u < ncand ? cand[q0 + u] : -1;
    else if (q0 + u < n - r0) row[u] = r0 + q0 + u;
  }
  const int last = jb - 1;
#pragma unroll
  for (int c = 0; c < kPW; ++c)
#pragma unroll
    for (int u = 0; u < R; ++u) a[u][c] = A[max(row[u], 0) + (int64_t)(c0 + min(c, last)) * lda];
#pragma unroll
  for (int c = 0; c < kPW; ++c)
#pragma unroll
    for (int u = 0; u < R; ++u) {
      pin(a[u][c]);
      if (row[u] < 0 || c >= jb) a[u][c] = 0.0;
    }
  int place[R];  // the step at which the row became a pivot
#pragma unroll
  for (int u = 0; u < R; ++u) place[u] = -1;
  if (lane < kPW) spiv[lane] = -1;
  // steps [t0, t1), of rows with LEN columns left at t0
  auto steps = [&](auto lenc, int t0, int t1) {
    constexpr int LEN = decltype(lenc)::value;
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
      // the lane's largest |entry 0| of a row still playing, the first on ties;
      // NaN counts as zero here (it reaches the result, which is checked)
      double v = -1.0;
      int ub = 0;
#pragma unroll
      for (int u = 0; u < R; ++u) {
        double x = fabs(a[u][0]);
        x = row[u] >= 0 ? (x >= 0.0 ? x : 0.0) : -1.0;
        if (x > v) { v = x; ub = u; }
      }
      const int lead = wave_argmax(v);
      if (lead < 0) return;  // no player left (uniform)
      const int uw = __builtin_amdgcn_readlane(ub, lead);
      double pr[LEN];
#pragma unroll
      for (int u = 0; u < R; ++u)
        if (R == 1 || uw == u) {  // uniform
#pragma unroll
          for (int c = 0; c < LEN; ++c) pr[c] = readlane_f64(a[u][c], lead);
          if (lane == lead) {
            spiv[t] = row[u];
            swho[t] = lane * R + u;
            row[u] = -1;
            place[u] = t;
          }
        }
      const double pv = pr[0];
#pragma unroll
      for (int u = 0; u < R; ++u)
        if (row[u] >= 0) {  // (a pivot's row stays as it was)
          const double l = pv != 0.0 ? a[u][0] / pv : 0.0;
#pragma unroll
          for (int c = 0; c + 1 < LEN; ++c) a[u][c] = fma(-l, pr[c + 1], a[u][c + 1]);
          if (fin) lbuf[(t * R + u) * 64 + lane] = l;
        }
    }
  };
  // (entries past a row's LEN are stale, and so are those past its end)
  steps(std::integral_constant<int, 32>(), 0, min(jb, 8));
  steps(std::integral_constant<int, 24>(), 8, min(jb, 16));
  steps(std::integral_constant<int, 16>(), 16, min(jb, 24));
  steps(std::integral_constant<int, 8>(), 24, jb);
  if (fin) {
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (place[u] >= 0) {
#pragma unroll
        for (int c = 0; c < kPW; ++c) srow[place[u]][c] = a[u][c];
      }
  }
  __syncthreads();
  if (!fin) {
    if (lane < kPW) out[blockIdx.x * kPW + lane] = spiv[lane];
    return;
  }
  // (at least jb players, so every pivot is there)
  const int p = lane < jb ? spiv[lane] : -1;
  if (lane < jb && !(fabs(srow[lane][0]) > 0.0)) atomicCAS(info, 0, c0 + lane + 1);  // zero (or NaN) pivot column
  constexpr int kEach = kPW * kPW / 64;
  double w[kEach];
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int e = lane + u * 64, i = e % kPW, c = e / kPW, ii = i < jb ? i : 0;
    const double lo = c < jb ? lbuf[(c * R + swho[ii] % R) * 64 + swho[ii] / R] : 0.0;
    const double up = srow[ii][c >= i ? c - i : 0];
    w[u] = (i < jb && c < jb) ? (c < i ? lo : up) : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int e = lane + u * 64, i = e % kPW, c = e / kPW;
    sM[e] = c < i ? w[u] : 0.0;
    // a column past jb of a narrow panel is not part of the factor
    if (i < jb && c < jb) blk[o + i + (o + c) * kNB] = w[u];
  }
  {
    // places that pivots left below the panel's top, and top rows that are no
    // pivots, both in order: as many of the one as of the other
    const bool below = p >= r0 + jb;
    const unsigned long long mb = __ballot(below);
    bool is_piv = lane >= jb;
#pragma unroll
    for (int t = 0; t < kPW; ++t)
      if (t < jb && spiv[t] == r0 + lane) is_piv = true;
    const unsigned long long ms = __ballot(!is_piv);
    const unsigned long long lt = (1ull << lane) - 1;
    const int nb = __popcll(mb);
    if (lane < kPW) mv->piv[lane] = p;
    if (below) mv->dst[__popcll(mb & lt)] = p;
    if (!is_piv) mv->src[__popcll(ms & lt)] = r0 + lane;
    if (lane < kPW && lane >= nb) {
      mv->dst[lane] = -1;
      mv->src[lane] = r0;
    }
  }
  if (o == 0) {  // a column of the second panel per quad (jb = 32 when there is one)
    if (jb2 <= 0) return;
    __syncthreads();
    const int q = lane & 3;
    double x[2][kPW / 4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = 16 * h + (lane >> 2), cc = c < jb2 ? c : 0;
#pragma unroll
      for (int j = 0; j < kPW / 4; ++j) x[h][j] = A[spiv[4 * j + q] + (int64_t)(c0 + kPW + cc) * lda];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = 16 * h + (lane >> 2);
      quad_substitute<kPW / 4, false>(x[h], kPW / 4, sM, nullptr, q, [&](int k, double v) {
        if (c < jb2) blk[4 * k + q + (kPW + c) * kNB] = v;
      });
    }
  } else {
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int e = lane + u * 64, i = e % kPW, c = e / kPW;
      w[u] = A[spiv[i < jb ? i : 0] + (int64_t)(c0 - kPW + c) * lda];
    }
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int e = lane + u * 64, i = e % kPW, c = e / kPW;
      if (i < jb) blk[o + i + c * kNB] = w[u];
    }
  }
}

// Rows below panel o (0 or kPW) of the block at j0: a row per quad of lanes,
// read from its own place or, where a pivot left, from the row moved there.
// l = a inv(U) by substitution; o == 0 also updates the row's jb2 columns of
// the second panel (they are the vector's second half), o > 0 also moves the
// multipliers of the first one.  Only the place itself is written, and moved
// rows come from the panel's top, which is not.
constexpr int kQuadT = 128;
template <int O, bool KEPT>
__global__ __launch_bounds__(kQuadT) void lu_rows_kernel(double* __restrict__ A, int64_t lda, int n, int j0, int jb,
                                                         int jb2, const double* __restrict__ blk,
                                                         const Moves* __restrict__ mv, Systems sys) {
  A += blockIdx.y * sys.a;
  blk += blockIdx.y * sys.blk;
  mv += blockIdx.y * sys.mv;
  constexpr int LEN = O == 0 ? kNB : kPW, NJ = LEN / 4;
  __shared__ double sM[kPW * LEN + LEN], sR[kPW];
  __shared__ alignas(16) int sdst[kPW], ssrc[kPW];
  const int tid = threadIdx.x;
  double st[kPW * LEN / kQuadT];
#pragma unroll
  for (int u = 0; u < kPW * LEN / kQuadT; ++u) {
    const int e = tid + u * kQuadT, i = e % LEN, c = e / LEN;
    st[u] = blk[O + c + (O + i) * kNB];
  }
#pragma unroll
  for (int u = 0; u < kPW * LEN / kQuadT; ++u) {
    const int e = tid + u * kQuadT, i = e % LEN, c = e / LEN;  // step c, column i of the vector
    double v = st[u];
    pin(v);
    const bool in = c < jb && (i < kPW ? i > c && i < jb : i - kPW < jb2);
    sM[e] = in ? v : 0.0;
  }
  if (tid < kPW) {
    const double d = blk[(O + tid) * (kNB + 1)];
    sR[tid] = tid < jb && d != 0.0 ? (KEPT ? d : 1.0 / d) : 0.0;
    sdst[tid] = mv->dst[tid];
    ssrc[tid] = mv->src[tid];
  }
  __syncthreads();
  const int q = tid & 3;
  const int i = j0 + O + jb + blockIdx.x * (kQuadT / 4) + (tid >> 2);
  if (i >= n) return;
  int from = i;
#pragma unroll
  for (int t = 0; t < kPW; ++t)
    if (sdst[t] == i) from = ssrc[t];
  double* Ai = A + i + (int64_t)j0 * lda;
  const double* Af = A + from + (int64_t)j0 * lda;
  auto inside = [&](int e) { return e < kPW ? e < jb : e - kPW < jb2; };
  double x[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) x[j] = Af[(int64_t)(O + (inside(4 * j + q) ? 4 * j + q : 0)) * lda];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    pin(x[j]);
    if (!inside(4 * j + q)) x[j] = 0.0;
  }
  if (O > 0 && from != i) {
    double y[kPW / 4];
#pragma unroll
    for (int j = 0; j < kPW / 4; ++j) y[j] = Af[(int64_t)(4 * j + q) * lda];
#pragma unroll
    for (int j = 0; j < kPW / 4; ++j) Ai[(int64_t)(4 * j + q) * lda] = y[j];
  }
  quad_substitute<NJ, true, KEPT>(x, kPW / 4, sM, sR, q, [&](int k, double v) {
    if (4 * k + q < jb) Ai[(int64_t)(O + 4 * k + q) * lda] = v;
  });
  if (O == 0) {
#pragma unroll
    for (int j = 0; j < kPW / 4; ++j)
      if (4 * j + q < jb2) Ai[(int64_t)(kPW + 4 * j + q) * lda] = x[j];
  }
}

// A column per quad: both panels' row moves, then U12 = inv(L11) (unit lower)
// of the block's rows.  The columns are c0.. of X (ncols) and all of Q (nq).
// A quad's lanes run in step, so its pivot rows are all read before the places
// they leave are filled, and the block's own rows are written last.
__device__ inline void move_rows(double* col, const Moves& mv, int q) {
  if (mv.dst[0] < 0) return;
  double w[kPW / 4];
  int d[kPW / 4];
#pragma unroll
  for (int j = 0; j < kPW / 4; ++j) {
    d[j] = mv.dst[4 * j + q];
    w[j] = col[mv.src[4 * j + q]];
  }
#pragma unroll
  for (int j = 0; j < kPW / 4; ++j)
    if (d[j] >= 0) col[d[j]] = w[j];
  __threadfence_block();  // another lane of the quad reads what this one moved
}
// tmp (optional): the moved block rows go there unsolved, jb x (ncols + nq).
__global__ __launch_bounds__(kQuadT) void lu_cols_kernel(double* X, int64_t ldx, int c0, int ncols, double* Q,
                                                         int64_t ldq, int nq, int j0, int jb,
                                                         const double* __restrict__ blk,
                                                         const Moves* __restrict__ mv, double* __restrict__ tmp,
                                                         Systems sys) {
  X += blockIdx.y * sys.a;
  Q += blockIdx.y * sys.q;
  blk += blockIdx.y * sys.blk;
  mv += blockIdx.y * sys.mv;
  if (tmp) tmp += blockIdx.y * sys.tmp;
  __shared__ double sM[kNB * kNB + kNB];
  __shared__ Moves smv[2];
  const int jb1 = min(jb, kPW), jb2 = jb - jb1;
  double st[kNB * kNB / kQuadT];
#pragma unroll
  for (int u = 0; u < kNB * kNB / kQuadT; ++u) st[u] = blk[threadIdx.x + u * kQuadT];
#pragma unroll
  for (int u = 0; u < kNB * kNB / kQuadT; ++u) pin(st[u]);
#pragma unroll
  for (int u = 0; u < kNB * kNB / kQuadT; ++u) {
    const int e = threadIdx.x + u * kQuadT, i = e % kNB, c = e / kNB;
    const double v = st[u];
    sM[e] = (i < jb && c < i) ? v : 0.0;
  }
  {
    const int* from = reinterpret_cast<const int*>(mv);
    int* to = reinterpret_cast<int*>(smv);
    const int have = (jb2 > 0 ? 2 : 1) * (int)(sizeof(Moves) / sizeof(int));
    for (int e = threadIdx.x; e < have; e += kQuadT) to[e] = from[e];
  }
  __syncthreads();
  const int q = threadIdx.x & 3;
  const int id = blockIdx.x * (kQuadT / 4) + (threadIdx.x >> 2);
  if (id >= ncols + nq) return;
  double* col = id < ncols ? X + (int64_t)(c0 + id) * ldx : Q + (int64_t)(id - ncols) * ldq;
  double x[kNB / 4];
#pragma unroll
  for (int j = 0; j < kPW / 4; ++j) {
    const int t = 4 * j + q;
    x[j] = col[t < jb1 ? smv[0].piv[t] : j0];
  }
#pragma unroll
  for (int j = 0; j < kPW / 4; ++j) {
    pin(x[j]);
    if (4 * j + q >= jb1) x[j] = 0.0;
  }
  move_rows(col, smv[0], q);
#pragma unroll
  for (int j = 0; j < kPW / 4; ++j) {
    const int t = 4 * j + q;
    x[kPW / 4 + j] = col[t < jb2 ? smv[1].piv[t] : j0];
  }
#pragma unroll
  for (int j = 0; j < kPW / 4; ++j) {
    pin(x[kPW / 4 + j]);
    if (4 * j + q >= jb2) x[kPW / 4 + j] = 0.0;
  }
  if (jb2 > 0) move_rows(col, smv[1], q);
  if (tmp) {
#pragma unroll
    for (int j = 0; j < kNB / 4; ++j) {
      // (the panels' rows are 32 apart in x, whatever jb is)
      const int t = 4 * j + q;
      if (t < jb) tmp[t + (int64_t)id * jb] = x[j];
    }
    return;
  }
  quad_substitute<kNB / 4, false>(x, kNB / 4, sM, nullptr, q, [&](int k, double v) {
    if (4 * k + q < jb) col[j0 + 4 * k + q] = v;
  });
}

// Backward substitution with one block's U, a column of Q per quad, as a
// forward one on the reversed order: Q[j0 .. j0 + jb) <- inv(U11) Q[j0 .. j0 + jb).
__global__ __launch_bounds__(kQuadT) void lu_back_kernel(double* __restrict__ Q, int64_t ldq, int nq, int j0, int jb,
                                                         const double* __restrict__ blk, Systems sys) {
  Q += blockIdx.y * sys.q;
  blk += blockIdx.y * sys.blk;
  __shared__ double sM[kNB * kNB + kNB], sR[kNB];
  double st[kNB * kNB / kQuadT];
#pragma unroll
  for (int u = 0; u < kNB * kNB / kQuadT; ++u) st[u] = blk[threadIdx.x + u * kQuadT];
#pragma unroll
  for (int u = 0; u < kNB * kNB / kQuadT; ++u) pin(st[u]);
#pragma unroll
  for (int u = 0; u < kNB * kNB / kQuadT; ++u) {
    const int e = threadIdx.x + u * kQuadT, i = e % kNB, c = e / kNB;  // row i, column c of U
    const double v = st[u];
    sM[(kNB - 1 - c) * kNB + kNB - 1 - i] = (c < jb && i < c) ? v : 0.0;
  }
  if (threadIdx.x < kNB) {
    const int c = threadIdx.x;
    sR[kNB - 1 - c] = c < jb ? 1.0 / blk[c * (kNB + 1)] : 1.0;
  }
  __syncthreads();
  const int q = threadIdx.x & 3;
  const int id = blockIdx.x * (kQuadT / 4) + (threadIdx.x >> 2);
  if (id >= nq) return;
  double* col = Q + (int64_t)id * ldq + j0;
  double x[kNB / 4];
#pragma unroll
  for (int j = 0; j < kNB / 4; ++j) {
    const int t = kNB - 1 - (4 * j + q);
    x[j] = col[t < jb ? t : 0];
  }
#pragma unroll
  for (int j = 0; j < kNB / 4; ++j) {
    pin(x[j]);
    if (kNB - 1 - (4 * j + q) >= jb) x[j] = 0.0;
  }
  quad_substitute<kNB / 4, true>(x, kNB / 4, sM, sR, q, [&](int k, double v) {
    const int t = kNB - 1 - (4 * k + q);
    if (t < jb) col[t] = v;
  });
}

// Xl = inverse of the block's unit lower triangle (KEPT form): a column of it
// per quad, by the sums of each entry in ascending order.
__global__ __launch_bounds__(4 * kNB) void lu_linv_kernel(const double* __restrict__ blk, int jb, double* __restrict__ Xl,
                                                          Systems sys) {
  blk += blockIdx.y * sys.blk;
  Xl += blockIdx.y * (int64_t)kNB * kNB;
  __shared__ double sM[kNB * kNB + kNB];
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < kNB / 4; ++u) {
    const int e = tid + u * 4 * kNB, i = e % kNB, c = e / kNB;
    double v = blk[e];
    pin(v);
    sM[e] = (i < jb && c < i) ? v : 0.0;
  }
  __syncthreads();
  const int q = tid & 3, c = tid >> 2;
  double x[kNB / 4];
#pragma unroll
  for (int j = 0; j < kNB / 4; ++j) x[j] = 4 * j + q == c ? 1.0 : 0.0;
  quad_substitute<kNB / 4, false>(x, kNB / 4, sM, nullptr, q, [&](int k, double v) {
    if (4 * k + q < jb && c < jb) Xl[4 * k + q + c * jb] = v;
  });
}

// Xu = inverses of the blocks' upper triangles (KEPT form), one block a
// workgroup, a column per thread, each entry one dot product in ascending order.
__global__ __launch_bounds__(kNB) void lu_uinv_kernel(const double* __restrict__ blks, int n, double* __restrict__ Xu,
                                                      Systems sys) {
  blks += blockIdx.y * sys.blk;
  Xu += blockIdx.y * sys.blk;
  __shared__ double s[kNB * kNB];
  __shared__ double x[kNB * (kNB + 1)];
  const int b = min(kNB, n - (int)blockIdx.x * kNB);
  const double* T = blks + (int64_t)blockIdx.x * kNB * kNB;
  double* X = Xu + (int64_t)blockIdx.x * kNB * kNB;
  for (int idx = threadIdx.x; idx < kNB * kNB; idx += kNB) s[idx] = T[idx];
  __syncthreads();
  const int c = threadIdx.x;
  if (c < b) {
    double* xc = x + c * (kNB + 1);
    for (int r = 0; r < b; ++r) xc[r] = 0.0;
    xc[c] = 1.0 / s[c + c * kNB];
    for (int r = c - 1; r >= 0; --r) {
      double acc = 0.0;
      for (int t = r + 1; t <= c; ++t) acc += s[r + t * kNB] * xc[t];
      xc[r] = -acc / s[r + r * kNB];
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < b * b; idx += kNB) X[idx] = x[idx % b + (idx / b) * (kNB + 1)];
}

// tmp = the jb rows of Q from j0 on (KEPT form), jb x nq.
__global__ __launch_bounds__(256) void lu_take_rows_kernel(const double* __restrict__ Q, int64_t ldq, int nq, int jb,
                                                           double* __restrict__ tmp, Systems sys) {
  Q += blockIdx.y * sys.q;
  tmp += blockIdx.y * sys.tmp;
  const int r = threadIdx.x % kNB, c = blockIdx.x * (256 / kNB) + threadIdx.x / kNB;
  if (r < jb && c < nq) tmp[r + (int64_t)c * jb] = Q[r + (int64_t)c * ldq];
}

// players a level of the tournament hands on
int64_t lu_named(int64_t players) { return cdiv(players, kLeaf) * kPW; }

}  // namespace

size_t lu_solve_workspace(int64_t n) { return lu_solve_workspace(n, n); }

size_t lu_solve_workspace(int64_t n, int64_t nrhs, int64_t systems) {
  size_t b = 0;
  b += 2 * ((size_t)lu_named(n) * sizeof(int) + 256);                     // tournament lists
  b += (size_t)kPW * kLeaf * sizeof(double);                              // multipliers of a deciding level
  b += (size_t)kNB * (n + std::max<int64_t>(nrhs, 0)) * sizeof(double) + 256;  // moved block rows (kept form)
  b += (size_t)(cdiv(n, kNB) + 1) * kNB * kNB * sizeof(double) + 512;     // inverse blocks (kept form)
  b += 2 * sizeof(Moves) + 256;                                           // row moves of a block
  b += (size_t)cdiv(n, kNB) * kNB * kNB * sizeof(double) + 256;           // diagonal blocks
  return (size_t)systems * b +
         std::max({gemm_f64_workspace(n, n, kNB), gemm_f64_workspace(n, std::max<int64_t>(nrhs, 1), kNB)}) + 256;
}

void lu_solve_f64(hipStream_t s, int64_t n, double* A, int64_t lda, double* Q, int64_t ldq, int64_t nrhs, Arena& ws,
                  int* info_dev, bool kept, int64_t systems, int64_t sa, int64_t sq) {
  if (n <= 0) return;
  DME_REQUIRE(n < (1ll << 30) && nrhs < (1ll << 30) && systems >= 1 && systems < 65536, DME_EINVAL,
              "LU: dimensions too large");
  const int nq = (int)std::max<int64_t>(nrhs, 0);
  const unsigned nz = (unsigned)systems;
  Systems sys;
  sys.a = sa;
  sys.q = sq;
  sys.blk = cdiv(n, kNB) * kNB * kNB;
  sys.tmp = (int64_t)kNB * (n + nq);
  sys.list = (int)lu_named(n);
  sys.mv = 2;
  sys.lbuf = kPW * kLeaf;
  int* lists[2] = {ws.get<int>((size_t)nz * sys.list), ws.get<int>((size_t)nz * sys.list)};
  Moves* mv = ws.get<Moves>((size_t)nz * sys.mv);
  double* lbuf = ws.get<double>((size_t)nz * sys.lbuf);
  double* blks = ws.get<double>((size_t)nz * sys.blk);
  double* tmp = kept ? ws.get<double>((size_t)nz * sys.tmp) : nullptr;
  double* linv = kept ? ws.get<double>((size_t)nz * kNB * kNB) : nullptr;
  double* uinv = kept ? ws.get<double>((size_t)nz * sys.blk) : nullptr;
  const size_t mark = ws.used;

  // pivots of panel o (its rows start at j0 + o) and the factor of its block
  auto select = [&](int64_t j0, int o, int jb, int jb2, double* blk) {
    const int r0 = (int)j0 + o;
    const int* cand = nullptr;
    int64_t players = n - r0;
    for (int lvl = 0;; ++lvl) {
      const int64_t wg = cdiv(players, kLeaf);
      int* out = lists[lvl & 1];
      // as few rows a lane as keep the level to its number of waves
      auto kern = players <= 64 ? lu_select_kernel<1> : players <= 128 ? lu_select_kernel<2> : lu_select_kernel<3>;
      hipLaunchKernelGGL(kern, dim3((unsigned)wg, nz), dim3(64), 0, s, A, lda, (int)n, r0, r0, jb, cand, (int)players,
                         out, wg == 1 ? 1 : 0, o, jb2, blk, mv + (o ? 1 : 0), lbuf, info_dev, sys);
      DME_HIP(hipGetLastError());
      if (wg == 1) return;
      cand = out;
      players = wg * kPW;
    }
  };
  // C += alpha X Y (or = for beta 0) of every system
  auto product = [&](int64_t M, int64_t N, int64_t K, double alpha, const double* X, int64_t ldx, int64_t sx,
                     const double* Y, int64_t ldy, int64_t sy, double beta, double* C, int64_t ldc, int64_t sc) {
    ws.used = mark;
    gemm_f64_batch(s, systems, M, N, K, alpha, X, ldx, sx, Y, ldy, sy, beta, C, ldc, sc, ws);
  };

  for (int64_t j0 = 0; j0 < n; j0 += kNB) {
    const int jb = (int)std::min<int64_t>(kNB, n - j0);
    const int jb1 = std::min(jb, kPW), jb2 = jb - jb1;
    double* blk = blks + (j0 / kNB) * kNB * kNB;
    select(j0, 0, jb1, jb2, blk);
    const int64_t below1 = n - j0 - jb1;
    if (below1 > 0) {
      hipLaunchKernelGGL((kept ? lu_rows_kernel<0, true> : lu_rows_kernel<0, false>),
                         dim3((unsigned)cdiv(below1, kQuadT / 4), nz), dim3(kQuadT), 0, s, A, lda, (int)n, (int)j0, jb1,
                         jb2, blk, mv, sys);
      DME_HIP(hipGetLastError());
    }
    const int64_t rest = n - j0 - jb;
    if (jb2 > 0) {
      select(j0, kPW, jb2, 0, blk);
      if (rest > 0) {
        hipLaunchKernelGGL((kept ? lu_rows_kernel<kPW, true> : lu_rows_kernel<kPW, false>),
                           dim3((unsigned)cdiv(rest, kQuadT / 4), nz), dim3(kQuadT), 0, s, A, lda, (int)n, (int)j0, jb2, 0,
                           blk, mv + 1, sys);
        DME_HIP(hipGetLastError());
      }
    }
    if (rest + nq > 0) {
      hipLaunchKernelGGL(lu_cols_kernel, dim3((unsigned)cdiv(rest + nq, kQuadT / 4), nz), dim3(kQuadT), 0, s, A, lda,
                         (int)(j0 + jb), (int)rest, Q, ldq, nq, (int)j0, jb, blk, mv, tmp, sys);
      DME_HIP(hipGetLastError());
    }
    double* A12 = A + j0 + (j0 + jb) * lda;
    if (kept && rest + nq > 0) {
      hipLaunchKernelGGL(lu_linv_kernel, dim3(1, nz), dim3(4 * kNB), 0, s, blk, jb, linv, sys);
      DME_HIP(hipGetLastError());
      product(jb, rest, jb, 1.0, linv, jb, kNB * kNB, tmp, jb, sys.tmp, 0.0, A12, lda, sa);
      product(jb, nq, jb, 1.0, linv, jb, kNB * kNB, tmp + (size_t)jb * rest, jb, sys.tmp, 0.0, Q + j0, ldq, sq);
    }
    if (rest > 0) {
      const double* L21 = A + (j0 + jb) + j0 * lda;
      product(rest, rest, jb, -1.0, L21, lda, sa, A12, lda, sa, 1.0, A + (j0 + jb) * (lda + 1), lda, sa);
      product(rest, nq, jb, -1.0, L21, lda, sa, Q + j0, ldq, sq, 1.0, Q + j0 + jb, ldq, sq);
    }
  }
  // backward substitution U X = Y
  if (nq > 0 && kept) {
    hipLaunchKernelGGL(lu_uinv_kernel, dim3((unsigned)cdiv(n, kNB), nz), dim3(kNB), 0, s, blks, (int)n, uinv, sys);
    DME_HIP(hipGetLastError());
  }
  if (nq > 0)
    for (int64_t b = cdiv(n, kNB) - 1; b >= 0; --b) {
      const int64_t j0 = b * kNB;
      const int jb = (int)std::min<int64_t>(kNB, n - j0);
      if (kept) {
        hipLaunchKernelGGL(lu_take_rows_kernel, dim3((unsigned)cdiv(nq, 256 / kNB), nz), dim3(256), 0, s, Q + j0, ldq,
                           nq, jb, tmp, sys);
        DME_HIP(hipGetLastError());
        product(jb, nq, jb, 1.0, uinv + b * kNB * kNB, jb, sys.blk, tmp, jb, sys.tmp, 0.0, Q + j0, ldq, sq);
      } else {
        hipLaunchKernelGGL(lu_back_kernel, dim3((unsigned)cdiv(nq, kQuadT / 4), nz), dim3(kQuadT), 0, s, Q, ldq, nq,
                           (int)j0, jb, blks + b * kNB * kNB, sys);
        DME_HIP(hipGetLastError());
      }
      if (j0 > 0) product(j0, nq, jb, -1.0, A + j0 * lda, lda, sa, Q + j0, ldq, sq, 1.0, Q, ldq, sq);
    }
  ws.used = mark;
}

}  // namespace dme
