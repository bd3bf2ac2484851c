// libbbp: batched truncated singular value decomposition by one-sided
// (Hestenes) Jacobi rotations, FP64.
//
// The compression step of the standard alternative to the zip-up fit (App.
// A: multiply the MPO into the MPS, then compress the result) truncates
// each bond by an SVD; the same primitive gives the singular values of the
// trace distance (App. C).  For a tall matrix A (m >= n) the columns are
// rotated pairwise until every pair is orthogonal: A V = U diag(S) with V
// the product of the rotations, S the column norms and U the normalised
// columns.
//
// One workgroup per matrix.  The matrix is held column-major in LDS (column
// j contiguous, so a pair's dot products are lane-strided reads), V beside
// it.  A sweep is n' - 1 rounds of the round-robin (circle) pairing of the
// n' = n rounded up to even columns: the n'/2 pairs of a round share no
// column, so the 16 waves rotate them side by side, a wave per pair, with
// one barrier per round.  Each pair's three sums (|a_p|^2, |a_q|^2,
// a_p . a_q) are accumulated per lane in row order and reduced across the
// wave in a fixed order (DPP moves within rows of 16 lanes, then the four row
// sums), so every result is reproducible bit for bit and independent of the
// other items of the batch.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "../../include/bbp.h"

namespace bbp {
namespace {

constexpr int kSvdWaves = 16, kSvdThreads = 64 * kSvdWaves;
constexpr int kSvdMaxN = 64;

struct SvdArgs {
  const double *A;
  double *U, *S, *V, *err2;
  int32_t *sweeps;
  int m, n, k, max_sweeps;
  double tol;
};

// v of lane (lane within its row of 16, permuted by the DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over the 64 lanes, the same bits in every lane: within each row of 16
// lanes by DPP moves (partner 1 apart, 2 apart, the other half of 8, the
// other half of 16; each step adds a lane's value to its partner's, so the
// partners hold equal sums), then the four row sums in a fixed order.
__device__ __forceinline__ double wave_total(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

// Columns of round r (0 <= r < np - 1) of the circle pairing of np (even)
// players: pair 0 is (r, np - 1), pair i > 0 is (r + i, r - i) mod np - 1.
__device__ __forceinline__ void round_pair(int r, int i, int np, int *p, int *q) {
  const int h = np - 1;
  int a, b;
  if (i == 0) {
    a = r;
    b = h;
  } else {
    a = (r + i) % h;
    b = (r - i + h) % h;
  }
  *p = min(a, b);
  *q = max(a, b);
}

__global__ __launch_bounds__(kSvdThreads) void k_svd_jacobi(SvdArgs g) {
  extern __shared__ double sm[];
  __shared__ double sig[kSvdMaxN];
  __shared__ int perm[kSvdMaxN], sgn[kSvdMaxN];
  __shared__ int rot[2];
  const int m = g.m, n = g.n, k = g.k, item = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double *a = sm;              // a[j m + i] = A[i][j]
  double *v = sm + (size_t)m * n;  // v[j n + i] = V[i][j]
  const double *Ag = g.A + (size_t)item * m * n;
  for (int t = tid; t < m * n; t += kSvdThreads) {
    const int i = t / n, j = t % n;
    a[(size_t)j * m + i] = Ag[t];
  }
  for (int t = tid; t < n * n; t += kSvdThreads) v[t] = (t / n == t % n) ? 1.0 : 0.0;
  const int np = n + (n & 1);
  int sweep = 0;
  bool clean = false;
  while (sweep < g.max_sweeps) {
    if (tid == 0) rot[sweep & 1] = 0;
    __syncthreads();
    for (int r = 0; r + 1 < np; ++r) {
      for (int pi = wave; pi < np / 2; pi += kSvdWaves) {
        int p, q;
        round_pair(r, pi, np, &p, &q);
        if (q >= n) continue;  // the padding column of an odd n
        double *ap = a + (size_t)p * m, *aq = a + (size_t)q * m;
        double al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll 8
        for (int i = lane; i < m; i += 64) {
          const double x = ap[i], y = aq[i];
          al = fma(x, x, al);
          be = fma(y, y, be);
          ga = fma(x, y, ga);
        }
        al = wave_total(al);
        be = wave_total(be);
        ga = wave_total(ga);
        // rotate unless the pair is already orthogonal to the tolerance
        if (!(fabs(ga) > g.tol * (sqrt(al) * sqrt(be)))) continue;
        const double ze = (be - al) / (2.0 * ga);
        const double t = (ze >= 0.0 ? 1.0 : -1.0) / (fabs(ze) + sqrt(1.0 + ze * ze));
        const double c = 1.0 / sqrt(1.0 + t * t), s = c * t;
#pragma unroll 8
        for (int i = lane; i < m; i += 64) {
          const double x = ap[i], y = aq[i];
          ap[i] = c * x - s * y;
          aq[i] = s * x + c * y;
        }
        double *vp = v + (size_t)p * n, *vq = v + (size_t)q * n;
        for (int i = lane; i < n; i += 64) {
          const double x = vp[i], y = vq[i];
          vp[i] = c * x - s * y;
          vq[i] = s * x + c * y;
        }
        if (lane == 0) atomicOr(&rot[sweep & 1], 1);
      }
      __syncthreads();  // the next round pairs these columns with others
    }
    ++sweep;
    if (rot[(sweep - 1) & 1] == 0) {
      clean = true;
      break;
    }
  }
  // singular values (column norms) and the sign of each column: the
  // largest-magnitude entry (the first of equal ones) made positive
  for (int j = wave; j < n; j += kSvdWaves) {
    const double *aj = a + (size_t)j * m;
    double ss = 0.0, big = -1.0;
    int at = m;
    for (int i = lane; i < m; i += 64) {
      const double x = aj[i];
      ss = fma(x, x, ss);
      if (fabs(x) > big) big = fabs(x), at = i;
    }
    ss = wave_total(ss);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ob = __shfl_xor(big, o, 64);
      const int oa = __shfl_xor(at, o, 64);
      if (ob > big || (ob == big && oa < at)) big = ob, at = oa;
    }
    if (lane == 0) {
      sig[j] = sqrt(ss);
      sgn[j] = (at < m && aj[at] < 0.0) ? -1 : 1;
    }
  }
  __syncthreads();
  // descending order, ties by column index; a NaN norm (non-finite input)
  // sorts last, so the ranks stay a permutation
  if (tid < n) {
    auto key = [](double x) { return x == x ? x : -1.0; };
    const double sj = key(sig[tid]);
    int rk = 0;
    for (int i = 0; i < n; ++i) {
      const double si = key(sig[i]);
      rk += (si > sj) || (si == sj && i < tid);
    }
    perm[rk] = tid;
  }
  __syncthreads();
  double *U = g.U + (size_t)item * m * k, *V = g.V + (size_t)item * n * k;
  for (int t = tid; t < m * k; t += kSvdThreads) {
    const int i = t / k, r = t % k, j = perm[r];
    const double sj = sig[j];
    U[t] = sj > 0.0 ? sgn[j] * (a[(size_t)j * m + i] / sj) : 0.0;
  }
  for (int t = tid; t < n * k; t += kSvdThreads) {
    const int i = t / k, r = t % k, j = perm[r];
    V[t] = sgn[j] * v[(size_t)j * n + i];
  }
  if (tid < k) g.S[(size_t)item * k + tid] = sig[perm[tid]];
  if (tid == 0) {
    if (g.err2) {
      double e = 0.0;
      for (int r = k; r < n; ++r) e = fma(sig[perm[r]], sig[perm[r]], e);
      g.err2[item] = e;
    }
    if (g.sweeps) g.sweeps[item] = clean ? sweep : -sweep;
  }
}

// ---------------------------------------------------------------------------
// The same iteration with the columns in registers (up to 512 rows): one
// workgroup per matrix of ceil(np / 8) waves, each holding the columns of four
// neighbouring pairs (slots i = 4 wave + 0..3: a_i, b_i; lane l holds rows l, l
// + 64, .. and row l of V).  The circle pairing moves every column one slot per
// round - a_i from a_(i+1), b_i from b_(i-1) - so only a wave's outermost two
// columns pass through LDS, with one barrier.  The twelve sums of a wave's
// four pairs are reduced together (each step of the lane reduction halves the
// values a lane carries, slot j ending in the lanes j of every four), and the
// rotations of the four pairs are then computed once, side by side in those
// lanes.
//
// Every sum, comparison and rotation is that of k_svd_jacobi, operation for
// operation, so both give the same bits: the sums are taken in the same row
// order and lane tree, and the products of a rotation are rounded the same way
// (c x - s y as fma(c, x, -(s y)), s x + c y as fma(s, x, c y)).
//
// Bound by the issue and latency of one wave per SIMD: about 1100
// instructions a round, among them a chain of three divisions and three square
// roots.  k_svd_jacobi moves the whole matrix through LDS three times a round,
// computes each pair's rotation in all lanes of a wave and fills a CU's LDS
// with one matrix.  There and here: 48 matrices of 512 x 32 730 and 660 us,
// 700 of 291 x 47 8.92 and 6.46 ms, one of 64 x 16 152 and 132 us.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ double mov_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double swap_rows(double x, bool far) {
  // x plus the x of the row of 16 lanes (or the half of 32) next to it
  const long long b = __double_as_longlong(x);
  const int lo = (int)b, hi = (int)(b >> 32);
  auto join = [](int l, int h) { return __longlong_as_double(((long long)h << 32) | (unsigned)l); };
  if (far) {
    auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return join(l[0], h[0]) + join(l[1], h[1]);
  }
  auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return join(l[0], h[0]) + join(l[1], h[1]);
}
// The totals of four values over the wave by wave_total's tree, that of v[j] in
// every lane with lane % 4 == j.
__device__ __forceinline__ double quad_totals(const double (&v)[4], bool odd, bool high) {
  const double x = (odd ? v[1] : v[0]) + mov_f64<0xB1>(odd ? v[0] : v[1]);
  const double y = (odd ? v[3] : v[2]) + mov_f64<0xB1>(odd ? v[2] : v[3]);
  double t = (high ? y : x) + mov_f64<0x4E>(high ? x : y);
  // the mirrored lane of the other quad, half row: reversing the quad first
  // (quad_perm [3, 2, 1, 0]) meets the same slot
  t += mov_f64<0x141>(mov_f64<0x1B>(t));
  t += mov_f64<0x140>(mov_f64<0x1B>(t));
  return swap_rows(swap_rows(t, false), true);
}

constexpr int kSvdSlots = 4;  // pairs a wave holds

template <int R, int MAXW>
__global__ __launch_bounds__(64 * MAXW) void k_svd_reg(SvdArgs g) {
  extern __shared__ double sm[];  // [parity][wave][down, up][R + 1][64]
  __shared__ double sig[kSvdMaxN];
  __shared__ int perm[kSvdMaxN], rank_of[kSvdMaxN], sgn[kSvdMaxN];
  __shared__ int rot[2][MAXW];
  constexpr int C = R + 1;  // values of a column a lane holds: R of A, one of V
  const int m = g.m, n = g.n, k = g.k, item = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int np = n + (n & 1), h = np - 1, P = np / 2;
  const double *Ag = g.A + (size_t)item * m * n;
  double a[kSvdSlots][C], b[kSvdSlots][C];
  // column of slot i at the start and end of a sweep (np: none)
  auto col_a = [&](int i) { return i < P ? i : np; };
  auto col_b = [&](int i) { return i < P ? (i ? h - i : h) : np; };
  auto load = [&](double (&x)[C], int col) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = lane + 64 * u;
      x[u] = col < n && i < m ? Ag[(size_t)i * n + col] : 0.0;
    }
    x[R] = col < n && lane == col ? 1.0 : 0.0;
  };
#pragma unroll
  for (int j = 0; j < kSvdSlots; ++j) {
    load(a[j], col_a(kSvdSlots * wave + j));
    load(b[j], col_b(kSvdSlots * wave + j));
  }
  const bool odd = lane & 1, high = lane & 2;
  const int slot = kSvdSlots * wave + (lane & 3);  // the pair this lane rotates
  int sweep = 0, par = 0;
  bool clean = false;
  while (sweep < g.max_sweeps) {
    bool any = false;
    for (int r = 0; r < h; ++r) {
      double sa[4], sb[4], sg[4];
#pragma unroll
      for (int j = 0; j < kSvdSlots; ++j) {
        sa[j] = sb[j] = sg[j] = 0.0;
#pragma unroll
        for (int u = 0; u < R; ++u) {
          sa[j] = fma(a[j][u], a[j][u], sa[j]);
          sb[j] = fma(b[j][u], b[j][u], sb[j]);
          sg[j] = fma(a[j][u], b[j][u], sg[j]);
        }
      }
      const double ta = quad_totals(sa, odd, high), tb = quad_totals(sb, odd, high);
      const double ga = quad_totals(sg, odd, high);
      // p is the pair's lower column, q the higher
      auto swapped = [&](int i) {
        const int ca = r + i < h ? r + i : r + i - h, cb = r >= i ? r - i : r - i + h;
        return i > 0 && cb < ca;
      };
      const bool sw = swapped(slot);
      const double al = sw ? tb : ta, be = sw ? ta : tb;
      const bool turn = fabs(ga) > g.tol * (sqrt(al) * sqrt(be));
      const double ze = (be - al) / (2.0 * ga);
      const double t = (ze >= 0.0 ? 1.0 : -1.0) / (fabs(ze) + sqrt(1.0 + ze * ze));
      const double c = 1.0 / sqrt(1.0 + t * t), s = c * t;
      const unsigned turns = (unsigned)__ballot(turn) & 15u;
      any = any || turns != 0;
      auto rotate = [&](auto J) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        if (!(turns >> j & 1)) return;
        const double cj = mov_f64<j * 0x55>(c), sj = mov_f64<j * 0x55>(s);
        if (!swapped(kSvdSlots * wave + j)) {
#pragma unroll
          for (int u = 0; u < C; ++u) {
            const double x = a[j][u], y = b[j][u];
            a[j][u] = fma(cj, x, -(sj * y));
            b[j][u] = fma(sj, x, cj * y);
          }
        } else {
#pragma unroll
          for (int u = 0; u < C; ++u) {
            const double x = b[j][u], y = a[j][u];
            b[j][u] = fma(cj, x, -(sj * y));
            a[j][u] = fma(sj, x, cj * y);
          }
        }
      };
      rotate(std::integral_constant<int, 0>{});
      rotate(std::integral_constant<int, 1>{});
      rotate(std::integral_constant<int, 2>{});
      rotate(std::integral_constant<int, 3>{});
      if (P == 1) continue;  // one pair: nothing moves
      // the next round's columns
      double *buf = sm + (size_t)par * nw * 2 * C * 64;
      if (nw > 1) {
        double *out = buf + (size_t)wave * 2 * C * 64 + lane;
#pragma unroll
        for (int u = 0; u < C; ++u) {
          out[u * 64] = a[0][u];
          out[(C + u) * 64] = b[3][u];
        }
        __syncthreads();
        par ^= 1;
      }
      const double *up = buf + (size_t)min(wave + 1, nw - 1) * 2 * C * 64 + lane;
      const double *dn = buf + ((size_t)max(wave - 1, 0) * 2 + 1) * C * 64 + lane;
      const int last = P - 1 - kSvdSlots * wave;  // the slot whose b becomes its a
      double a0[C];
#pragma unroll
      for (int u = 0; u < C; ++u) a0[u] = a[0][u];
#pragma unroll
      for (int j = 0; j < kSvdSlots; ++j) {
        if (j == last) {
#pragma unroll
          for (int u = 0; u < C; ++u) a[j][u] = b[j][u];
        } else if (j < 3) {
#pragma unroll
          for (int u = 0; u < C; ++u) a[j][u] = a[j < 3 ? j + 1 : 3][u];
        } else {  // slots past the last pair stay zero
#pragma unroll
          for (int u = 0; u < C; ++u) a[j][u] = wave + 1 < nw ? up[u * 64] : 0.0;
        }
      }
#pragma unroll
      for (int j = kSvdSlots - 1; j >= 2; --j)
#pragma unroll
        for (int u = 0; u < C; ++u) b[j][u] = b[j - 1][u];
      if (wave == 0) {
#pragma unroll
        for (int u = 0; u < C; ++u) b[1][u] = a0[u];
      } else {
#pragma unroll
        for (int u = 0; u < C; ++u) {
          b[1][u] = b[0][u];
          b[0][u] = dn[u * 64];
        }
      }
    }
    ++sweep;
    if (nw > 1) {
      if (lane == 0) rot[sweep & 1][wave] = any;
      __syncthreads();
      any = false;
      for (int w = 0; w < nw; ++w) any = any || rot[sweep & 1][w] != 0;
    }
    if (!any) {
      clean = true;
      break;
    }
  }
  // singular values, signs, order: as k_svd_jacobi
  auto finish = [&](const double (&x)[C], int col) __attribute__((always_inline)) {
    if (col >= n) return;
    double ss = 0.0, big = -1.0, at_v = 0.0;
    int at = m;
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = lane + 64 * u;
      ss = fma(x[u], x[u], ss);
      if (i < m && fabs(x[u]) > big) big = fabs(x[u]), at = i, at_v = x[u];
    }
    ss = wave_total(ss);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ob = __shfl_xor(big, o, 64), ov = __shfl_xor(at_v, o, 64);
      const int oa = __shfl_xor(at, o, 64);
      if (ob > big || (ob == big && oa < at)) big = ob, at = oa, at_v = ov;
    }
    if (lane == 0) {
      sig[col] = sqrt(ss);
      sgn[col] = (at < m && at_v < 0.0) ? -1 : 1;
    }
  };
#pragma unroll
  for (int j = 0; j < kSvdSlots; ++j) {
    finish(a[j], col_a(kSvdSlots * wave + j));
    finish(b[j], col_b(kSvdSlots * wave + j));
  }
  __syncthreads();
  for (int c = tid; c < n; c += blockDim.x) {
    auto key = [](double x) { return x == x ? x : -1.0; };
    const double sc = key(sig[c]);
    int rk = 0;
    for (int i = 0; i < n; ++i) {
      const double si = key(sig[i]);
      rk += (si > sc) || (si == sc && i < c);
    }
    perm[rk] = c;
    rank_of[c] = rk;
  }
  __syncthreads();
  double *U = g.U + (size_t)item * m * k, *V = g.V + (size_t)item * n * k;
  auto store = [&](const double (&x)[C], int col) __attribute__((always_inline)) {
    if (col >= n) return;
    const int rk = rank_of[col];
    if (rk >= k) return;
    const double sj = sig[col];
    const int sg = sgn[col];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int i = lane + 64 * u;
      if (i < m) U[(size_t)i * k + rk] = sj > 0.0 ? sg * (x[u] / sj) : 0.0;
    }
    if (lane < n) V[lane * k + rk] = sg * x[R];
  };
#pragma unroll
  for (int j = 0; j < kSvdSlots; ++j) {
    store(a[j], col_a(kSvdSlots * wave + j));
    store(b[j], col_b(kSvdSlots * wave + j));
  }
  if (tid < k) g.S[(size_t)item * k + tid] = sig[perm[tid]];
  for (int i = tid + blockDim.x; i < k; i += blockDim.x) g.S[(size_t)item * k + i] = sig[perm[i]];
  if (tid == 0) {
    if (g.err2) {
      double e = 0.0;
      for (int r = k; r < n; ++r) e = fma(sig[perm[r]], sig[perm[r]], e);
      g.err2[item] = e;
    }
    if (g.sweeps) g.sweeps[item] = clean ? sweep : -sweep;
  }
}

// The register kernel's instance for up to `rows` rows: R the row chunks of 64
// it holds, MAXW the waves the widest matrix of that height needs under
// BBP_SVD_MAX_WORDS; and the columns from which it is the faster one (the two
// give the same bits).  Beyond 512 rows few columns fit, so one to four waves
// do what k_svd_jacobi's sixteen share: 256 matrices of 576 x 31 took 938 us in
// registers against 858, of 1024 x 19 794 against 485.  The same holds for few
// columns below that while a CU has one matrix (`one`, batches up to 256) or
// two, all that k_svd_jacobi's waves leave room for (`two`, up to 512; matrices
// of one wave, 8 columns, are the faster in registers there, `narrow`).  In
// LDS and in registers, us: one 512 x 9 matrix 92 and 137, one 512 x 24 412 and
// 436, 512 x 28 553 and 527; one 256 x 9 101 and 115, 256 x 20 292 and 247; 384
// of 256 x 9 126 and 163, of 256 x 12 216 and 208, of 64 x 8 83 and 73.  In
// larger batches registers win (2048 of 256 x 9 422 and 323) but for the first
// columns of a third wave at 385 to 448 rows, where a chunk is empty, and at 512
// (`many`; 2048 of 512 x 17 1340 and 1610).  At 512 rows k_svd_jacobi's loops
// over rows are whole steps of eight, at 449 to 511 one by one (480 x 14 6 %
// slower than in registers where 512 x 14 is 24 % faster).
using SvdKernel = void (*)(SvdArgs);
struct SvdChoice {
  SvdKernel k;
  int rows, R, maxw;
  int one, two, many;
  bool narrow;
};
const SvdChoice kSvdReg[] = {
    {k_svd_reg<1, 8>, 64, 1, 8, 10, 10, 0, true},
    {k_svd_reg<2, 8>, 128, 2, 8, 10, 10, 0, true},
    {k_svd_reg<3, 8>, 192, 3, 8, 11, 12, 0, true},
    {k_svd_reg<4, 8>, 256, 4, 8, 11, 12, 0, true},
    {k_svd_reg<5, 8>, 320, 5, 8, 18, 12, 0, true},
    {k_svd_reg<6, 7>, 384, 6, 7, 18, 12, 0, true},
    {k_svd_reg<8, 6>, 448, 8, 6, 18, 18, 18, false},
    {k_svd_reg<8, 6>, 511, 8, 6, 10, 10, 0, true},
    {k_svd_reg<8, 6>, 512, 8, 6, 26, 20, 20, false},
};
// The instance that takes the batch, or null: k_svd_jacobi.
const SvdChoice *svd_in_registers(int batch, int m, int n, int waves) {
  for (const SvdChoice &c : kSvdReg) {
    if (m > c.rows) continue;
    const bool ok = batch <= 256   ? n >= c.one
                    : batch <= 512 ? n >= c.two || (c.narrow && n <= 2 * kSvdSlots)
                                   : n <= 4 * kSvdSlots || n >= c.many;
    return ok && waves <= c.maxw ? &c : nullptr;
  }
  return nullptr;
}

}  // namespace
}  // namespace bbp

extern "C" bbp_status bbp_svd_jacobi(int32_t batch, int32_t m, int32_t n, int32_t k,
                                     const double *A, double *U, double *S, double *V,
                                     double *err2, int32_t *sweeps, int32_t max_sweeps,
                                     double tol, void *hip_stream) {
  using namespace bbp;
  if (batch < 0 || n < 1 || n > kSvdMaxN || m < n || k < 1 || k > n || max_sweeps < 1 ||
      max_sweeps > 100 || !(tol >= 0.0 && tol < 1.0) ||
      (size_t)m * n + (size_t)n * n > BBP_SVD_MAX_WORDS)
    return BBP_EINVAL;
  if (batch == 0) return BBP_OK;
  if (!A || !U || !S || !V) return BBP_EINVAL;
  static std::once_flag once;
  static hipError_t attr = hipSuccess;
  std::call_once(once, [] {
    for (const SvdChoice &c : kSvdReg) {
      attr = hipFuncSetAttribute((const void *)c.k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 2 * c.maxw * 2 * (c.R + 1) * 64 * (int)sizeof(double));
      if (attr != hipSuccess) return;
    }
    attr = hipFuncSetAttribute((const void *)k_svd_jacobi,
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(BBP_SVD_MAX_WORDS * sizeof(double)));
  });
  if (attr != hipSuccess) return BBP_EDEVICE;
  SvdArgs g;
  g.A = A;
  g.U = U;
  g.S = S;
  g.V = V;
  g.err2 = err2;
  g.sweeps = sweeps;
  g.m = m;
  g.n = n;
  g.k = k;
  g.max_sweeps = max_sweeps;
  g.tol = tol > 0.0 ? tol : std::sqrt((double)m) * DBL_EPSILON;
  const int waves = ((n + 1) / 2 + kSvdSlots - 1) / kSvdSlots;
  if (const SvdChoice *c = svd_in_registers(batch, m, n, waves)) {
    const size_t xch = waves > 1 ? (size_t)2 * waves * 2 * (c->R + 1) * 64 * sizeof(double) : 0;
    hipLaunchKernelGGL(c->k, dim3(batch), dim3(64 * waves), xch, (hipStream_t)hip_stream, g);
    return hipGetLastError() == hipSuccess ? BBP_OK : BBP_EDEVICE;
  }
  const size_t lds = ((size_t)m * n + (size_t)n * n) * sizeof(double);
  hipLaunchKernelGGL(k_svd_jacobi, dim3(batch), dim3(kSvdThreads), lds,
                     (hipStream_t)hip_stream, g);
  return hipGetLastError() == hipSuccess ? BBP_OK : BBP_EDEVICE;
}
