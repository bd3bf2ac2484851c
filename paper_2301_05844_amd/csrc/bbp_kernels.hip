// HIP kernels of libbbp for gfx950 (MI355X): the split-layer fit visit of
// block BP (App. A of Guo, Poletti, Arad), Householder QR/LQ, and the small
// gather / extract / normalise / overlap steps around it.
//
// Every MPS site lives in a zero-padded slot of S = K*P*K doubles (K the
// bond cap, P = D^2 the fused double-layer leg), so all contractions of a
// batch have the same shape; zero padding stays exactly zero through every
// contraction, and the QR works on the true panel only.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "bbp_internal.h"

namespace bbp {

// ---------------------------------------------------------------------------
// Launch timing
// ---------------------------------------------------------------------------
namespace {
struct TimedLaunch {
  int cls;
  hipEvent_t a, b;
  double flops, bytes, pflops, pbytes;
};
// Launch timing is process-wide; its lists are guarded so contexts used from
// several host threads (the request server) can time concurrently.
struct TimingState {
  std::atomic<bool> on{false};
  std::recursive_mutex mu;
  std::vector<TimedLaunch> done;
  std::vector<hipEvent_t> pool;
  long long launches[KC_COUNT] = {};
  double ms[KC_COUNT] = {}, flops[KC_COUNT] = {}, bytes[KC_COUNT] = {};
  double pflops[KC_COUNT] = {}, pbytes[KC_COUNT] = {};
};
TimingState &timing() {
  static TimingState t;
  return t;
}
hipEvent_t take_event() {
  TimingState &t = timing();
  std::lock_guard<std::recursive_mutex> lk(t.mu);
  if (!t.pool.empty()) {
    hipEvent_t e = t.pool.back();
    t.pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}
// Folds completed event pairs into the per-class totals.
hipError_t drain() {
  TimingState &t = timing();
  std::lock_guard<std::recursive_mutex> lk(t.mu);
  for (TimedLaunch &l : t.done) {
    hipError_t e = hipEventSynchronize(l.b);
    if (e != hipSuccess) return e;
    float ms = 0.f;
    e = hipEventElapsedTime(&ms, l.a, l.b);
    if (e != hipSuccess) return e;
    t.launches[l.cls] += 1;
    t.ms[l.cls] += ms;
    t.flops[l.cls] += l.flops;
    t.bytes[l.cls] += l.bytes;
    t.pflops[l.cls] += l.pflops;
    t.pbytes[l.cls] += l.pbytes;
    t.pool.push_back(l.a);
    t.pool.push_back(l.b);
  }
  t.done.clear();
  return hipSuccess;
}
// Brackets one launch with events when timing is on.  f, b: algorithmic
// counts on the true extents; pf, pb: padded counts and the kernel's own
// byte traffic (the same as f, b where a launch has no padding).
struct Span {
  int cls;
  hipStream_t st;
  double flops, bytes, pflops, pbytes;
  hipEvent_t a = nullptr;
  Span(int c, hipStream_t s, double f, double b, double pf = -1.0, double pb = -1.0)
      : cls(c), st(s), flops(f), bytes(b), pflops(pf < 0 ? f : pf), pbytes(pb < 0 ? b : pb) {
    if (!timing().on) return;
    std::lock_guard<std::recursive_mutex> lk(timing().mu);
    if (timing().done.size() > 4096) (void)drain();
    a = take_event();
    if (a && hipEventRecord(a, st) != hipSuccess) a = nullptr;
  }
  ~Span() {
    if (!a) return;
    std::lock_guard<std::recursive_mutex> lk(timing().mu);
    hipEvent_t b = take_event();
    if (b && hipEventRecord(b, st) == hipSuccess)
      timing().done.push_back(TimedLaunch{cls, a, b, flops, bytes, pflops, pbytes});
  }
};
const char *kClassNames[KC_COUNT] = {"fit_visit", "fit_T1",  "fit_ket",
                                     "fit_bra",   "fit_local", "fit_env",
                                     "fit_end",   "qr",       "other"};
}  // namespace

void timing_enable(bool on) { timing().on = on; }
bool timing_enabled() { return timing().on; }
void timing_reset() {
  TimingState &t = timing();
  std::lock_guard<std::recursive_mutex> lk(t.mu);
  (void)drain();
  for (int i = 0; i < KC_COUNT; ++i) {
    t.launches[i] = 0;
    t.ms[i] = t.flops[i] = t.bytes[i] = t.pflops[i] = t.pbytes[i] = 0.0;
  }
}
hipError_t timing_query(int cls, const char **name, long long *launches,
                        double *ms, double *flops, double *bytes, double *pflops,
                        double *pbytes) {
  TimingState &t = timing();
  std::lock_guard<std::recursive_mutex> lk(t.mu);
  hipError_t e = drain();
  if (e != hipSuccess) return e;
  if (name) *name = kClassNames[cls];
  if (launches) *launches = t.launches[cls];
  if (ms) *ms = t.ms[cls];
  if (flops) *flops = t.flops[cls];
  if (bytes) *bytes = t.bytes[cls];
  if (pflops) *pflops = t.pflops[cls];
  if (pbytes) *pbytes = t.pbytes[cls];
  return hipSuccess;
}

namespace {

constexpr int kThreads = 256;

// ---------------------------------------------------------------------------
// Batched FP64 GEMM engine.  C(it, m, n) = sum_k A(it, m, k) B(it, k, n) for
// the items of a batch (blockIdx.z).  The operand and result index maps are
// supplied by an op struct (a(), b(), st()); each workgroup stages BK-deep
// slices of A and B in LDS and 16 x 16 threads accumulate TM x TN tiles.
// ---------------------------------------------------------------------------
typedef double v4d __attribute__((ext_vector_type(4)));

// LDS row strides that keep the MFMA operand reads free of bank conflicts
// (64-bit words, 32 word pairs per bank row; a read serves 16 lanes along the
// tile and 2 lane groups along k together): a row that the 16 lanes walk as
// the A operand gets a stride of 2 (mod 32), a row that 2 lane groups walk as
// the B operand a stride of 16 (mod 32).
__host__ __device__ constexpr int pad_a(int x) { return x + (34 - x % 32) % 32; }
__host__ __device__ constexpr int pad_b(int x) { return x + (48 - x % 32) % 32; }

__device__ __forceinline__ v4d mfma16(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Device global memory seen through a pointer whose origin the compiler
// cannot trace (taken from a pointer table or a struct member): accesses
// through the returned pointer are global loads and stores, not flat ones,
// which would also count against the LDS wait counter.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gmem(T *p) {
  return (__attribute__((address_space(1))) T *)p;
}

// Loads and stores through a buffer descriptor: the base lives in SGPRs and
// each lane supplies a 32-bit byte offset, so a loop keeps one 32-bit offset
// per element instead of a 64-bit address.  Descriptor word 3 selects the
// 32-bit data format, which untyped buffer accesses on this GPU family
// require.  The hardware checks every offset against the `bytes` declared: a
// load at or beyond it returns zero and a store there is dropped; the visit
// and the environment update load the elements outside their operands that
// way (offset `bytes`).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const double *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const float *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ double buf_ld(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, 0));
}
template <class T>
__device__ __forceinline__ void buf_st_t(__amdgpu_buffer_rsrc_t r, unsigned byte_off, T v);
template <>
__device__ __forceinline__ void buf_st_t<double>(__amdgpu_buffer_rsrc_t r, unsigned o, double v) {
  typedef unsigned int v2u __attribute__((__vector_size__(8)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), r, o, 0, 0);
}
template <>
__device__ __forceinline__ void buf_st_t<float>(__amdgpu_buffer_rsrc_t r, unsigned o, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, o, 0, 0);
}
template <class T> __device__ __forceinline__ T buf_ld_t(__amdgpu_buffer_rsrc_t r, unsigned byte_off);
template <> __device__ __forceinline__ double buf_ld_t<double>(__amdgpu_buffer_rsrc_t r, unsigned o) {
  return buf_ld(r, o);
}
template <> __device__ __forceinline__ float buf_ld_t<float>(__amdgpu_buffer_rsrc_t r, unsigned o) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
}

// Workgroups are dealt to the 8 XCDs round-robin by linear id, and each XCD
// has its own L2.  For a (tile, item) grid this returns the tile and item of
// the calling workgroup such that every tile of item i < 8 floor(items / 8)
// runs on XCD i % 8 (an item's shared operands stay in one L2); the items
// beyond follow in plain order.
__device__ __forceinline__ void xcd_tile_item(int *tile, int *item) {
  constexpr int kXcds = 8;
  const int nx = gridDim.x, ny = gridDim.y, ny8 = ny - ny % kXcds;
  const int w = blockIdx.x + nx * blockIdx.y;
  if (w >= nx * ny8) {
    *item = ny8 + (w - nx * ny8) / nx;
    *tile = (w - nx * ny8) % nx;
    return;
  }
  const int xcd = w % kXcds, slot = w / kXcds;
  *item = (slot / nx) * kXcds + xcd;
  *tile = slot % nx;
}

// x of lane Q of the same four lanes
template <int Q>
__device__ __forceinline__ double quad_bcast(double x) {
  constexpr int ctrl = Q | (Q << 2) | (Q << 4) | (Q << 6);  // quad_perm
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), ctrl, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// f(integral_constant<int, I>) for I = I0 .. N-1, unrolled at compile time.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Orders one wave's LDS writes before its later LDS reads (other lanes).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Contraction type of the specialised kernels: FP64, or FP32 on FP32 MFMA
// with FP32 accumulation (the precision option).  LDS stride residues for
// 4-byte words: A-operand rows 4 (mod 64), B-operand rows 16 (mod 64).
typedef float v4f __attribute__((ext_vector_type(4)));
template <class T> struct Mma;
// crow(r, lq): tile row held by accumulator register r of a lane in row
// group lq (FP64 MFMA: 4r + lq; FP32 16x16x4 MFMA: 4lq + r, as probed).
template <> struct Mma<double> {
  typedef v4d acc;
  static __device__ __forceinline__ int crow(int r, int lq) { return 4 * r + lq; }
  static __device__ __forceinline__ v4d run(double a, double b, v4d c) { return mfma16(a, b, c); }
  static __host__ __device__ constexpr int pad_a(int x) { return bbp::pad_a(x); }
  static __host__ __device__ constexpr int pad_b(int x) { return bbp::pad_b(x); }
  // smallest A-operand row stride >= x whose 16 rows x 2 lane groups of a
  // half wave fall in distinct banks: any stride = 2 (mod 4)
  static __host__ __device__ constexpr int pad_a_min(int x) { return x + (6 - x % 4) % 4; }
};
template <> struct Mma<float> {
  typedef v4f acc;
  static __device__ __forceinline__ int crow(int r, int lq) { return 4 * lq + r; }
  static __device__ __forceinline__ v4f run(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __host__ __device__ constexpr int pad_a(int x) { return x + (68 - x % 64) % 64; }
  static __host__ __device__ constexpr int pad_b(int x) { return x + (80 - x % 64) % 64; }
  static __host__ __device__ constexpr int pad_a_min(int x) { return x + (12 - x % 8) % 8; }
};

// BF16 contraction step (the precision option's lowest stage): FP32 operands
// rounded to BF16 (nearest even), BF16 MFMA 16x16x16 with FP32 accumulation.
// Each lane supplies four k values of its A row and B column; the product
// sums over the 16 (lane group, slot) pairs, so any assignment of k values
// to slots is valid as long as A and B use the same one.  The accumulator
// layout is that of the FP32 MFMA (Mma<float>::crow).
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4f mfma_bf16(const float *a, const float *b, v4f c) {
  v4bf x, y;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[j] = (__bf16)a[j];
    y[j] = (__bf16)b[j];
  }
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, x),
                                                   __builtin_bit_cast(v4s, y), c, 0, 0, 0);
}

template <int BM, int BN, int BK, class Op>
__global__ __launch_bounds__(kThreads) void k_gemm(Op op) {
  const int it = blockIdx.z;
  if (op.flag && !op.flag[it]) return;
  // 16 x 16 MFMA tiles of the BM x BN block, spread over the four waves
  constexpr int TMX = BM / 16, TNX = BN / 16, NT = TMX * TNX;
  constexpr int TPW = (NT + 3) / 4;
  __shared__ double As[BK][BM + 1];
  __shared__ double Bs[BK][BN + 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  v4d acc[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) acc[q] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < op.Kd; k0 += BK) {
    for (int i = tid; i < BM * BK; i += kThreads) {
      const int kk = i % BK, mm = i / BK;
      const int m = m0 + mm, k = k0 + kk;
      As[kk][mm] = (m < op.M && k < op.Kd) ? op.a(it, m, k) : 0.0;
    }
    for (int i = tid; i < BK * BN; i += kThreads) {
      const int nn = i % BN, kk = i / BN;
      const int n = n0 + nn, k = k0 + kk;
      Bs[kk][nn] = (n < op.N && k < op.Kd) ? op.b(it, k, n) : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      const int t = wave + 4 * q;
      if (t < NT) {
        const int tm = (t / TNX) * 16, tn = (t % TNX) * 16;
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
              As[kk + lq][tm + lr], Bs[kk + lq][tn + lr], acc[q], 0, 0, 0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int t = wave + 4 * q;
    if (t < NT) {
      const int tm = (t / TNX) * 16, tn = (t % TNX) * 16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + tm + 4 * r + lq, n = n0 + tn + lr;
        if (m < op.M && n < op.N) op.st(it, m, n, acc[q][r]);
      }
    }
  }
}

template <int BM, int BN, int BK, class Op>
hipError_t run_gemm(const Op &op, int items, hipStream_t st) {
  if (items <= 0 || op.M <= 0 || op.N <= 0) return hipSuccess;
  dim3 grid((op.N + BN - 1) / BN, (op.M + BM - 1) / BM, items);
  hipLaunchKernelGGL((k_gemm<BM, BN, BK, Op>), grid, dim3(kThreads), 0, st,
                     op);
  return hipGetLastError();
}

// Split-K form for a few output tiles per item and a long reduction (the
// end-site local update: one 32 x 32 tile from K P = 512 terms at chi = 32,
// which one workgroup per item walks in eight dependent chunks): NS
// workgroups per tile each reduce one contiguous k range into a partial
// tile of `part` ([item][NS][M][N]), and k_splitk_sum adds the NS partials
// of every element in a fixed order (k range 0 first) and stores the sum
// through the op.
template <int BM, int BN, int BK, int NS, class Op>
__global__ __launch_bounds__(kThreads) void k_gemm_part(Op op, double *part,
                                                        size_t part_stride) {
  const int it = blockIdx.z;
  if (op.flag && !op.flag[it]) return;
  constexpr int TMX = BM / 16, TNX = BN / 16, NT = TMX * TNX;
  constexpr int TPW = (NT + 3) / 4;
  __shared__ double As[BK][BM + 1];
  __shared__ double Bs[BK][BN + 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int ks = blockIdx.x % NS;
  const int m0 = blockIdx.y * BM, n0 = (blockIdx.x / NS) * BN;
  const int span = ((op.Kd + NS - 1) / NS + BK - 1) / BK * BK;
  const int kb = ks * span, ke = min(op.Kd, kb + span);
  v4d acc[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) acc[q] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int k0 = kb; k0 < ke; k0 += BK) {
    for (int i = tid; i < BM * BK; i += kThreads) {
      const int kk = i % BK, mm = i / BK;
      const int m = m0 + mm, k = k0 + kk;
      As[kk][mm] = (m < op.M && k < ke) ? op.a(it, m, k) : 0.0;
    }
    for (int i = tid; i < BK * BN; i += kThreads) {
      const int nn = i % BN, kk = i / BN;
      const int n = n0 + nn, k = k0 + kk;
      Bs[kk][nn] = (n < op.N && k < ke) ? op.b(it, k, n) : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      const int t = wave + 4 * q;
      if (t < NT) {
        const int tm = (t / TNX) * 16, tn = (t % TNX) * 16;
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4)
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(
              As[kk + lq][tm + lr], Bs[kk + lq][tn + lr], acc[q], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  double *pp = part + (size_t)it * part_stride + (size_t)ks * op.M * op.N;
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int t = wave + 4 * q;
    if (t < NT) {
      const int tm = (t / TNX) * 16, tn = (t % TNX) * 16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + tm + 4 * r + lq, n = n0 + tn + lr;
        if (m < op.M && n < op.N) pp[(size_t)m * op.N + n] = acc[q][r];
      }
    }
  }
}

template <int NS, class Op>
__global__ __launch_bounds__(kThreads) void k_splitk_sum(Op op, const double *part,
                                                         size_t part_stride) {
  const int it = blockIdx.y;
  if (op.flag && !op.flag[it]) return;
  const size_t mn = (size_t)op.M * op.N;
  const double *pp = part + (size_t)it * part_stride;
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < mn;
       i += (size_t)gridDim.x * kThreads) {
    double v = pp[i];
#pragma unroll
    for (int ks = 1; ks < NS; ++ks) v += pp[(size_t)ks * mn + i];
    op.st(it, (int)(i / op.N), (int)(i % op.N), v);
  }
}

// Split-K GEMM of `items` items: part holds NS M N doubles per item (stride
// part_stride).
template <int BM, int BN, int BK, int NS, class Op>
hipError_t run_gemm_splitk(const Op &op, int items, double *part, size_t part_stride,
                           hipStream_t st) {
  if (items <= 0 || op.M <= 0 || op.N <= 0) return hipSuccess;
  if (part_stride < (size_t)NS * op.M * op.N) return hipErrorInvalidValue;
  dim3 grid(NS * ((op.N + BN - 1) / BN), (op.M + BM - 1) / BM, items);
  hipLaunchKernelGGL((k_gemm_part<BM, BN, BK, NS, Op>), grid, dim3(kThreads), 0, st, op,
                     part, part_stride);
  const int blocks = (int)std::min<size_t>(8, ((size_t)op.M * op.N + kThreads - 1) / kThreads);
  hipLaunchKernelGGL((k_splitk_sum<NS, Op>), dim3(blocks, items), dim3(kThreads), 0, st, op,
                     (const double *)part, part_stride);
  return hipGetLastError();
}

// Site tensor A'[s][u][l][d][r] of the rotated block, flat index.
__device__ __forceinline__ size_t aidx(int D, int s, int u, int l, int dd,
                                       int r) {
  return ((((size_t)s * D + u) * D + l) * D + dd) * D + r;
}

struct Shape {
  int K, P, D, d;
};

// ---- inner-site visit ---------------------------------------------------
// Front view: "front" is the side the sweep comes from (left for LR, right
// for RL).  X_f[xf][a][xb], A_f[s][wf][l][wb][a] with wf the MPO leg on the
// front side, F the front environment, G the back environment.

// T1[yf][wfb][ab][xb][wfk][ak] = sum_xf F[yf][wf][xf] X_f[xf][a][xb]
struct OpK1 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  Ptr X, F;
  double *t1;
  size_t t1s;
  __device__ double a(int it, int m, int k) const {
    return F.at(it)[(size_t)m * s.K + k];
  }
  __device__ double b(int it, int k, int n) const {
    const int a = n / s.K, xb = n - a * s.K;
    const double *x = X.at(it);
    return rl ? x[((size_t)xb * s.P + a) * s.K + k]
              : x[((size_t)k * s.P + a) * s.K + xb];
  }
  __device__ void st(int it, int m, int n, double v) const {
    const int D = s.D, K = s.K, P = s.P;
    const int yf = m / P, wf = m - yf * P, wfk = wf / D, wfb = wf - wfk * D;
    const int a = n / K, xb = n - a * K, ak = a / D, ab = a - ak * D;
    const size_t idx =
        (((((size_t)yf * D + wfb) * D + ab) * K + xb) * D + wfk) * D + ak;
    t1[(size_t)it * t1s + idx] = v;
  }
};

// T2[yf][xb][lk][wbk][s][wfb][ab] = sum_{wfk,ak} T1[...][wfk][ak] Aket_f[s][wfk][lk][wbk][ak]
struct OpK2 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  const double *t1;
  size_t t1s;
  const double *A;  // item 0, site (j-1, c)
  size_t as;
  double *t2;
  size_t t2s;
  __device__ double a(int it, int m, int k) const {
    return t1[(size_t)it * t1s + (size_t)m * s.P + k];
  }
  __device__ double b(int it, int k, int n) const {
    const int D = s.D;
    const int wfk = k / D, ak = k - wfk * D;
    const int sp = n / s.P, r = n - sp * s.P, lk = r / D, wbk = r - lk * D;
    const double *A0 = A + (size_t)it * as;
    return rl ? A0[aidx(D, sp, wbk, lk, wfk, ak)]
              : A0[aidx(D, sp, wfk, lk, wbk, ak)];
  }
  __device__ void st(int it, int m, int n, double v) const {
    const int D = s.D, K = s.K;
    int t = m;
    const int xb = t % K;
    t /= K;
    const int ab = t % D;
    t /= D;
    const int wfb = t % D;
    const int yf = t / D;
    const int sp = n / s.P, r = n - sp * s.P, lk = r / D, wbk = r - lk * D;
    const size_t idx =
        (((((((size_t)yf * K + xb) * D + lk) * D + wbk) * s.d + sp) * D + wfb) *
             D +
         ab);
    t2[(size_t)it * t2s + idx] = v;
  }
};

// T3[yf][lk][lb][xb][wbk][wbb] = sum_{s,wfb,ab} T2[...] Abra_f[s][wfb][lb][wbb][ab]
struct OpK3 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  const double *t2;
  size_t t2s;
  const double *A;
  size_t as;
  double *t3;
  size_t t3s;
  __device__ double a(int it, int m, int k) const {
    return t2[(size_t)it * t2s + (size_t)m * Kd + k];
  }
  __device__ double b(int it, int k, int n) const {
    const int D = s.D;
    const int sp = k / s.P, r = k - sp * s.P, wfb = r / D, ab = r - wfb * D;
    const int lb = n / D, wbb = n - lb * D;
    const double *A0 = A + (size_t)it * as;
    return rl ? A0[aidx(D, sp, wbb, lb, wfb, ab)]
              : A0[aidx(D, sp, wfb, lb, wbb, ab)];
  }
  __device__ void st(int it, int m, int n, double v) const {
    const int D = s.D, K = s.K, P = s.P;
    int t = m;
    const int wbk = t % D;
    t /= D;
    const int lk = t % D;
    t /= D;
    const int xb = t % K;
    const int yf = t / K;
    const int lb = n / D, wbb = n - lb * D;
    const size_t idx =
        (((size_t)yf * P + lk * D + lb) * K + xb) * P + wbk * D + wbb;
    t3[(size_t)it * t3s + idx] = v;
  }
};

// Yt[yf][l][yb] = sum_{xb,wb} T3[yf][l][xb][wb] G[yb][wb][xb]
struct OpK4 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  const double *t3;
  size_t t3s;
  Ptr G, Y;
  __device__ double a(int it, int m, int k) const {
    return t3[(size_t)it * t3s + (size_t)m * Kd + k];
  }
  __device__ double b(int it, int k, int n) const {
    const int xb = k / s.P, wb = k - xb * s.P;
    return G.at(it)[((size_t)n * s.P + wb) * s.K + xb];
  }
  __device__ void st(int it, int m, int n, double v) const {
    const int yf = m / s.P, l = m - yf * s.P;
    const size_t idx = rl ? ((size_t)n * s.P + l) * s.K + yf
                          : ((size_t)yf * s.P + l) * s.K + n;
    Y.at(it)[idx] = v;
  }
};

// env'[yb][wb][xb] = sum_{yf,l} Y[yf][l][yb] T3[yf][l][xb][wb]
struct OpK5 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  const double *t3;
  size_t t3s;
  Ptr Y, E;
  __device__ double a(int it, int m, int k) const {
    const int yf = k / s.P, l = k - yf * s.P;
    const size_t idx = rl ? ((size_t)m * s.P + l) * s.K + yf
                          : ((size_t)yf * s.P + l) * s.K + m;
    return Y.at(it)[idx];
  }
  __device__ double b(int it, int k, int n) const {
    return t3[(size_t)it * t3s + (size_t)k * N + n];
  }
  __device__ void st(int it, int m, int n, double v) const {
    const int xb = n / s.P, wb = n - xb * s.P;
    E.at(it)[((size_t)m * s.P + wb) * s.K + xb] = v;
  }
};

// ---- environment update after the QR, Lenv' = T3 . Y ----------------------
// E[y'][wb][xb] = sum_{yf, l} Y[yf][l][y'] T3[yf][l][xb][wb]  (RL: Y[y'][l][yf]).
// One workgroup per (item, 16 CG columns n = (xb, wb)) of CG KS waves: wave w
// owns the 16 columns w % CG and all MT row tiles of y', over the k part w / CG
// of every chunk.  The T3 operand is read straight from global memory (16 lanes,
// 128 contiguous bytes); Y is staged in LDS in chunks of 32 KS k = (yf, l).
// The next chunk of both is fetched into registers while the current one is
// multiplied; one barrier per chunk.  The KS partial sums of a column tile are
// added at the end in a fixed order (k part 0, 1, ...).
struct EnvArgs {
  int K, P, rl;
  const double *t3;
  size_t t3s;
  Ptr Y, E;
  // true extents of site j of column c (null: the full bond cap K): the k
  // range stops at the true front bond of Y and the T3 columns past the
  // true X bond are not read (the pair-per-wave visit does not write them)
  const FitDims *dims;
  int W, c, j, N;
};

// CG column groups of 16 and KS k parts per workgroup, a wave each.  Batches
// that fill the CUs: four groups and, up to 32 rows (MT <= 2), two k parts;
// from MT = 3 one, which leaves the registers for T3 two chunks ahead at MT =
// 3.  Small batches (FILL = false), where each chunk waits for a round trip to
// memory (2 us: T3 and Y come from other XCDs): half the columns, and twice (MT
// = 2) or four times the k range a chunk, as much as LDS holds at MT = 4.  One
// item of 32 rows 17.8 -> 13.4 us, four of 48 40.4 -> 26.7, one of 64 rows and
// 2304 columns 144 -> 88; of 16 rows it was slower (6.0 and 6.4 us).
template <int MT, bool FILL = true> struct EnvShape {
  static constexpr int CG = FILL ? 4 : 2;
  static constexpr int KS = FILL ? (MT <= 2 ? 2 : 1) : 4;
  static constexpr int kThreads = 64 * CG * KS;
  static constexpr int kWaves = MT <= 2 && FILL ? 4 : 2;  // waves per SIMD the registers allow
};

// B16 (T = float): BF16 MFMA, the eight T3 rows a lane holds per chunk
// feeding two 16-deep steps (rows 4i + lq, i = 0-3 and 4-7).
template <int MT, class T, bool B16 = false, bool FILL = true>
__global__ __launch_bounds__((EnvShape<MT, FILL>::kThreads))
__attribute__((amdgpu_waves_per_eu((EnvShape<MT, FILL>::kWaves)))) void k_env(EnvArgs e) {
  typedef EnvShape<MT, FILL> S;
  typedef Mma<T> M;
  typedef typename M::acc Acc;
  constexpr int KS = S::KS, CG = S::CG, NT = S::kThreads;
  constexpr int MW = MT * 16, AS = M::pad_b(MW), CH = 32 * KS;
  constexpr int NA = CH * MW / NT;  // A elements staged per thread
  __shared__ T As[2][CH][AS];
  const int K = e.K, P = e.P, N = K * P;
  int tile, it;
  xcd_tile_item(&tile, &it);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4, cg = wave % CG, h = wave / CG;
  const int n = (tile * CG + cg) * 16 + lr;
  // k = (yf, l) runs to the true front bond of Y, columns n = (xb, wb) to the
  // true X bond; past them every product is zero (Y padding) or T3 was not
  // written, so they are skipped (or masked) without changing any sum.  E is
  // still written in full (zeros in the padding).
  int Kd = K * P, Nt = N;
  if (e.dims) {
    const SiteExt ex = site_ext(e.dims[(size_t)it * e.W + e.c], e.j, e.N, e.rl != 0);
    Kd = ex.yf * P;
    Nt = ex.xb * P;
  }
  if (tile * 16 * CG >= Nt) {  // every column of the tile is padding
    auto *Ez = gmem(e.E.at(it));
    const int nz = tile * 16 * CG + tid % (16 * CG);
    if (nz < N) {
      const int xb = nz / P, wb = nz - xb * P;
      for (int m = tid / (16 * CG); m < K; m += NT / (16 * CG))
        Ez[((size_t)m * P + wb) * K + xb] = 0.0;
    }
    return;
  }
  // Y (K P K doubles) and this item's T3 (K P x K P) through buffer
  // descriptors; an element outside the operand (or past the true extents)
  // loads at the descriptor's end, where the range check returns zero
  const T *T3 = reinterpret_cast<const T *>(e.t3) + (size_t)it * e.t3s;
  const unsigned ybytes = (unsigned)(K * P * K) * 8u;
  const unsigned tbytes = (unsigned)(Kd * N) * (unsigned)sizeof(T);
  const __amdgpu_buffer_rsrc_t yrs = buf_rsrc(e.Y.at(it), ybytes);
  const __amdgpu_buffer_rsrc_t trs = buf_rsrc(T3, tbytes);
  const bool rl = e.rl != 0;
  // Y elements of the next chunk (raw loads, staged in LDS by put)
  double an[NA];
  // RL layout: (yf, l) of k = k0 + kk for each staged element, packed as
  // yf * 256 + l and carried from chunk to chunk (no division in the loop)
  int yfl[NA];
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int kk = (tid + u * NT) / MW;
    yfl[u] = (kk / P) * 256 + kk % P;
  }
  const int dyfl = (CH / P) * 256 + CH % P;
  auto fetch_a = [&](int k0) {  // chunks in order 0, CH, 2 CH, ...
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int i = tid + u * NT, kk = i / MW, m = i % MW, k = k0 + kk;
      const bool ok = m < K && k < Kd;
      const unsigned off = rl ? (m * P + (yfl[u] & 255)) * K + (yfl[u] >> 8) : k * K + m;
      an[u] = buf_ld(yrs, ok ? off * 8u : ybytes);
      yfl[u] += dyfl;
      if ((yfl[u] & 255) >= P) yfl[u] += 256 - P;
    }
  };
  // T3 rows of chunk k0 for this wave's k part (two chunks are in flight)
  auto fetch_b = [&](int k0, T (&b)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = k0 + h * 32 + 4 * i + lq;
      const bool ok = n < Nt && k < Kd;
      b[i] = buf_ld_t<T>(trs, ok ? (unsigned)(k * N + n) * (unsigned)sizeof(T) : tbytes);
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int i = tid + u * NT;
      As[buf][i / MW][i % MW] = (T)an[u];
    }
  };
  // two accumulation chains per row tile, one where MT tiles already give
  // three or more independent chains
  constexpr int NC = MT >= 3 ? 1 : 2;
  Acc acc[MT][NC];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[mt][q] = Acc{0, 0, 0, 0};
  // T3 rows are fetched DB chunks ahead (two while the registers allow)
  constexpr int DB = MT <= 3 ? 2 : 1;
  T b0[8], b1[8];
  fetch_a(0);
  fetch_b(0, b0);
  if (DB == 2 && CH < Kd) fetch_b(CH, b1);
  put(0);
  __syncthreads();
  int buf = 0;
  // one chunk: multiply with the staged Y and the given T3 rows, then
  // refill those rows DB chunks ahead and stage the next Y chunk
  auto step = [&](int k0, T (&b)[8]) {
    if (k0 + CH < Kd) fetch_a(k0 + CH);
    if constexpr (B16) {  // copy out, refill, then two BF16 steps per row tile
      float bc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) bc[i] = (float)b[i];
      if (k0 + DB * CH < Kd) fetch_b(k0 + DB * CH, b);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        float a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = As[buf][h * 32 + 4 * i + lq][mt * 16 + lr];
        acc[mt][0] = mfma_bf16(a, bc, acc[mt][0]);
        acc[mt][NC - 1] = mfma_bf16(a + 4, bc + 4, acc[mt][NC - 1]);
      }
    } else if constexpr (DB == 1) {  // copy out, then refill the same registers
      T bc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) bc[i] = b[i];
      if (k0 + CH < Kd) fetch_b(k0 + CH, b);
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][i % NC] =
              M::run(As[buf][h * 32 + 4 * i + lq][mt * 16 + lr], bc[i], acc[mt][i % NC]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const T bc = b[i];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][i % NC] =
              M::run(As[buf][h * 32 + 4 * i + lq][mt * 16 + lr], bc, acc[mt][i % NC]);
      }
      if (k0 + 2 * CH < Kd) fetch_b(k0 + 2 * CH, b);
    }
    if (k0 + CH < Kd) put(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  };
  for (int k0 = 0; k0 < Kd; k0 += DB * CH) {
    step(k0, b0);
    if (DB == 2 && k0 + CH < Kd) step(k0 + CH, b1);
  }
  Acc c[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) c[mt] = NC == 1 ? acc[mt][0] : acc[mt][0] + acc[mt][NC - 1];
  if (KS > 1) {  // k parts 1.. hand their sums to part 0 through LDS
    T *red = &As[0][0][0];
    static_assert((KS - 1) * CG * MT * 4 * 64 <= 2 * CH * AS, "reduction fits");
    if (h > 0) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[((((h - 1) * CG + cg) * MT + mt) * 4 + r) * 64 + lane] = c[mt][r];
    }
    __syncthreads();
    if (h > 0) return;
#pragma unroll
    for (int hh = 1; hh < KS; ++hh)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          c[mt][r] += red[((((hh - 1) * CG + cg) * MT + mt) * 4 + r) * 64 + lane];
  }
  if (n >= N) return;
  const int xb = n / P, wb = n - xb * P;
  auto *E = gmem(e.E.at(it));
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mt * 16 + M::crow(r, lq);
      if (m < K) E[((size_t)m * P + wb) * K + xb] = (double)c[mt][r];
    }
  }
}

// ---- end-site visit (message site as MPO: Mend[a][q][a']) ----------------
// T[a][q][xb] = sum_{a'} Mend[a][q][a'] X_e[a'][xb]
struct OpE1 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  Ptr Mend, Xe;
  double *t3;
  size_t t3s;
  __device__ double a(int it, int m, int k) const {
    return Mend.at(it)[(size_t)m * s.K + k];
  }
  __device__ double b(int it, int k, int n) const {
    return rl ? Xe.at(it)[(size_t)n * s.K + k] : Xe.at(it)[(size_t)k * s.K + n];
  }
  __device__ void st(int it, int m, int n, double v) const {
    t3[(size_t)it * t3s + (size_t)m * s.K + n] = v;
  }
};

// Yt_e[a][yb] = sum_{q,xb} T[a][q][xb] G[yb][q][xb]
struct OpE2 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  const double *t3;
  size_t t3s;
  Ptr G, Ye;
  __device__ double a(int it, int m, int k) const {
    return t3[(size_t)it * t3s + (size_t)m * Kd + k];
  }
  __device__ double b(int it, int k, int n) const {
    return gmem((const double *)G.at(it))[(size_t)n * Kd + k];
  }
  __device__ void st(int it, int m, int n, double v) const {
    gmem(Ye.at(it))[rl ? (size_t)n * s.K + m : (size_t)m * s.K + n] = v;
  }
};

// env'[yb][q][xb] = sum_a Y_e[a][yb] T[a][q][xb]
struct OpE3 {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  bool rl;
  const double *t3;
  size_t t3s;
  Ptr Ye, E;
  __device__ double a(int it, int m, int k) const {
    return rl ? Ye.at(it)[(size_t)m * s.K + k] : Ye.at(it)[(size_t)k * s.K + m];
  }
  __device__ double b(int it, int k, int n) const {
    return t3[(size_t)it * t3s + (size_t)k * N + n];
  }
  __device__ void st(int it, int m, int n, double v) const {
    E.at(it)[(size_t)m * N + n] = v;
  }
};

// Y <- Y . L with L[k][n] = R[n][k]: rows of the slot times the bond.
struct OpApplyL {
  int M, N, Kd;
  const int32_t *flag;
  Shape s;
  Ptr Y;
  const double *rbuf;
  double *tmp;
  size_t S;
  __device__ double a(int it, int m, int k) const {
    return Y.at(it)[(size_t)m * s.K + k];
  }
  __device__ double b(int it, int k, int n) const {
    return rbuf[(size_t)it * s.K * s.K + (size_t)n * s.K + k];
  }
  __device__ void st(int it, int m, int n, double v) const {
    tmp[(size_t)it * S + (size_t)m * s.K + n] = v;
  }
};

// Transfer-matrix steps of <a|b>.
struct OpOv1 {  // U[b'][q][a] = sum_{a'} E[a'][b'] a_i[a'][q][a]
  int M, N, Kd;
  const int32_t *flag;
  int K;
  const double *E;
  const double *const *ap;
  size_t off;
  double *U;
  size_t S;
  __device__ double a(int it, int m, int k) const {
    return E[(size_t)it * K * K + (size_t)k * K + m];
  }
  __device__ double b(int it, int k, int n) const {
    return ap[it][off + (size_t)k * N + n];
  }
  __device__ void st(int it, int m, int n, double v) const {
    U[(size_t)it * S + (size_t)m * N + n] = v;
  }
};
struct OpOv2 {  // E'[a][b] = sum_{b',q} U[b'][q][a] b_i[b'][q][b]
  int M, N, Kd;
  const int32_t *flag;
  int K, P;
  const double *U;
  size_t S;
  const double *const *bp;
  size_t off;
  double *E;
  __device__ double a(int it, int m, int k) const {
    return U[(size_t)it * S + (size_t)k * K + m];
  }
  __device__ double b(int it, int k, int n) const {
    return bp[it][off + (size_t)k * K + n];
  }
  __device__ void st(int it, int m, int n, double v) const {
    E[(size_t)it * K * K + (size_t)m * K + n] = v;
  }
};

// ---------------------------------------------------------------------------
// Fused fit visit on FP64 MFMA (v_mfma_f64_16x16x4f64).  One workgroup per
// (item, tile of TY front bonds yf); it walks all tiles of TX back bonds xb
// and, per tile, runs four LDS-resident contractions:
//   (a) T1[yf,wf][a,xb]      = sum_xf F[yf][wf][xf] X_f[xf][a][xb]
//   (b) T2[wfb,ab][s,lk,wbk] = sum_{wfk,ak} T1 Aket_f[s][wfk][lk][wbk][ak]  (per pair)
//   (c) T3[lk,wbk][lb,wbb]   = sum_{s,wfb,ab} T2 Abra_f[s][wfb][lb][wbb][ab] (per pair)
//   (e) Yt[yf,l][yb]        += sum_{xb,wb} T3 G[yb][wb][xb]
// T3 goes to HBM once (the environment update reads it); T1 and T2 never do.
// MFMA operand layout: lane l supplies A[l%16][l/16] and B[l/16][l%16];
// accumulator register r holds D[4r + l/16][l%16].
// ---------------------------------------------------------------------------
struct VisitArgs {
  int K, P, D, d, TY, TX;
  int rl, do_local;
  // true extents of site j of column c (null: the full bond cap K); only
  // the pair-per-wave D = 4 kernel uses them to skip zero padding
  const FitDims *dims;
  // where the padding is run all the same: the true extents that the same
  // kernel's sums are ordered by (null: the full bond cap)
  const FitDims *order;
  int W, c, j, N;
  Ptr F, X, G, Y;
  const double *aket;
  size_t aket_stride;
  const double *abra;
  size_t abra_stride;
  double *t3;
  size_t t3_stride;
};

constexpr int kVisitThreads = 512;
constexpr int kVisitWaves = kVisitThreads / 64;

// One batched LDS GEMM: for batch p < nb, C_p[M][N] = A_p[M][Kd] B_p[Kd][N];
// 16 x 16 output tiles spread over the waves, two per wave at a time when
// there are enough; each tile keeps two accumulators (even and odd k-steps)
// and its operands are read two k-steps ahead of the MFMAs.  afn/bfn read
// operands (zero outside), sfn stores the result tile element.  T: FP64, or
// FP32 on FP32 MFMA with FP32 accumulation; B16 (T = float): BF16 MFMA, 32
// k per step, lane slot s holding k = k0 + 4s + lq (slots 0-3 and 4-7 feed
// the two accumulators).
template <class T, bool B16 = false, class AF, class BF, class SF>
__device__ __forceinline__ void lds_gemm(int nb, int M, int N, int Kd, AF afn,
                                         BF bfn, SF sfn) {
  typedef Mma<T> MM;
  typedef typename MM::acc Acc;
  const Acc zero = Acc{0, 0, 0, 0};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int tm = (M + 15) >> 4, tn = (N + 15) >> 4;
  const int ntiles = nb * tm * tn;
  for (int t0 = wave; t0 < ntiles; t0 += 2 * kVisitWaves) {
    int p[2], m0[2], n0[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int t = min(t0 + h * kVisitWaves, ntiles - 1);
      p[h] = t / (tm * tn);
      const int r2 = t - p[h] * tm * tn;
      m0[h] = (r2 / tn) << 4;
      n0[h] = (r2 % tn) << 4;
    }
    const bool two = t0 + kVisitWaves < ntiles;
    Acc acc[2][2] = {{zero, zero}, {zero, zero}};
    if constexpr (B16) {
      static_assert(sizeof(T) == 4, "BF16 steps stage FP32 operands");
      for (int k0 = 0; k0 < Kd; k0 += 32) {
        float av[2][8], bv[2][8];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            const int k = k0 + 4 * s + lq, am = m0[h] + lr, bn = n0[h] + lr;
            const bool on = h == 0 || two;
            av[h][s] = (on && am < M && k < Kd) ? (float)afn(p[h], am, k) : 0.f;
            bv[h][s] = (on && bn < N && k < Kd) ? (float)bfn(p[h], k, bn) : 0.f;
          }
        const bool hi = k0 + 16 < Kd;  // slots 4-7 hold k0 + 16 .. k0 + 31
        acc[0][0] = mfma_bf16(av[0], bv[0], acc[0][0]);
        if (hi) acc[0][1] = mfma_bf16(av[0] + 4, bv[0] + 4, acc[0][1]);
        if (two) {
          acc[1][0] = mfma_bf16(av[1], bv[1], acc[1][0]);
          if (hi) acc[1][1] = mfma_bf16(av[1] + 4, bv[1] + 4, acc[1][1]);
        }
      }
    } else {
      for (int k0 = 0; k0 < Kd; k0 += 8) {
        T av[2][2], bv[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int k = k0 + 4 * u + lq, am = m0[h] + lr, bn = n0[h] + lr;
            const bool on = h == 0 || two;
            av[h][u] = (on && am < M && k < Kd) ? afn(p[h], am, k) : (T)0;
            bv[h][u] = (on && bn < N && k < Kd) ? bfn(p[h], k, bn) : (T)0;
          }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          acc[0][u] = MM::run(av[0][u], bv[0][u], acc[0][u]);
          if (two) acc[1][u] = MM::run(av[1][u], bv[1][u], acc[1][u]);
        }
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && !two) break;
      const Acc c = acc[h][0] + acc[h][1];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0[h] + MM::crow(r, lq), n = n0[h] + lr;
        if (m < M && n < N) sfn(p[h], m, n, c[r]);
      }
    }
  }
}

// Doubles of dynamic LDS for one fused-visit workgroup with tiles TY x TX.
__host__ __device__ inline size_t visit_lds(int K, int P, int d, int TY, int TX) {
  const size_t P2 = (size_t)P * P;
  return (size_t)TY * P * pad_a(K) + (size_t)K * pad_b(P * TX) + (size_t)TY * TX * P2 +
         (size_t)TY * TX * P * pad_b(d * P) + (size_t)TY * TX * P2 +
         (size_t)TX * P * pad_b(K) + 2 * (size_t)d * P2;
}

// DT > 0 fixes D (and P = D^2) at compile time; DT = 0 reads them at run time.
// B16 (T = float): every contraction on BF16 MFMA with FP32 accumulation.
// LDS layouts (index order, fastest last):
//   Fs [ty, wf][xf]          stride pad_a(K)
//   Xs [xf][a, tx]           stride pad_b(P TX)
//   T1s[pair][wfk, akx][wfb, abx]
//   T2s[pair][wfb, abx][s, lk, wbk]   stride pad_b(d P)
//   T3s[pair][wbk, wbb][lk, lb]
//   Gs [tx, wb][yb]          stride pad_b(K)
//   Ak, Ab [s][wf][a][l][wb] of the front view (ket and bra roles alike)
template <int DT, class T, bool B16 = false>
__global__ __launch_bounds__(kVisitThreads) void k_visit(VisitArgs v) {
  extern __shared__ double sm_raw[];
  T *sm = reinterpret_cast<T *>(sm_raw);
  typedef Mma<T> MM;
  typedef typename MM::acc Acc;
  constexpr bool kFixed = DT > 0;
  const int D = kFixed ? DT : v.D;
  const int P = kFixed ? DT * DT : v.P;
  const int K = v.K, d = v.d, TY = v.TY, TX = v.TX;
  const int dP = d * P, P2 = P * P;
  const int FS = pad_a(K), XS = pad_b(P * TX), T2S = pad_b(dP), GS = pad_b(K);
  const int it = blockIdx.y, y0 = blockIdx.x * TY;
  const int tid = threadIdx.x;
  T *Fs = sm;
  T *Xs = Fs + (size_t)TY * P * FS;
  T *T1s = Xs + (size_t)K * XS;
  T *T2s = T1s + (size_t)TY * TX * P2;
  T *T3s = T2s + (size_t)TY * TX * P * T2S;
  T *Gs = T3s + (size_t)TY * TX * P2;
  T *Ak = Gs + (size_t)TX * P * GS;
  T *Ab = Ak + (size_t)d * P2;
  const auto *F = gmem((const double *)v.F.at(it));
  const auto *X = gmem((const double *)v.X.at(it));
  const auto *G = gmem((const double *)v.G.at(it));
  const double *ak = v.aket + (size_t)it * v.aket_stride;
  const double *ab = v.abra + (size_t)it * v.abra_stride;
  T *T3g = reinterpret_cast<T *>(v.t3) + (size_t)it * v.t3_stride;
  const bool rl = v.rl != 0;

  // front-view site tensors A_f[s][wf][l][wb][a] (RL swaps the u/d legs),
  // stored as [s][wf][a][l][wb]
  for (int i = tid; i < d * P2; i += kVisitThreads) {
    int t = i;
    const int wb = t % D; t /= D;
    const int l = t % D; t /= D;
    const int a = t % D; t /= D;
    const int wf = t % D;
    const int s = t / D;
    const int u = rl ? wb : wf, dd = rl ? wf : wb;
    const size_t src = ((((size_t)s * D + u) * D + l) * D + dd) * D + a;
    Ak[i] = (T)ak[src];
    Ab[i] = (T)ab[src];
  }
  // F rows of this y tile: F[yf][wf][xf]
  for (int i = tid; i < TY * P * K; i += kVisitThreads) {
    const int row = i / K, xf = i - row * K;
    const int yf = y0 + row / P;
    Fs[row * FS + xf] = (T)(yf < K ? F[(size_t)(y0 * P + row) * K + xf] : 0.0);
  }
  // Yt accumulators: tiles of [(ty,l)][yb], kept in registers.  With at
  // most half as many tiles as waves, each tile's k range is split over two
  // waves (kh = 0, 1) and the halves are summed at the end.
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  const int Me = TY * P, tme = (Me + 15) >> 4, tne = (K + 15) >> 4;
  const int ntile_e = tme * tne;
  const bool split_e = 2 * ntile_e <= kVisitWaves;
  constexpr int kMaxE = 4;  // tiles per wave (host keeps ntile_e <= 4 * waves)
  Acc accE[kMaxE];
#pragma unroll
  for (int q = 0; q < kMaxE; ++q) accE[q] = Acc{0, 0, 0, 0};

  for (int x0 = 0; x0 < K; x0 += TX) {
    __syncthreads();  // previous tile's Xs/Gs/T3s consumers are done
    // X_f[xf][a][xb] for the tile, as Xs[xf][a*TX + tx]; the loop runs along
    // the contiguous global index (xb for LR, xf for RL)
    for (int i = tid; i < K * P * TX; i += kVisitThreads) {
      int xf, a, tx;
      if (rl) {
        xf = i % K;
        const int r = i / K;
        a = r % P;
        tx = r / P;
      } else {
        tx = i % TX;
        const int r = i / TX;
        a = r % P;
        xf = r / P;
      }
      const int xb = x0 + tx;
      double val = 0.0;
      if (xb < K)
        val = rl ? X[((size_t)xb * P + a) * K + xf] : X[((size_t)xf * P + a) * K + xb];
      Xs[xf * XS + a * TX + tx] = (T)val;
    }
    if (v.do_local)
      // G[yb][wb][xb] as Gs[(tx*P + wb)][yb], read along xb
      for (int i = tid; i < TX * P * K; i += kVisitThreads) {
        const int tx = i % TX, r = i / TX;
        const int wb = r % P, yb = r / P, xb = x0 + tx;
        Gs[(tx * P + wb) * GS + yb] = (T)(xb < K ? G[((size_t)yb * P + wb) * K + xb] : 0.0);
      }
    __syncthreads();
    // (a) T1: rows (ty, wf), cols (a, tx), stored [pair][wfk, akx][wfb, abx]
    lds_gemm<T, B16>(
        1, TY * P, P * TX, K,
        [&](int, int m, int k) { return Fs[m * FS + k]; },
        [&](int, int k, int n) { return Xs[k * XS + n]; },
        [&](int, int m, int n, T val) {
          const int ty = m / P, wf = m - ty * P, a = n / TX, tx = n - a * TX;
          const int wfk = wf / D, wfb = wf - wfk * D, akx = a / D, abx = a - akx * D;
          T1s[(ty * TX + tx) * P2 + (wfk * D + akx) * P + wfb * D + abx] = val;
        });
    __syncthreads();
    // (b) ket: per pair, rows m = (wfb, abx), k = (wfk, akx), cols n = (s, lk, wbk)
    lds_gemm<T, B16>(
        TY * TX, P, dP, P,
        [&](int p, int m, int k) { return T1s[p * P2 + k * P + m]; },
        [&](int, int k, int n) {
          const int s = n / P;
          return Ak[(s * P + k) * P + (n - s * P)];
        },
        [&](int p, int m, int n, T val) { T2s[(p * P + m) * T2S + n] = val; });
    __syncthreads();
    // (c) bra: per pair, rows m = (lk, wbk), k = (s, wfb, abx), cols n = (lb, wbb);
    // stored as T3s[pair][wb][l]
    lds_gemm<T, B16>(
        TY * TX, P, P, dP,
        [&](int p, int m, int k) {
          const int s = k / P;
          return T2s[(p * P + (k - s * P)) * T2S + s * P + m];
        },
        [&](int, int k, int n) { return Ab[k * P + n]; },
        [&](int p, int m, int n, T val) {
          const int lk = m / D, wbk = m - lk * D, lb = n / D, wbb = n - lb * D;
          T3s[p * P2 + (wbk * D + wbb) * P + lk * D + lb] = val;
        });
    __syncthreads();
    // T3 tile to HBM as T3[yf][l][xb][wb]
    for (int i = tid; i < TY * TX * P2; i += kVisitThreads) {
      int t = i;
      const int wb = t % P; t /= P;
      const int tx = t % TX; t /= TX;
      const int l = t % P;
      const int ty = t / P;
      const int yf = y0 + ty, xb = x0 + tx;
      if (yf < K && xb < K)
        T3g[(((size_t)yf * P + l) * K + xb) * P + wb] = T3s[(ty * TX + tx) * P2 + wb * P + l];
    }
    // (e) local update, accumulated over the xb tiles
    if (v.do_local) {
      const int Ke = TX * P;
      const int kh = split_e ? wave / (kVisitWaves / 2) : 0;
      const int wt = split_e ? wave % (kVisitWaves / 2) : wave;
      const int wstep = split_e ? kVisitWaves / 2 : kVisitWaves;
      const int kb = split_e ? kh * (Ke / 2) : 0, ke = split_e ? kb + Ke / 2 : Ke;
#pragma unroll
      for (int q = 0; q < kMaxE; ++q) {
        const int t = wt + q * wstep;
        if (t >= ntile_e) break;
        const int m0 = (t / tne) << 4, n0 = (t % tne) << 4;
        const int am = m0 + lr, bn = n0 + lr;
        const int ty = am / P, l = am - ty * P;
        Acc acc[2] = {accE[q], Acc{0, 0, 0, 0}};
        if constexpr (B16) {  // 32 k per step, slot s holding k0 + 4s + lq
          for (int k0 = kb; k0 < ke; k0 += 32) {
            float av[8], bv[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
              const int k = k0 + 4 * s + lq;
              const int tx = k / P, wb = k - tx * P;
              av[s] = (am < Me && k < ke) ? T3s[(ty * TX + tx) * P2 + wb * P + l] : 0.f;
              bv[s] = (bn < K && k < ke) ? Gs[k * GS + bn] : 0.f;
            }
            acc[0] = mfma_bf16(av, bv, acc[0]);
            if (k0 + 16 < ke) acc[1] = mfma_bf16(av + 4, bv + 4, acc[1]);
          }
        } else {
          for (int k0 = kb; k0 < ke; k0 += 8) {
            T av[2], bv[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int k = k0 + 4 * u + lq;
              const int tx = k / P, wb = k - tx * P;
              av[u] = (am < Me && k < ke) ? T3s[(ty * TX + tx) * P2 + wb * P + l] : (T)0;
              bv[u] = (bn < K && k < ke) ? Gs[k * GS + bn] : (T)0;
            }
            acc[0] = MM::run(av[0], bv[0], acc[0]);
            acc[1] = MM::run(av[1], bv[1], acc[1]);
          }
        }
        accE[q] = acc[0] + acc[1];
      }
    }
  }
  if (v.do_local && split_e) {  // add the second k half into the first
    __syncthreads();
    T *red = sm;  // every LDS buffer is free after the last tile
    if (wave >= kVisitWaves / 2) {
      const int wt = wave - kVisitWaves / 2;
#pragma unroll
      for (int q = 0; q < kMaxE; ++q) {
        const int t = wt + q * (kVisitWaves / 2);
        if (t >= ntile_e) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(t * 4 + r) * 64 + lane] = accE[q][r];
      }
    }
    __syncthreads();
    if (wave < kVisitWaves / 2) {
#pragma unroll
      for (int q = 0; q < kMaxE; ++q) {
        const int t = wave + q * (kVisitWaves / 2);
        if (t >= ntile_e) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) accE[q][r] += red[(t * 4 + r) * 64 + lane];
      }
    }
  }
  if (v.do_local && (!split_e || wave < kVisitWaves / 2)) {
    auto *Y = gmem(v.Y.at(it));
    const int wstep = split_e ? kVisitWaves / 2 : kVisitWaves;
#pragma unroll
    for (int q = 0; q < kMaxE; ++q) {
      const int t = wave + q * wstep;
      if (t >= ntile_e) break;
      const int m0 = (t / tne) << 4, n0 = (t % tne) << 4;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + MM::crow(r, lq), yb = n0 + lr;
        const int ty = m / P, l = m - ty * P, yf = y0 + ty;
        if (m < Me && yb < K && yf < K) {
          const size_t idx = rl ? ((size_t)yb * P + l) * K + yf
                                : ((size_t)yf * P + l) * K + yb;
          Y[idx] = (double)accE[q][r];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Fused fit visit specialised for D = 4 (P = 16) and d = 2, tiles TY x TX
// fixed at compile time.  Same four contractions and layouts as k_visit; every
// MFMA operand is read through a per-lane pointer with a compile-time step, the
// k loops are unrolled, and the operand tiles are zero-padded in LDS (rows and
// columns up to a multiple of 4 in k, of 16 in yb) so that no bounds test sits
// in an MFMA loop.
// ---------------------------------------------------------------------------
__host__ __device__ inline int ceil4(int x) { return (x + 3) & ~3; }
__host__ __device__ inline int ceil16(int x) { return (x + 15) & ~15; }

// LDS elements (of T) of one k_visit4 workgroup.
template <class T>
__host__ __device__ inline size_t visit4_lds(int K, int TY, int TX) {
  typedef Mma<T> M;
  const int K4 = ceil4(K);
  return (size_t)TY * 16 * M::pad_a(K4) + (size_t)K4 * M::pad_b(16 * TX) + (size_t)TY * TX * 256 +
         (size_t)TY * TX * 16 * M::pad_b(32) + (size_t)TY * TX * 256 +
         (size_t)TX * 16 * M::pad_b(K) + 2 * 2 * 256;
}

// acc[0] / acc[1] += sum over N k-steps (even / odd) of A(pa + i*da) B(pb + i*db)
template <int N, class T>
__device__ __forceinline__ void mma_steps(typename Mma<T>::acc (&acc)[2], const T *pa, int da,
                                          const T *pb, int db) {
  T av[N], bv[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    av[i] = pa[i * da];
    bv[i] = pb[i * db];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i & 1] = Mma<T>::run(av[i], bv[i], acc[i & 1]);
}

template <int TY, int TX, class T>
__global__ __launch_bounds__(kVisitThreads) void k_visit4(VisitArgs v) {
  extern __shared__ double sm_raw[];
  T *sm = reinterpret_cast<T *>(sm_raw);
  typedef Mma<T> M;
  typedef typename M::acc Acc;
  const Acc zero = Acc{0, 0, 0, 0};
  constexpr int D = 4, P = 16, P2 = 256, NP = TY * TX;
  constexpr int XS = M::pad_b(16 * TX), T2S = M::pad_b(32);
  const int K = v.K, K4 = ceil4(K), FS = M::pad_a(K4), GS = M::pad_b(K), KY = ceil16(K);
  const int it = blockIdx.y, y0 = blockIdx.x * TY;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  T *Fs = sm;
  T *Xs = Fs + TY * 16 * FS;
  T *T1s = Xs + K4 * XS;
  T *T2s = T1s + NP * P2;
  T *T3s = T2s + NP * 16 * T2S;
  T *Gs = T3s + NP * P2;
  T *Ak = Gs + TX * 16 * GS;
  T *Ab = Ak + 2 * P2;
  const auto *F = gmem((const double *)v.F.at(it));
  const auto *X = gmem((const double *)v.X.at(it));
  const auto *G = gmem((const double *)v.G.at(it));
  const double *ak = v.aket + (size_t)it * v.aket_stride;
  const double *ab = v.abra + (size_t)it * v.abra_stride;
  T *T3g = reinterpret_cast<T *>(v.t3) + (size_t)it * v.t3_stride;
  const bool rl = v.rl != 0;

  // site tensors as [s][wf][a][l][wb] of the front view (RL swaps u and d)
  for (int i = tid; i < 2 * P2; i += kVisitThreads) {
    const int wb = i & 3, l = (i >> 2) & 3, a = (i >> 4) & 3, wf = (i >> 6) & 3, s = i >> 8;
    const int u = rl ? wb : wf, dd = rl ? wf : wb;
    const int src = ((((s * D + u) * D + l) * D + dd) * D + a);
    Ak[i] = (T)ak[src];
    Ab[i] = (T)ab[src];
  }
  // F rows of the y tile, zero beyond K (and beyond the lattice edge in yf)
  for (int row = wave; row < TY * 16; row += kVisitWaves) {
    const bool ok = y0 + (row >> 4) < K;
    for (int xf = lane; xf < K4; xf += 64)
      Fs[row * FS + xf] = (T)((ok && xf < K) ? F[(size_t)(y0 * P + row) * K + xf] : 0.0);
  }
  // local-update accumulators: TY x (KY/16) tiles of [(ty, l)][yb]; each
  // tile's k range (tx, wb) is split over two waves when tiles are few
  const int tne = KY >> 4, ntile_e = TY * tne;
  const bool split_e = 2 * ntile_e <= kVisitWaves;
  constexpr int kMaxE = 4;
  Acc accE[kMaxE];
#pragma unroll
  for (int q = 0; q < kMaxE; ++q) accE[q] = zero;

  // The X and G tiles of the next xb step are fetched into registers while
  // the current step computes.  Each thread moves up to kLd elements of each;
  // their offsets (global relative to the tile, LDS) are decoded once.
  constexpr int kLd = 8;  // host keeps K4*16*TX and KY*16*TX within 8*512
  int xg[kLd], xl[kLd], gg[kLd], gl[kLd];
  T xr[kLd], gr[kLd];
#pragma unroll
  for (int u = 0; u < kLd; ++u) {
    const int i = tid + u * kVisitThreads;
    int xf, a, tx;
    if (rl) {
      xf = i % K4;
      const int r = i / K4;
      a = r & 15;
      tx = r >> 4;
    } else {
      tx = i % TX;
      const int r = i / TX;
      a = r & 15;
      xf = r >> 4;
    }
    const bool ok = i < K4 * 16 * TX && xf < K;
    xg[u] = !ok ? -1 : (rl ? (tx * P + a) * K + xf : (xf * P + a) * K + tx);
    xl[u] = i < K4 * 16 * TX ? xf * XS + a * TX + tx : -1;
    xl[u] |= (tx << 24);  // keep tx to test xb < K per step
    const int gtx = i % TX, gr2 = i / TX, wb = gr2 & 15, yb = gr2 >> 4;
    const bool gok = i < KY * 16 * TX && yb < K;
    gg[u] = gok ? (yb * P + wb) * K + gtx : -1;
    gl[u] = i < KY * 16 * TX ? ((gtx * 16 + wb) * GS + yb) | (gtx << 24) : -1;
  }
  auto fetch = [&](int x0) {
#pragma unroll
    for (int u = 0; u < kLd; ++u) {
      const int xtx = (xl[u] >> 24) & 0x7f, gtx = (gl[u] >> 24) & 0x7f;
      const size_t xo = rl ? (size_t)x0 * P * K : (size_t)x0;
      xr[u] = (T)((xg[u] >= 0 && x0 + xtx < K) ? X[xo + xg[u]] : 0.0);
      gr[u] = (T)((v.do_local && gg[u] >= 0 && x0 + gtx < K) ? G[(size_t)x0 + gg[u]] : 0.0);
    }
  };
  fetch(0);

  for (int x0 = 0; x0 < K; x0 += TX) {
    __syncthreads();  // the previous step's readers of Xs, Gs, T3s are done
#pragma unroll
    for (int u = 0; u < kLd; ++u) {
      if (xl[u] >= 0) Xs[xl[u] & 0xffffff] = xr[u];
      if (gl[u] >= 0) Gs[gl[u] & 0xffffff] = gr[u];
    }
    __syncthreads();
    if (x0 + TX < K) fetch(x0 + TX);
    // (a) T1: tiles (ty, tn): rows (ty, wf), cols n = (a, tx) in [16 tn, 16 tn + 16)
    for (int t = wave; t < TY * TX; t += kVisitWaves) {
      const int ty = t / TX, tn = t % TX;
      Acc acc[2] = {zero, zero};
      const T *pa = Fs + (ty * 16 + lr) * FS + lq;
      const T *pb = Xs + lq * XS + tn * 16 + lr;
      int k0 = 0;
      for (; k0 + 16 <= K4; k0 += 16) mma_steps<4>(acc, pa + k0, 4, pb + k0 * XS, 4 * XS);
      for (; k0 < K4; k0 += 4) mma_steps<1>(acc, pa + k0, 4, pb + k0 * XS, 4 * XS);
      const Acc c = acc[0] + acc[1];
      const int n = tn * 16 + lr, a = n / TX, tx = n % TX;
      T *dst = T1s + (ty * TX + tx) * P2 + (a >> 2) * 16 + (a & 3);
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // wf = (wfk, wfb)
        const int wf = M::crow(r, lq);
        dst[(wf >> 2) * 64 + (wf & 3) * 4] = c[r];
      }
    }
    __syncthreads();
    // (b) ket: per pair, rows m = (wfb, abx), k = (wfk, akx), cols n = (s, lk, wbk)
    for (int t = wave; t < 2 * NP; t += kVisitWaves) {
      const int pp = t >> 1, sn = t & 1;
      Acc acc[2] = {zero, zero};
      mma_steps<4>(acc, T1s + pp * P2 + lq * 16 + lr, 64, Ak + sn * P2 + lq * 16 + lr, 64);
      const Acc c = acc[0] + acc[1];
      T *dst = T2s + pp * 16 * T2S + sn * 16 + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) dst[M::crow(r, lq) * T2S] = c[r];
    }
    __syncthreads();
    // (c) bra: per pair, rows m = (lk, wbk), k = (s, wfb, abx), cols n = (lb, wbb)
    for (int t = wave; t < NP; t += kVisitWaves) {
      Acc acc[2] = {zero, zero};
#pragma unroll
      for (int sn = 0; sn < 2; ++sn)
        mma_steps<4>(acc, T2s + (t * 16 + lq) * T2S + sn * 16 + lr, 4 * T2S,
                     Ab + (sn * 16 + lq) * 16 + lr, 64);
      const Acc c = acc[0] + acc[1];
      // m = (lk, wbk), n = lr: lb = lr/4, wbb = lr%4
      T *dst = T3s + t * P2 + (lr & 3) * 16 + (lr >> 2);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = M::crow(r, lq);
        dst[(m & 3) * 64 + (m >> 2) * 4] = c[r];
      }
    }
    __syncthreads();
    // T3 tile to HBM as T3[yf][l][xb][wb]
    for (int i = tid; i < NP * P2; i += kVisitThreads) {
      const int wb = i & 15, r = i >> 4, tx = r % TX, r2 = r / TX, l = r2 & 15, ty = r2 >> 4;
      const int yf = y0 + ty, xb = x0 + tx;
      if (yf < K && xb < K)
        T3g[(((size_t)yf * P + l) * K + xb) * P + wb] = T3s[(ty * TX + tx) * P2 + wb * 16 + l];
    }
    // (e) local update: Yt[(ty, l)][yb] += sum_{tx, wb} T3[(ty, l)][(tx, wb)] G[(tx, wb)][yb]
    if (v.do_local) {
      const int half = split_e ? wave / (kVisitWaves / 2) : 0;
      const int wt = split_e ? wave % (kVisitWaves / 2) : wave;
      const int wstep = split_e ? kVisitWaves / 2 : kVisitWaves;
#pragma unroll
      for (int q = 0; q < kMaxE; ++q) {
        const int t = wt + q * wstep;
        if (t >= ntile_e) break;
        const int ty = t / tne, n0 = (t % tne) << 4;
        Acc acc[2] = {accE[q], zero};
#pragma unroll
        for (int tx = 0; tx < TX; ++tx)
#pragma unroll
          for (int wh = 0; wh < 2; ++wh) {  // wb in [8 wh, 8 wh + 8)
            if (split_e && ((tx * 2 + wh) & 1) != half) continue;
            mma_steps<2>(acc, T3s + (ty * TX + tx) * P2 + (wh * 8 + lq) * 16 + lr, 64,
                         Gs + (tx * 16 + wh * 8 + lq) * GS + n0 + lr, 4 * GS);
          }
        accE[q] = acc[0] + acc[1];
      }
    }
  }
  if (v.do_local && split_e) {  // add the second k half into the first
    __syncthreads();
    T *red = sm;
    if (wave >= kVisitWaves / 2) {
      const int wt = wave - kVisitWaves / 2;
#pragma unroll
      for (int q = 0; q < kMaxE; ++q) {
        const int t = wt + q * (kVisitWaves / 2);
        if (t >= ntile_e) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(t * 4 + r) * 64 + lane] = accE[q][r];
      }
    }
    __syncthreads();
    if (wave < kVisitWaves / 2) {
#pragma unroll
      for (int q = 0; q < kMaxE; ++q) {
        const int t = wave + q * (kVisitWaves / 2);
        if (t >= ntile_e) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) accE[q][r] += red[(t * 4 + r) * 64 + lane];
      }
    }
  }
  if (v.do_local && (!split_e || wave < kVisitWaves / 2)) {
    auto *Y = gmem(v.Y.at(it));
    const int wstep = split_e ? kVisitWaves / 2 : kVisitWaves;
#pragma unroll
    for (int q = 0; q < kMaxE; ++q) {
      const int t = wave + q * wstep;
      if (t >= ntile_e) break;
      const int ty = t / tne, n0 = (t % tne) << 4, yf = y0 + ty, yb = n0 + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = M::crow(r, lq);
        if (yb < K && yf < K) {
          const size_t idx = rl ? ((size_t)yb * P + l) * K + yf : ((size_t)yf * P + l) * K + yb;
          Y[idx] = (double)accE[q][r];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same visit with one (yf, xb) pair per wave (TY * TX waves): each wave
// runs T1 -> ket -> bra -> T3 store -> its local-update contribution for its
// own pair with wave-level LDS ordering only, so an xb step needs just the
// two barriers around the X/G refill.  The local-update partials of the TX
// waves that share yf are summed at the end in a fixed order.
//
// The ket's output tile for one s, C[(wfb, abx)][(lk, wbk)], sits in the MFMA
// accumulator with register i of lane (lr, lq) holding row 4i + lq (FP64) or
// 4lq + i (FP32) of column lr: that is the bra's A operand (rows (lk, wbk),
// k = (s, wfb, abx)) for k step i, with the bra's B rows read in the matching
// k order.  T2 therefore never leaves registers.  T1 and T3 share one LDS
// region per pair (T1 is consumed by the ket before the bra writes T3).
//
// NE = ceil(K / 16) bounds the local-update tiles; each thread moves LD
// elements of the X and G tiles per step.
// LDS: Fs [(ty, wf)][xf] (row stride pad_a_min(K4)); Xs [tx][xf][a] (rows
// of 16, tile stride 16 K4 + 32 / TX); per pair T1 [wfk,akx][wfb,abx] and
// T3 [wbk,wbb][lk,lb] (rows of 16); Gs [(tx, wb)][yb] (stride pad_b(K));
// Ak, Ab [s][wf][a][l][wb].  Rows of Fs, Xs, T1, T3 and Gs are stored with
// their column index XOR-ed by a function of the row (v4p_*_sw below), which
// leaves every MFMA operand read conflict-free and also makes the accesses
// that walk a column (the refill stores, the MFMA result stores, the T3 read
// for the HBM store) hit distinct LDS banks, for both a half wave over 32
// 8-byte banks and a quarter wave over 16 (the F, T1 and T3 swizzles were
// chosen to satisfy both).
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int v4p_x_sw(int xf) { return (xf >> 1) & 15; }
__host__ __device__ constexpr int v4p_t1_sw(int k) { return (k & 3) << 2; }
__host__ __device__ constexpr int v4p_t3_sw(int wb) {
  return ((wb & 3) << 2) ^ (((wb >> 2) & 1) * 5) ^ (((wb >> 3) & 1) << 1);
}
__host__ __device__ constexpr int v4p_f_sw(int row) { return (row >> 3) & 1; }
__host__ __device__ constexpr int v4p_g_sw(int row) { return ((row >> 1) ^ ((row >> 4) << 2)) & 15; }
__host__ __device__ constexpr int v4p_xt(int K4, int TX) { return 16 * K4 + 32 / TX; }
template <class T>
__host__ __device__ inline size_t visit4p_lds(int K, int TY, int TX) {
  typedef Mma<T> M;
  const int K4 = ceil4(K), tne = ceil16(K) / 16;
  const size_t body = (size_t)TY * 16 * M::pad_a_min(K4) + (size_t)TX * v4p_xt(K4, TX) +
                      (size_t)TY * TX * 256 + (size_t)TX * 16 * M::pad_b(K) + 2 * 2 * 256;
  return std::max(body, (size_t)TY * TX * tne * 256);
}

// One wave per (yf, xb) pair of a TY x TX tile: NT threads.  LD elements of
// each of the X and G tiles (16 NE x 16 x TX) per thread and step.  Up to
// NE = 3 (K <= 48) three workgroups share a CU (2 x 2 pairs at NE = 2, LDS
// <= 47 KB; 4 x 1 at NE = 3, LDS <= 52 KB), so the registers are held to 3
// waves per SIMD; at NE = 4 to 2, and for the 1 x 4 tiles of small batches
// (which leave most of the CUs free anyway) to 2.
template <int TY, int TX, int NE>
struct Visit4pShape {
  static constexpr int NWV = TY * TX, NT = 64 * NWV;
  static constexpr int LD = (NE * 16 * 16 * TX + NT - 1) / NT;
};

template <int TY, int TX, class T, int NE>
__global__ __launch_bounds__(64 * TY * TX)
__attribute__((amdgpu_waves_per_eu(NE <= 3 && TY > 1 ? 3 : 2)))
void k_visit4p(VisitArgs v) {
  constexpr int NT = Visit4pShape<TY, TX, NE>::NT, NWV = Visit4pShape<TY, TX, NE>::NWV;
  extern __shared__ double sm_raw[];
  T *sm = reinterpret_cast<T *>(sm_raw);
  typedef Mma<T> M;
  typedef typename M::acc Acc;
  const Acc zero = Acc{0, 0, 0, 0};
  constexpr int D = 4, P = 16, P2 = 256, NP = TY * TX;
  constexpr int LD = Visit4pShape<TY, TX, NE>::LD;
  constexpr bool f64 = sizeof(T) == 8;
  const int K = v.K, K4 = ceil4(K), FS = M::pad_a_min(K4), GS = M::pad_b(K), KY = ceil16(K);
  const int XT = v4p_xt(K4, TX);
  int tile, it;
  xcd_tile_item(&tile, &it);
  const int y0 = tile * TY;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lq = lane >> 4;
  // True extents of this item's operands; every slot entry beyond them is
  // zero, so tiles, xb steps, k blocks and local-update tiles past them
  // would only add zeros: they are skipped, which leaves every sum's order
  // over its nonzero terms, and so its bits, unchanged.  Y is still written
  // in full (zeros in the padding).
  int nyf = K, nyb = K, nxf = K, nxb = K;
  if (v.dims) {
    const SiteExt ex = site_ext(v.dims[(size_t)it * v.W + v.c], v.j, v.N, v.rl != 0);
    nyf = ex.yf;
    nyb = ex.yb;
    nxf = ex.xf;
    nxb = ex.xb;
  }
  if (y0 >= nyf) {  // every front bond of the tile is padding: Y rows are zero
    if (v.do_local) {
      auto *Yz = gmem(v.Y.at(it));
      const int rows = min(TY, K - y0);
      for (int i = tid; i < rows * P * K; i += NT) {
        const int yb = i % K, l = (i / K) % P, yf = y0 + i / (K * P);
        Yz[v.rl ? ((size_t)yb * P + l) * K + yf : ((size_t)yf * P + l) * K + yb] = 0.0;
      }
    }
    return;
  }
  const int K4x = ceil4(nxf), tnb = ceil16(nyb) >> 4;
  // T1 sums whole blocks of 16 xf in two chains and the rest in one: cut at the
  // true X bond also where the padding is run, so that both sum alike
  int K4s = K4x;
  if (v.order) K4s = ceil4(site_ext(v.order[(size_t)it * v.W + v.c], v.j, v.N, v.rl != 0).xf);
  T *Fs = sm;
  T *Xs = Fs + TY * 16 * FS;
  T *T13s = Xs + TX * XT;
  T *Gs = T13s + NP * P2;
  T *Ak = Gs + TX * 16 * GS;
  T *Ab = Ak + 2 * P2;
  const auto *F = gmem((const double *)v.F.at(it));
    const double *ak = v.aket + (size_t)it * v.aket_stride;
  const double *ab = v.abra + (size_t)it * v.abra_stride;
  T *T3g = reinterpret_cast<T *>(v.t3) + (size_t)it * v.t3_stride;
  const __amdgpu_buffer_rsrc_t t3rs =
      __builtin_amdgcn_make_buffer_rsrc(T3g, 0, (int)((unsigned)K * P * K * P * sizeof(T)), 0x00020000);
  const bool rl = v.rl != 0;
  const int ty = wave / TX, tx = wave % TX, pp = wave;  // this wave's pair
  T *Tp = T13s + pp * P2;

  for (int i = tid; i < 2 * P2; i += NT) {
    const int wb = i & 3, l = (i >> 2) & 3, a = (i >> 4) & 3, wf = (i >> 6) & 3, s = i >> 8;
    const int u = rl ? wb : wf, dd = rl ? wf : wb;
    const int src = ((((s * D + u) * D + l) * D + dd) * D + a);
    Ak[i] = (T)ak[src];
    Ab[i] = (T)ab[src];
  }
  for (int row = wave; row < TY * 16; row += NWV) {
    const bool ok = y0 + (row >> 4) < nyf;
    for (int xf = lane; xf < K4; xf += 64)
      Fs[row * FS + (xf ^ v4p_f_sw(row))] = (T)((ok && xf < nxf) ? F[(size_t)(y0 * P + row) * K + xf] : 0.0);
  }
  const int tne = KY >> 4;  // <= NE
  Acc accE[NE];
#pragma unroll
  for (int q = 0; q < NE; ++q) accE[q] = zero;

  // X and G of the next xb step are fetched into registers while the
  // current step computes.  Thread element u is i = tid + NT u of the tile
  // [xf][a][tx] (rl: [tx][a][xf]) and [yb][wb][tx], each index taken over
  // the compile-time extent XF = 16 NE >= K4; the decode is recomputed where
  // needed rather than held in registers.
  constexpr int XF = 16 * NE, NX = XF * 16 * TX;
  auto xdec = [&](int u, int &txx, int &a, int &xf) {
    const int i = tid + u * NT;
    if (rl) {
      xf = i % XF;
      a = (i / XF) & 15;
      txx = i / (XF * 16);
    } else {
      txx = i % TX;
      a = (i / TX) & 15;
      xf = i / (TX * 16);
    }
  };
  auto gdec = [&](int u, int &gtx, int &wb, int &yb) {
    const int i = tid + u * NT;
    gtx = i % TX;
    wb = (i / TX) & 15;
    yb = i / (TX * 16);
  };
  // raw loads of the pending step: nothing waits on them before the refill at
  // the next step.  X and G of one item are K P K doubles each; an element
  // outside the tile loads at offset K P K doubles, past the descriptor's
  // range, and reads zero.  Without the local update there is no G (null):
  // nothing is loaded from it.
  double xr[LD], gr[LD];
  const unsigned xgbytes = (unsigned)K * P * K * sizeof(double);
  const __amdgpu_buffer_rsrc_t xrs = buf_rsrc(v.X.at(it), xgbytes);
  const __amdgpu_buffer_rsrc_t grs = buf_rsrc(v.do_local ? v.G.at(it) : v.X.at(it), xgbytes);
  auto fetch = [&](int x0) {
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      int txx, a, xf;
      xdec(u, txx, a, xf);
      const bool xv = tid + u * NT < NX && xf < nxf && x0 + txx < nxb;
      const unsigned off = rl ? ((x0 + txx) * P + a) * K + xf : (xf * P + a) * K + x0 + txx;
      xr[u] = buf_ld(xrs, xv ? off * 8u : xgbytes);
    }
    if (v.do_local) {
#pragma unroll
      for (int u = 0; u < LD; ++u) {
        int gtx, wb, yb;
        gdec(u, gtx, wb, yb);
        const bool gv = tid + u * NT < NX && yb < nyb && x0 + gtx < nxb;
        gr[u] = buf_ld(grs, gv ? ((yb * P + wb) * K + x0 + gtx) * 8u : xgbytes);
      }
    }
  };
  fetch(0);

  for (int x0 = 0; x0 < nxb; x0 += TX) {
    __syncthreads();  // the previous step's readers of Xs, Gs and T3 are done
#pragma unroll
    for (int u = 0; u < LD; ++u) {  // rows up to K4 and K rows of G (zero where not real)
      if (tid + u * NT >= NX) continue;
      int txx, a, xf, gtx, wb, yb;
      xdec(u, txx, a, xf);
      gdec(u, gtx, wb, yb);
      if (xf < K4) Xs[txx * XT + xf * 16 + (a ^ v4p_x_sw(xf))] = (T)xr[u];
      const int grow = gtx * 16 + wb;
      if (yb < KY) Gs[grow * GS + (yb ^ v4p_g_sw(grow))] = (T)(v.do_local ? gr[u] : 0.0);
    }
    __syncthreads();
    if (x0 + TX < nxb) fetch(x0 + TX);
    // (a) T1 of the pair: rows wf, cols a, k = xf
    {
      Acc acc[2] = {zero, zero};
      const T *pa = Fs + (ty * 16 + lr) * FS + (lq ^ v4p_f_sw(lr));
      const T *px = Xs + tx * XT;
      // Xs row xf = k0 + lq (k0 = 0 mod 4): swizzle ((k0 >> 1) & 15) ^ (lq >> 1)
      const int xb0 = lq * 16 + (lr ^ (lq >> 1));
      int k0 = 0;
      for (; k0 + 16 <= K4s; k0 += 16) {
        const T *pk = px + k0 * 16;
        const int sw = (k0 >> 1) & 8;
        T av[4], bv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          av[i] = pa[k0 + 4 * i];
          bv[i] = pk[(xb0 ^ (sw | 2 * i)) + 64 * i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i & 1] = M::run(av[i], bv[i], acc[i & 1]);
      }
      for (; k0 < K4x; k0 += 4)
        acc[0] = M::run(pa[k0], px[k0 * 16 + (xb0 ^ ((k0 >> 1) & 15))], acc[0]);
      const Acc c = acc[0] + acc[1];
      // a = lr (akx = lr/4, abx = lr%4), wf = (wfk, wfb): row (wfk, akx),
      // column (wfb, abx)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int wf = M::crow(r, lq), row = (wf >> 2) * 4 + (lr >> 2);
        Tp[row * 16 + (((wf & 3) * 4 + (lr & 3)) ^ v4p_t1_sw(row))] = c[r];
      }
    }
    wave_lds_order();
    // (b) ket, one tile per s: rows m = (wfb, abx), k = (wfk, akx), cols n = (lk, wbk)
    Acc t2[2];
#pragma unroll
    for (int sn = 0; sn < 2; ++sn) {
      Acc acc[2] = {zero, zero};
      // T1 row 4i + lq: its swizzle depends on lq only
      mma_steps<4>(acc, Tp + lq * 16 + (lr ^ v4p_t1_sw(lq)), 64, Ak + sn * P2 + lq * 16 + lr, 64);
      t2[sn] = acc[0] + acc[1];
    }
    wave_lds_order();  // every lane's T1 reads precede the T3 writes below
    // (c) bra: rows m = (lk, wbk), k = (s, wfb, abx), cols n = (lb, wbb); the
    // A operand of k step i is register i of t2[s]
    {
      Acc acc[2] = {zero, zero};
#pragma unroll
      for (int sn = 0; sn < 2; ++sn) {
        // B rows in the order the accumulator holds k: 4i + lq (FP64), 4lq + i (FP32)
        const T *pb = f64 ? Ab + (sn * 16 + lq) * 16 + lr : Ab + (sn * 16 + 4 * lq) * 16 + lr;
        constexpr int db = f64 ? 64 : 16;
        T bv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) bv[i] = pb[i * db];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i & 1] = M::run(t2[sn][i], bv[i], acc[i & 1]);
      }
      const Acc c = acc[0] + acc[1];
#pragma unroll
      for (int r = 0; r < 4; ++r) {  // m = (lk, wbk), n = lr = (lb, wbb)
        const int m = M::crow(r, lq), wb = (m & 3) * 4 + (lr & 3), l = (m >> 2) * 4 + (lr >> 2);
        Tp[wb * 16 + (l ^ v4p_t3_sw(wb))] = c[r];
      }
    }
    wave_lds_order();
    // T3 of the pair to HBM as T3[yf][l][xb][wb] (16 lanes per 128-byte row),
    // through the item's descriptor (32-bit offsets)
    {
      const int yf = y0 + ty, xb = x0 + tx;
      if (yf < nyf && xb < nxb) {
        const unsigned o0 = (unsigned)(yf * P * K + xb) * P;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int idx = u * 64 + lane, wb = idx & 15, l = idx >> 4;
          buf_st_t<T>(t3rs, (o0 + (unsigned)(l * K * P + wb)) * (unsigned)sizeof(T),
                      Tp[wb * 16 + (l ^ v4p_t3_sw(wb))]);
        }
      }
    }
    // (e) this pair's contribution to Yt[(ty, l)][yb]: k = wb of column tx
    if (v.do_local) {
      // A: T3 row wb = 4i + lq, column lr: swizzle t3_sw(lq) ^ t3_sw(4i) (linear);
      // B: Gs row tx 16 + 4i + lq: swizzle w ^ (lq >> 1) ^ 2i, w from tx
      const int ta = lq * 16 + (lr ^ v4p_t3_sw(lq));
      const int w = ((tx & 1) << 3) ^ ((tx << 2) & 15);
      const int gb = (tx * 16 + lq) * GS + (lr ^ w ^ (lq >> 1));
#pragma unroll
      for (int q = 0; q < NE; ++q) {
        if (q >= tnb) break;
        T av[4], bv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          av[i] = Tp[(ta ^ v4p_t3_sw(4 * i)) + 64 * i];
          bv[i] = Gs[(gb ^ (2 * i)) + 4 * i * GS + q * 16];
        }
        Acc acc[2] = {accE[q], zero};
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i & 1] = M::run(av[i], bv[i], acc[i & 1]);
        accE[q] = acc[0] + acc[1];
      }
    }
  }
  if (!v.do_local) return;
  // sum the TX partials of each yf tile in a fixed order (tx = 0, 1, ...)
  __syncthreads();
  T *red = sm;
#pragma unroll
  for (int q = 0; q < NE; ++q) {
    if (q >= tne) break;
#pragma unroll
    for (int r = 0; r < 4; ++r) red[((pp * tne + q) * 4 + r) * 64 + lane] = accE[q][r];
  }
  __syncthreads();
  if (tx != 0) return;
  auto *Y = gmem(v.Y.at(it));
  const int yf = y0 + ty;
#pragma unroll
  for (int q = 0; q < NE; ++q) {
    if (q >= tne) break;
    const int yb = q * 16 + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      T acc = red[((pp * tne + q) * 4 + r) * 64 + lane];
      for (int t2i = 1; t2i < TX; ++t2i) acc += red[(((pp + t2i) * tne + q) * 4 + r) * 64 + lane];
      const int l = M::crow(r, lq);
      if (yb < K && yf < K) {
        const size_t idx = rl ? ((size_t)yb * P + l) * K + yf : ((size_t)yf * P + l) * K + yb;
        Y[idx] = (double)acc;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The pair-per-wave visit for the other bond dimensions (D = 2, 3, 5, 6;
// d = 2, bond caps <= 64, FP64).  As above each wave takes one (yf, xb) pair
// through T1 -> ket -> bra -> T3 -> local update with wave-level LDS ordering,
// T2 stays in registers, and an xb step has the two barriers of the X/G
// refill.  The fused leg P = D^2 fills PT = ceil(P / 16) MFMA tiles; a tile's
// rows and columns past P hold whatever lies behind in LDS and are never
// stored, only the contracted index needs zeros there (the last k step of a
// P-long sum masks both operands when 4 does not divide P).  F is held in
// registers (the A operand of T1, the same for every xb).
//
// Bound by what a wave waits for between its MFMAs, not by their rate: at D = 6,
// K = 64 (576 MFMAs a pair, 64 % of them on real entries) the matrix cores are
// busy 35 % of the launch, because F, T3 and accE fill all 512 registers of the
// one wave a SIMD holds (48 more spilled) and nothing covers its LDS reads; at D
// = 3 (23 MFMAs a pair at K = 18) a launch is a few steps long and they are busy
// 10 %.  k_visit, which the shapes used before, runs the same contractions phase
// by phase over one workgroup (six barriers a step, index decodes by division at
// every element).  A launch there and here: the 24 to 48 messages of a D = 3, chi
// = 18 sweep 54.6 and 19.4 us, one D = 3, chi = 15 message 24.8 and 9.9 us, one D
// = 6, chi = 64 message 1053 and 105 us (27 TFLOP/s of real entries).
//
// Tiles: TX = 4 pairs along xb of one yf (TY = 1) where four X and G tiles
// fit in LDS (D <= 3; D = 5, 6 up to 32 rows), so that a single message still
// spreads over K workgroups; otherwise four yf of one xb, with the xb range
// split over `nsplit` workgroups (see visitp_tiles).
// ---------------------------------------------------------------------------
template <int D, int TY, int TX, int NE>
struct VisitPShape {
  static constexpr int P = D * D, PT = (P + 15) / 16, PK = (P + 3) / 4, NW = TY * TX,
                       NT = 64 * NW, XF = 16 * NE;
  // LDS row strides (doubles): 16 (mod 32) keeps the two k rows a half wave
  // reads in different banks; D >= 5 with TX = 4 has no room for that
  static constexpr bool tight = D >= 5 && TX > 1;
  static constexpr int TS = tight ? P : (P <= 16 ? 16 : 48);
  static constexpr int GS = tight ? XF : XF + (NE % 2 ? 0 : 16);
  static constexpr int nT = NW * P * TS, nA = 2 * P * TS, nX = TX * XF * TS, nG = TX * P * GS;
  static constexpr int nRed = TX > 1 ? NW * PT * NE * 256 : 0;
  // 64 doubles behind the last array: reads of padded rows and columns
  static constexpr int body = nT + 2 * nA + nX + nG + 64;
  static constexpr size_t lds = sizeof(double) * (body > nRed ? body : nRed);
  static constexpr int LDX = (XF * P * TX + NT - 1) / NT;
};

struct VisitPArgs {
  VisitArgs v;
  int nsplit;        // xb ranges, one per workgroup of a yf tile
  double *part;      // nsplit > 1: partial Yt, [item][split][K P K]
  size_t part_stride;
  const FitDims *dims;  // true bonds that the split is cut by (null: the bond cap)
};

template <int D, int TY, int TX, int NE>
__global__ __launch_bounds__(64 * TY * TX)
__attribute__((amdgpu_waves_per_eu(D >= 5 ? 1 : (D == 3 && NE > 2 ? 2 : 3))))
void k_visitp(VisitPArgs g) {
  typedef VisitPShape<D, TY, TX, NE> Sh;
  constexpr int P = Sh::P, PT = Sh::PT, PK = Sh::PK, NT = Sh::NT, XF = Sh::XF, TS = Sh::TS,
                GS = Sh::GS, LDX = Sh::LDX;
  extern __shared__ double sm_raw[];
  const VisitArgs &v = g.v;
  const int K = v.K;
  int tile, it;
  xcd_tile_item(&tile, &it);
  const int sp = tile % g.nsplit, y0 = (tile / g.nsplit) * TY;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int ty = wave / TX, tx = wave % TX, yf = y0 + ty;
  const bool rl = v.rl != 0;
  // true extents of this item's operands (see k_visit4p)
  int nyf = K, nyb = K, nxf = K, nxb = K;
  if (v.dims) {
    const SiteExt ex = site_ext(v.dims[(size_t)it * v.W + v.c], v.j, v.N, rl);
    nyf = ex.yf;
    nyb = ex.yb;
    nxf = ex.xf;
    nxb = ex.xb;
  }
  // this workgroup's xb range: nsplit contiguous ranges of whole steps, cut by
  // the true bond also where the padding is run (the last one takes it then),
  // so that the partial sums hold the same terms either way
  int steps = (nxb + TX - 1) / TX;
  if (g.dims) {
    const SiteExt ex = site_ext(g.dims[(size_t)it * v.W + v.c], v.j, v.N, rl);
    steps = (ex.xb + TX - 1) / TX;
  }
  const int xlo = steps * sp / g.nsplit * TX;
  const int xhi = sp == g.nsplit - 1 ? nxb : min(nxb, steps * (sp + 1) / g.nsplit * TX);
  double *Yout = g.nsplit > 1
                     ? g.part + (size_t)it * g.part_stride + (size_t)sp * K * P * K
                     : v.Y.at(it);
  if (y0 >= nyf) {  // every front bond of the tile is padding: Y rows are zero
    if (v.do_local) {
      const int rows = min(TY, K - y0);
      for (int i = tid; i < rows * P * K; i += NT) {
        const int yb = i % K, l = (i / K) % P, y = y0 + i / (K * P);
        gmem(Yout)[rl ? ((size_t)yb * P + l) * K + y : ((size_t)y * P + l) * K + yb] = 0.0;
      }
    }
    return;
  }
  double *Tp = sm_raw + wave * P * TS;  // this wave's T1, then T3
  double *Ak = sm_raw + Sh::nT;
  double *Ab = Ak + Sh::nA;
  double *Xs = Ab + Sh::nA;
  double *Gs = Xs + Sh::nX;
  const unsigned xgbytes = (unsigned)K * P * K * 8u;
  const __amdgpu_buffer_rsrc_t xrs = buf_rsrc(v.X.at(it), xgbytes);
  const __amdgpu_buffer_rsrc_t frs = buf_rsrc(v.F.at(it), xgbytes);
  const __amdgpu_buffer_rsrc_t grs = buf_rsrc(v.do_local ? v.G.at(it) : v.X.at(it), xgbytes);
  double *T3g = v.t3 + (size_t)it * v.t3_stride;
  const __amdgpu_buffer_rsrc_t t3rs = buf_rsrc(T3g, (unsigned)K * P * K * P * 8u);

  // site tensors of the front view (RL swaps u and d) as [s][wf, a][l, wb]
  {
    const auto *ak = gmem(v.aket + (size_t)it * v.aket_stride);
    const auto *ab = gmem(v.abra + (size_t)it * v.abra_stride);
    for (int i = tid; i < 2 * P * P; i += NT) {
      const int n = i % P, k = (i / P) % P, s = i / (P * P);
      const int wb = n % D, l = n / D, a = k % D, wf = k / D;
      const int src = (((s * D + (rl ? wb : wf)) * D + l) * D + (rl ? wf : wb)) * D + a;
      Ak[(s * P + k) * TS + n] = ak[src];
      Ab[(s * P + k) * TS + n] = ab[src];
    }
  }
  // F rows of this wave's yf: A operand of T1 (row wf, k = xf), zero outside
  double fr[PT][4 * NE];
#pragma unroll
  for (int mt = 0; mt < PT; ++mt)
#pragma unroll
    for (int ks = 0; ks < 4 * NE; ++ks) {
      const int wf = 16 * mt + lr, xf = 4 * ks + lq;
      const bool ok = wf < P && xf < nxf && yf < nyf;
      fr[mt][ks] = buf_ld(frs, ok ? (unsigned)((yf * P + wf) * K + xf) * 8u : xgbytes);
    }
  v4d accE[PT][NE];
#pragma unroll
  for (int mt = 0; mt < PT; ++mt)
#pragma unroll
    for (int q = 0; q < NE; ++q) accE[mt][q] = v4d{0.0, 0.0, 0.0, 0.0};

  // X [xf][a] and G [wb][yb] of the next step, fetched into registers while
  // the current one computes (up to 10 elements a thread; where TX = 4 tiles
  // of D >= 5 take more, they are loaded at the refill: a step there computes
  // for 13 us); elements outside load past the descriptor's end (zero).
  // Element u of a thread is i = tid + NT u of [tx][a][xf] (RL) or
  // [xf][a][tx] (LR), and of [yb][wb][tx].
  constexpr bool pre = LDX <= 10;
  double xr[LDX], gr[LDX];
  auto xdec = [&](int u, int &txx, int &a, int &xf) __attribute__((always_inline)) {
    const int i = tid + u * NT;
    if (rl) {
      xf = i % XF;
      a = (i / XF) % P;
      txx = i / (XF * P);
    } else {
      txx = i % TX;
      a = (i / TX) % P;
      xf = i / (TX * P);
    }
  };
  auto gdec = [&](int u, int &txx, int &wb, int &yb) __attribute__((always_inline)) {
    const int i = tid + u * NT;
    txx = i % TX;
    wb = (i / TX) % P;
    yb = i / (TX * P);
  };
  auto fetch = [&](int x0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < LDX; ++u) {
      int txx, a, xf;
      xdec(u, txx, a, xf);
      const int xb = x0 + txx;
      const bool ok = tid + u * NT < XF * P * TX && xf < nxf && xb < xhi;
      const unsigned off = rl ? (xb * P + a) * K + xf : (xf * P + a) * K + xb;
      xr[u] = buf_ld(xrs, ok ? off * 8u : xgbytes);
    }
    if (v.do_local) {
#pragma unroll
      for (int u = 0; u < LDX; ++u) {
        int txx, wb, yb;
        gdec(u, txx, wb, yb);
        const int xb = x0 + txx;
        const bool ok = tid + u * NT < XF * P * TX && yb < nyb && xb < xhi;
        gr[u] = buf_ld(grs, ok ? (unsigned)((yb * P + wb) * K + xb) * 8u : xgbytes);
      }
    }
  };
  auto refill = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < LDX; ++u) {
      int txx, a, xf;
      xdec(u, txx, a, xf);
      if (tid + u * NT < XF * P * TX) Xs[(txx * XF + xf) * TS + a] = xr[u];
    }
    if (v.do_local) {
#pragma unroll
      for (int u = 0; u < LDX; ++u) {
        int txx, wb, yb;
        gdec(u, txx, wb, yb);
        if (tid + u * NT < XF * P * TX) Gs[(txx * P + wb) * GS + yb] = gr[u];
      }
    }
  };
  if (pre && xlo < xhi) fetch(xlo);

  for (int x0 = xlo; x0 < xhi; x0 += TX) {
    if (!pre) fetch(x0);
    __syncthreads();  // the previous step's readers of Xs and Gs are done
    refill();
    __syncthreads();
    if (pre && x0 + TX < xhi) fetch(x0 + TX);
    const int xb = x0 + tx;
    if (xb >= xhi || yf >= nyf) continue;  // a wave without a pair
    // (a) T1: rows wf, cols a, k = xf; stored [wfk, akx][wfb, abx]
    {
      v4d acc[PT][PT];
#pragma unroll
      for (int mt = 0; mt < PT; ++mt)
#pragma unroll
        for (int nt = 0; nt < PT; ++nt) acc[mt][nt] = v4d{0.0, 0.0, 0.0, 0.0};
      const double *px = Xs + (tx * XF + lq) * TS + lr;
      static_for<0, 4 * NE>([&](auto KS) __attribute__((always_inline)) {
        constexpr int ks = decltype(KS)::value;
        if (4 * ks >= nxf) return;
#pragma unroll
        for (int nt = 0; nt < PT; ++nt) {
          const double b = px[4 * ks * TS + 16 * nt];
#pragma unroll
          for (int mt = 0; mt < PT; ++mt) acc[mt][nt] = mfma16(fr[mt][ks], b, acc[mt][nt]);
        }
        // large tiles: operand reads stay near their MFMAs, not in registers
        if (PT > 1 && ks % 2) __builtin_amdgcn_sched_barrier(0);
      });
#pragma unroll
      for (int mt = 0; mt < PT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int wf = 16 * mt + 4 * r + lq;
          if (16 * mt + 4 * r >= P) continue;
#pragma unroll
          for (int nt = 0; nt < PT; ++nt) {
            const int a = 16 * nt + lr;
            if (wf < P && a < P)
              Tp[((wf / D) * D + a / D) * TS + (wf % D) * D + a % D] = acc[mt][nt][r];
          }
        }
    }
    wave_lds_order();
    // (b), (c) per column tile (lk, wbk) of the ket's output: its accumulator
    // register i of tile mt is the bra's A operand for k = 16 mt + 4 i + lq
    v4d t3[PT][PT];
#pragma unroll
    for (int nt = 0; nt < PT; ++nt) {
#pragma unroll
      for (int n2 = 0; n2 < PT; ++n2) t3[nt][n2] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        v4d t2[PT];
#pragma unroll
        for (int mt = 0; mt < PT; ++mt) t2[mt] = v4d{0.0, 0.0, 0.0, 0.0};
        const double *pa = Tp + lq * TS + lr, *pb = Ak + (s * P + lq) * TS + 16 * nt + lr;
#pragma unroll
        for (int ks = 0; ks < PK; ++ks) {
          const bool in = 4 * ks + 3 < P || 4 * ks + lq < P;
          const double b = in ? pb[4 * ks * TS] : 0.0;
#pragma unroll
          for (int mt = 0; mt < PT; ++mt)
            t2[mt] = mfma16(in ? pa[4 * ks * TS + 16 * mt] : 0.0, b, t2[mt]);
          if (PT > 1 && ks % 2) __builtin_amdgcn_sched_barrier(0);
        }
        const double *pc = Ab + (s * P + lq) * TS + lr;
#pragma unroll
        for (int mt = 0; mt < PT; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int k0 = 16 * mt + 4 * i;
            if (k0 >= P) continue;
            const bool in = k0 + 3 < P || k0 + lq < P;
            const double a = in ? t2[mt][i] : 0.0;
#pragma unroll
            for (int n2 = 0; n2 < PT; ++n2)
              t3[nt][n2] = mfma16(a, in ? pc[k0 * TS + 16 * n2] : 0.0, t3[nt][n2]);
            if (PT > 1 && i % 2) __builtin_amdgcn_sched_barrier(0);
          }
      }
    }
    wave_lds_order();  // every lane's T1 reads precede the T3 writes below
#pragma unroll
    for (int nt = 0; nt < PT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * nt + 4 * r + lq;  // (lk, wbk)
        if (16 * nt + 4 * r >= P) continue;
#pragma unroll
        for (int n2 = 0; n2 < PT; ++n2) {
          const int n = 16 * n2 + lr;  // (lb, wbb)
          if (m < P && n < P)
            Tp[((m % D) * D + n % D) * TS + (m / D) * D + n / D] = t3[nt][n2][r];
        }
      }
    wave_lds_order();
    // T3 of the pair to HBM as T3[yf][l][xb][wb]
#pragma unroll
    for (int u = 0; u < (P * P + 63) / 64; ++u) {
      const int i = lane + 64 * u, wb = i % P, l = i / P;
      if (i < P * P)
        buf_st_t<double>(t3rs, (unsigned)(((yf * P + l) * K + xb) * P + wb) * 8u, Tp[wb * TS + l]);
    }
    // (e) this pair's contribution to Yt[l][yb]: k = wb
    if (v.do_local) {
      const double *pa = Tp + lq * TS + lr, *pb = Gs + (tx * P + lq) * GS + lr;
#pragma unroll
      for (int ks = 0; ks < PK; ++ks) {
        const bool in = 4 * ks + 3 < P || 4 * ks + lq < P;
        double a[PT];
#pragma unroll
        for (int mt = 0; mt < PT; ++mt) a[mt] = in ? pa[4 * ks * TS + 16 * mt] : 0.0;
#pragma unroll
        for (int q = 0; q < NE; ++q) {
          if (16 * q >= nyb) break;
          const double b = in ? pb[4 * ks * GS + 16 * q] : 0.0;
#pragma unroll
          for (int mt = 0; mt < PT; ++mt) accE[mt][q] = mfma16(a[mt], b, accE[mt][q]);
        }
        if (PT > 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (!v.do_local) return;
  if constexpr (TX > 1) {  // sum the TX partials of each yf in a fixed order
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < PT; ++mt)
#pragma unroll
      for (int q = 0; q < NE; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sm_raw[(((wave * PT + mt) * NE + q) * 4 + r) * 64 + lane] = accE[mt][q][r];
    __syncthreads();
    if (tx != 0) return;
#pragma unroll
    for (int mt = 0; mt < PT; ++mt)
#pragma unroll
      for (int q = 0; q < NE; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int o = 1; o < TX; ++o)
            accE[mt][q][r] += sm_raw[((((wave + o) * PT + mt) * NE + q) * 4 + r) * 64 + lane];
  }
  if (yf >= K) return;
#pragma unroll
  for (int mt = 0; mt < PT; ++mt)
#pragma unroll
    for (int q = 0; q < NE; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = 16 * mt + 4 * r + lq, yb = 16 * q + lr;
        if (l < P && yb < K)
          gmem(Yout)[rl ? ((size_t)yb * P + l) * K + yf : ((size_t)yf * P + l) * K + yb] =
              accE[mt][q][r];
      }
}

// Y = the sum of the nsplit partial Yt of each item, in order.
__global__ __launch_bounds__(kThreads) void k_sum_parts(Ptr Y, const double *part,
                                                        size_t part_stride, int nsplit, size_t n) {
  const int it = blockIdx.y;
  const auto *p = gmem(part) + (size_t)it * part_stride;
  auto *y = gmem(Y.at(it));
  const size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x;
  if (i >= n) return;
  double t = p[i];
#pragma unroll 4
  for (int k = 1; k < nsplit; ++k) t += p[(size_t)k * n + i];
  y[i] = t;
}

// ---------------------------------------------------------------------------
// Householder QR (LAPACK conventions: dlarfg reflectors, dorg2r formation).
// One workgroup per item; the true panel (rows r = r1*n2 + r2, columns c at
// base[r1*s1 + r2*s2 + c*sc]) is copied column-major into LDS, factorised,
// and Q written back in place (panels too large for LDS: k_qrg below).
// ---------------------------------------------------------------------------
// x / n and x % n for 0 <= x < 2^22 and 1 <= n < 2^22 through one FP32
// multiply: x and 1/n are within one rounding of exact, so the truncated
// product is the quotient or one off, and the remainder's sign and size
// correct it.  Replaces an integer division (a few dozen VALU operations)
// in the panel copies.
struct DivN {
  int n;
  float inv;
  __device__ explicit DivN(int n_) : n(n_), inv(1.0f / (float)n_) {}
  __device__ __forceinline__ int quot(int x) const {
    int q = (int)((float)x * inv);
    const int r = x - q * n;
    if (r < 0) --q;
    else if (r >= n) ++q;
    return q;
  }
};

struct QrArgs {
  FitDims *dims;
  int W, c, j, mode, K, P;
  Ptr Y;
  double *rbuf;
  double *scratch;
  size_t scratch_stride;
  const int32_t *flag;
  int want_r;
};

constexpr int kQrLds = 19968;  // doubles (156 KB of the 160 KB LDS)

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ __launch_bounds__(kThreads) void k_qr(QrArgs q) {
  const int it = blockIdx.x;
  if (q.flag && !q.flag[it]) return;
  const FitDims &dm = q.dims[(size_t)it * q.W + q.c];
  const int K = q.K, P = q.P, j = q.j;
  int n1, n2, ncol;
  size_t s1, s2, sc;
  switch (q.mode) {
    case LR_INNER:
      n1 = dm.bl[j]; s1 = (size_t)P * K; n2 = P; s2 = K; ncol = dm.br[j]; sc = 1;
      break;
    case RL_INNER:  // rows (l, yb), l-major, as in the QR of the transpose
      n1 = P; s1 = K; n2 = dm.br[j]; s2 = 1; ncol = dm.bl[j]; sc = (size_t)P * K;
      break;
    case LR_TOP:
      n1 = dm.p[j]; s1 = K; n2 = 1; s2 = 0; ncol = dm.br[j]; sc = 1;
      break;
    default:  // RL_BOT
      n1 = dm.p[j]; s1 = 1; n2 = 1; s2 = 0; ncol = dm.bl[j]; sc = K;
      break;
  }
  const int m = n1 * n2, n = ncol;
  double *base = q.Y.at(it);
  __shared__ double lds[kQrLds];
  __shared__ double red[8];
  __shared__ double tau_s[128];
  double *A = lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  const DivN divm(m), dn2(n2);
  for (int idx = tid; idx < m * n; idx += kThreads) {
    const int col = divm.quot(idx), r = idx - col * m;
    const int r1 = dn2.quot(r), r2 = r - r1 * n2;
    A[idx] = base[r1 * s1 + r2 * s2 + col * sc];
  }
  __syncthreads();

  for (int k = 0; k < n; ++k) {
    double *v = A + (size_t)k * m;
    double part = 0.0;
    for (int i = k + 1 + tid; i < m; i += kThreads) part += v[i] * v[i];
    part = wave_sum(part);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    if (tid == 0) {
      const double sigma2 = red[0] + red[1] + red[2] + red[3];
      const double alpha = v[k];
      double tau = 0.0, scal = 0.0, beta = alpha;
      if (sigma2 > 0.0) {
        const double nrm = sqrt(alpha * alpha + sigma2);
        beta = alpha >= 0.0 ? -nrm : nrm;
        tau = (beta - alpha) / beta;
        scal = 1.0 / (alpha - beta);
      }
      tau_s[k] = tau;
      red[4] = scal;
      v[k] = beta;
    }
    __syncthreads();
    const double scal = red[4], tau = tau_s[k];
    if (tau != 0.0)
      for (int i = k + 1 + tid; i < m; i += kThreads) v[i] *= scal;
    __syncthreads();
    if (tau != 0.0) {
      for (int jj = k + 1 + wave; jj < n; jj += kThreads / 64) {
        double *a = A + (size_t)jj * m;
        double w = 0.0;
        for (int i = k + 1 + lane; i < m; i += 64) w += v[i] * a[i];
        w = wave_sum(w) + a[k];
        w *= tau;
        if (lane == 0) a[k] -= w;
        for (int i = k + 1 + lane; i < m; i += 64) a[i] -= v[i] * w;
      }
    }
    __syncthreads();
  }

  if (q.want_r) {
    double *R = q.rbuf + (size_t)it * K * K;
    for (int idx = tid; idx < K * K; idx += kThreads) {
      const int r = idx / K, cc = idx - r * K;
      R[idx] = (r < n && cc < n && r <= cc) ? A[(size_t)cc * m + r] : 0.0;
    }
  }
  __syncthreads();

  // Q = H_0 ... H_{n-1} [I; 0], formed in place from the last reflector.
  for (int k = n - 1; k >= 0; --k) {
    double *v = A + (size_t)k * m;
    const double tau = tau_s[k];
    if (k < n - 1 && tau != 0.0) {
      for (int jj = k + 1 + wave; jj < n; jj += kThreads / 64) {
        double *a = A + (size_t)jj * m;
        double w = 0.0;
        for (int i = k + 1 + lane; i < m; i += 64) w += v[i] * a[i];
        w = wave_sum(w) + a[k];
        w *= tau;
        if (lane == 0) a[k] -= w;
        for (int i = k + 1 + lane; i < m; i += 64) a[i] -= v[i] * w;
      }
    }
    __syncthreads();
    for (int i = tid; i < m; i += kThreads) {
      if (i > k) v[i] *= -tau;
      else if (i == k) v[i] = 1.0 - tau;
      else v[i] = 0.0;
    }
    __syncthreads();
  }

  for (int idx = tid; idx < m * n; idx += kThreads) {
    const int col = divm.quot(idx), r = idx - col * m;
    const int r1 = dn2.quot(r), r2 = r - r1 * n2;
    base[r1 * s1 + r2 * s2 + col * sc] = A[idx];
  }
}

// ---------------------------------------------------------------------------
// The same Householder QR for tall panels kept in a global scratch (D = 6
// and larger bonds): one workgroup of 16 waves per item.  Each reflector is
// staged in LDS once (read in place where a panel has more than kQrgRows
// rows), and a wave updates up to kQrgCols trailing columns in
// one pass over the rows (one dot product and one axpy per column, the
// columns' loads interleaved), so the trailing matrix is read twice and
// written once per reflector.  Reflectors, their order and the formation of
// Q are those of the kernel above.
// ---------------------------------------------------------------------------
constexpr int kQrgThreads = 1024;
constexpr int kQrgWaves = kQrgThreads / 64;
constexpr int kQrgRows = 8192;  // rows of the staged reflector (64 KB of LDS)
constexpr int kQrgCols = 8;     // trailing columns per wave and pass (n <= 128)

// a_c -= tau v (a_kc + v^T a_c) for the columns c = c0, c0 + kQrgWaves, ...
// (< n) of this wave; v = (1, vs[k+1..m-1]).  Rows go kQrgUnroll at a time
// per lane, their loads issued together (the panel streams from L2).
constexpr int kQrgUnroll = 2;
__device__ __forceinline__ void qrg_apply(double *A, const double *vs, int m, int n, int k,
                                          double tau, int c0, int lane) {
  double *a[kQrgCols];
  double w[kQrgCols];
  int nc = 0;
#pragma unroll
  for (int u = 0; u < kQrgCols; ++u) {
    const int c = c0 + u * kQrgWaves;
    a[u] = A + (size_t)(c < n ? c : k) * m;
    w[u] = 0.0;
    if (c < n) nc = u + 1;
  }
  if (nc == 0) return;
  for (int i0 = k + 1 + lane; i0 < m; i0 += 64 * kQrgUnroll) {
    double v[kQrgUnroll], x[kQrgUnroll][kQrgCols];
#pragma unroll
    for (int r = 0; r < kQrgUnroll; ++r) {
      const int i = i0 + 64 * r;
      v[r] = i < m ? vs[i] : 0.0;
#pragma unroll
      for (int u = 0; u < kQrgCols; ++u) x[r][u] = (u < nc && i < m) ? a[u][i] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < kQrgUnroll; ++r)
#pragma unroll
      for (int u = 0; u < kQrgCols; ++u) w[u] = fma(v[r], x[r][u], w[u]);
  }
#pragma unroll
  for (int u = 0; u < kQrgCols; ++u) {
    if (u >= nc) break;
    w[u] = tau * (wave_sum(w[u]) + a[u][k]);
  }
  if (lane == 0) {
#pragma unroll
    for (int u = 0; u < kQrgCols; ++u)
      if (u < nc) a[u][k] -= w[u];
  }
  for (int i0 = k + 1 + lane; i0 < m; i0 += 64 * kQrgUnroll) {
    double v[kQrgUnroll], x[kQrgUnroll][kQrgCols];
#pragma unroll
    for (int r = 0; r < kQrgUnroll; ++r) {
      const int i = i0 + 64 * r;
      v[r] = i < m ? vs[i] : 0.0;
#pragma unroll
      for (int u = 0; u < kQrgCols; ++u) x[r][u] = (u < nc && i < m) ? a[u][i] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < kQrgUnroll; ++r) {
      const int i = i0 + 64 * r;
      if (i >= m) break;
#pragma unroll
      for (int u = 0; u < kQrgCols; ++u)
        if (u < nc) a[u][i] = x[r][u] - v[r] * w[u];
    }
  }
}

// Copies between the strided panel and the column-major scratch, eight
// elements in flight per thread.
template <bool kIn>
__device__ __forceinline__ void qrg_copy(double *A, double *base, int m, int n, int n2,
                                         size_t s1, size_t s2, size_t sc, int tid) {
  constexpr int U = 8;
  const int total = m * n;
  const DivN divm(m), dn2(n2);
  for (int i0 = tid; i0 < total; i0 += kQrgThreads * U) {
    double x[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int idx = i0 + r * kQrgThreads;
      const int col = divm.quot(idx), row = idx - col * m;
      const int r1 = dn2.quot(row), r2 = row - r1 * n2;
      const size_t g = r1 * s1 + r2 * s2 + col * sc;
      x[r] = idx < total ? (kIn ? base[g] : A[idx]) : 0.0;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int idx = i0 + r * kQrgThreads;
      if (idx >= total) break;
      const int col = divm.quot(idx), row = idx - col * m;
      const int r1 = dn2.quot(row), r2 = row - r1 * n2;
      const size_t g = r1 * s1 + r2 * s2 + col * sc;
      if (kIn) A[idx] = x[r];
      else base[g] = x[r];
    }
  }
}

__global__ __launch_bounds__(kQrgThreads) void k_qrg(QrArgs q) {
  const int it = blockIdx.x;
  if (q.flag && !q.flag[it]) return;
  const FitDims &dm = q.dims[(size_t)it * q.W + q.c];
  const int K = q.K, P = q.P, j = q.j;
  int n1, n2, ncol;
  size_t s1, s2, sc;
  switch (q.mode) {
    case LR_INNER:
      n1 = dm.bl[j]; s1 = (size_t)P * K; n2 = P; s2 = K; ncol = dm.br[j]; sc = 1;
      break;
    case RL_INNER:  // rows (l, yb), l-major, as in the QR of the transpose
      n1 = P; s1 = K; n2 = dm.br[j]; s2 = 1; ncol = dm.bl[j]; sc = (size_t)P * K;
      break;
    case LR_TOP:
      n1 = dm.p[j]; s1 = K; n2 = 1; s2 = 0; ncol = dm.br[j]; sc = 1;
      break;
    default:  // RL_BOT
      n1 = dm.p[j]; s1 = 1; n2 = 1; s2 = 0; ncol = dm.bl[j]; sc = K;
      break;
  }
  const int m = n1 * n2, n = ncol;
  double *base = q.Y.at(it);
  __shared__ double vs[kQrgRows];
  __shared__ double red[kQrgWaves];
  __shared__ double tau_s[128];
  __shared__ double scal_s;
  double *A = q.scratch + (size_t)it * q.scratch_stride;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool stage = m <= kQrgRows;

  qrg_copy<true>(A, base, m, n, n2, s1, s2, sc, tid);
  __syncthreads();

  for (int k = 0; k < n; ++k) {
    double *v = A + (size_t)k * m;
    double part = 0.0;
    for (int i = k + 1 + tid; i < m; i += kQrgThreads) part = fma(v[i], v[i], part);
    part = wave_sum(part);
    if (lane == 0) red[wave] = part;
    __syncthreads();
    if (tid == 0) {  // dlarfg
      double sigma2 = 0.0;
      for (int w = 0; w < kQrgWaves; ++w) sigma2 += red[w];
      const double alpha = v[k];
      double tau = 0.0, scal = 0.0, beta = alpha;
      if (sigma2 > 0.0) {
        const double nrm = sqrt(alpha * alpha + sigma2);
        beta = alpha >= 0.0 ? -nrm : nrm;
        tau = (beta - alpha) / beta;
        scal = 1.0 / (alpha - beta);
      }
      tau_s[k] = tau;
      scal_s = scal;
      v[k] = beta;
    }
    __syncthreads();
    const double tau = tau_s[k];
    if (tau != 0.0) {
      const double scal = scal_s;
      for (int i = k + 1 + tid; i < m; i += kQrgThreads) {
        const double x = v[i] * scal;
        v[i] = x;
        if (stage) vs[i] = x;
      }
      __syncthreads();
      qrg_apply(A, stage ? vs : v, m, n, k, tau, k + 1 + wave, lane);
    }
    __syncthreads();
  }

  if (q.want_r) {
    double *R = q.rbuf + (size_t)it * K * K;
    for (int idx = tid; idx < K * K; idx += kQrgThreads) {
      const int r = idx / K, cc = idx - r * K;
      R[idx] = (r < n && cc < n && r <= cc) ? A[(size_t)cc * m + r] : 0.0;
    }
  }
  __syncthreads();

  // Q = H_0 ... H_{n-1} [I; 0], formed in place from the last reflector.
  for (int k = n - 1; k >= 0; --k) {
    double *v = A + (size_t)k * m;
    const double tau = tau_s[k];
    if (stage)
      for (int i = k + 1 + tid; i < m; i += kQrgThreads) vs[i] = v[i];
    __syncthreads();
    if (k < n - 1 && tau != 0.0) qrg_apply(A, stage ? vs : v, m, n, k, tau, k + 1 + wave, lane);
    if (!stage) __syncthreads();  // column k is read in place by the update
    for (int i = tid; i < m; i += kQrgThreads) {
      if (i > k) v[i] = -tau * (stage ? vs[i] : v[i]);
      else if (i == k) v[i] = 1.0 - tau;
      else v[i] = 0.0;
    }
    __syncthreads();
  }

  qrg_copy<false>(A, base, m, n, n2, s1, s2, sc, tid);
}

// ---------------------------------------------------------------------------
// Blocked Householder QR on FP64 MFMA tiles, workgroups of NW waves.  A column
// tile (16 columns, up to 16 NW RT rows) stays in registers as 16x16 tiles in
// the MFMA accumulator layout (register s of lane (lr, lc) holds row 4s + lr,
// column lc of its tile); wave w owns row tiles w, w + NW, ....  Columns are
// factorised in blocks of 16 as in dgeqrf (qm_factor below), and the block
// reflector I - V T V^T (T from dlarft) is applied to the columns on the
// right on MFMA (W = V^T A, A -= V T^T W).  Q is formed backwards over the
// blocks as in dorgqr: the block reflector updates the columns on the right,
// and the block's own columns are E - V (T V_top^T), E the unit columns.  The
// reflectors are those of the unblocked algorithm (dgeqr2); only the rounding
// order of sums and updates differs.  Cross-wave sums are taken in a fixed
// order that every wave repeats, so all waves hold the same bits.
//
// Two kernels use it: k_qrm holds a whole panel in one workgroup, k_qrb one
// column tile per workgroup, a launch per block.
// ---------------------------------------------------------------------------

// V column c of the block starts at c * VS + (c & 14) doubles: with the column
// stride VS = 16 (mod 32) and that shift, both the per-lane column walk (lane
// (lr, lc) reads column lc, rows 4s + lr) and the MFMA operand read (column
// 4kk + lr, row lc) touch 32 distinct banks per half-wave, and the per-lane
// part of every address stays a base plus compile-time offsets.
template <int VS>
__device__ __forceinline__ int qm_col(int c) { return c * VS + (c & 14); }

// Sum over the four 16-lane rows: the 4x4x4 MFMA multiplies a matrix of ones
// (row index: the lane row of the result) by x (k: the lane row), so the same
// bits land in every row after one instruction (35 cycles) instead of two
// rounds of permlane swaps (70 cycles, 14 instructions).  Needs all 64 lanes
// active.
__device__ __forceinline__ double sum_rows4(double x) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, x, 0.0, 0, 0, 0);
}

__device__ __forceinline__ int cl_index(int i, int j) {  // accumulator slot of (i, j)
  return (i >> 2) * 64 + (i & 3) * 16 + j;
}

// x of lane SRC of the same 16-lane row (64-bit row_newbcast)
template <int SRC>
__device__ __forceinline__ double row_bcast(double x) {
  return __longlong_as_double(
      __builtin_amdgcn_mov_dpp(__double_as_longlong(x), 0x150 + SRC, 0xf, 0xf, true));
}

// p[s] += x[s] bcast(x[s]) and x[s] += bcast(x[s]) c for the four registers of
// a tile, bcast the value of lane SRC of the 16-lane row: FMAs that take it
// as their DPP operand.  Broadcasts of their own (which the compiler does not
// fold into the FMA) double a column step's FP64 instructions.  s_nop 1 covers
// the two wait states between a VALU write of x and its DPP read.
// The results are early-clobber operands: later instructions of a block still
// read inputs, which may not share a register with an earlier result.
template <int SRC>
__device__ __forceinline__ void dot_bcast(double (&p)[4], const v4d &x) {
  asm volatile(
      "s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %4, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %6, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %7, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
      : "+&v"(p[0]), "+&v"(p[1]), "+&v"(p[2]), "+&v"(p[3])
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "n"(SRC));
}
// x[s] += y_s bcast(g), bcast the value of lanes Q + s of the 16-lane row
template <int Q>
__device__ __forceinline__ void fma_bcast4(double (&x)[4], double y0, double y1, double y2,
                                           double y3, double g) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %8, %4 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %8, %5 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %8, %6 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %8, %7 row_newbcast:%12 row_mask:0xf bank_mask:0xf"
      : "+&v"(x[0]), "+&v"(x[1]), "+&v"(x[2]), "+&v"(x[3])
      : "v"(y0), "v"(y1), "v"(y2), "v"(y3), "v"(g), "n"(Q), "n"(Q + 1), "n"(Q + 2), "n"(Q + 3));
}
template <int SRC>
__device__ __forceinline__ void axpy_bcast(v4d &x, double c) {
  double x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
  asm volatile(
      "s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %1, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
      : "+&v"(x0), "+&v"(x1), "+&v"(x2), "+&v"(x3)
      : "v"(c), "n"(SRC));
  x = v4d{x0, x1, x2, x3};
}

// dlarfg's scalars from alpha and sigma^2 > 0: nrm = sqrt(alpha^2 + sigma^2),
// beta = -sign(alpha) nrm, tau = (beta - alpha) / beta, scal = 1 / (alpha -
// beta).  The hardware's reciprocal square root and reciprocal (relative error
// 2^-24) start a third-order step each (their error cubed, below FP64
// rounding), and one residual correction rounds the result: over 2^21 random
// pairs at each of several scales beta is the square root's and tau and scal
// are the divisions' results bit for bit, from alpha^2 + sigma^2 of 2^-970 up to
// overflow (below, the square root's residual underflows and beta is off by up
// to 2 ulp; tau and scal are still those of that beta).  Panels whose columns
// depend on each other rely on exact values (tau = 2 where sigma vanishes beside
// alpha).  The compiler's square root and two divisions are a chain of 270
// cycles on the factorisation's critical path, this one of about 130.
struct Reflector {
  double tau, scal, beta;
};
__device__ __forceinline__ Reflector make_reflector(double alpha, double sigma2) {
  Reflector h{0.0, 0.0, alpha};
  if (!(sigma2 > 0.0)) return h;
  const double s2 = fma(alpha, alpha, sigma2);
  const double y0 = __builtin_amdgcn_rsq(s2);
  const double e = fma(-(s2 * y0), y0, 1.0);
  const double y = fma(y0 * e, fma(e, 0.375, 0.5), y0);
  double nrm = s2 * y;
  nrm = fma(fma(-nrm, nrm, s2), 0.5 * y, nrm);
  h.beta = alpha >= 0.0 ? -nrm : nrm;
  const double u = alpha - h.beta;
  const double r0 = __builtin_amdgcn_rcp(u);
  const double g = fma(-u, r0, 1.0);
  const double r1 = fma(r0, fma(g, g, g), r0);
  h.scal = fma(r1, fma(-u, r1, 1.0), r1);
  // tau = |u| / nrm, with 1 / nrm from y
  const double yn = fma(y, fma(-nrm, y, 1.0), y), ua = fabs(u);
  const double t = ua * yn;
  h.tau = fma(fma(-t, nrm, ua), yn, t);
  return h;
}

// LDS of one block's factorisation.  wp holds the waves' partial sums per
// column, the NW partials of a column side by side (row stride NW + 2: 16
// lanes write 16 columns without a bank conflict, and a lane reads NW / 4
// partials as one run).
template <int NW>
struct QmShared {
  double wp[2][NW > 1 ? 16 : 1][NW + 2], wq[2][16];
  double G[16][16];   // G[k][c] = v_c^T v_k, c < k
  double T[16][17];   // dlarft's T
};

// Sum of the waves' 16x16 accumulators into Ws (accumulator slots).
template <int NW>
__device__ __forceinline__ void qm_reduce(const v4d &acc, double (*wred)[256], double *Ws,
                                          int tid = threadIdx.x) {
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int r = 0; r < 4; ++r) wred[wave][r * 64 + lane] = acc[r];
  __syncthreads();
  if (tid < 256) {
    double x = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) x += wred[w][tid];
    Ws[tid] = x;
  }
  __syncthreads();
}

// Factorises a column tile: columns b0 .. b0 + nbb - 1 of the panel, b0 = 16 b
// (b < NW, so that the diagonal lies in row tile t = 0 of wave b), reflectors
// scaled in place below the diagonal, beta on it, T in sh.T (visible to the
// calling workgroup after its next barrier).
//
// Step k broadcasts column k along each 16-lane row and forms, in one pass
// and one cross-wave sum, x^T a_c for every column c (x = column k below the
// diagonal); the row-k entries a_kc travel beside them.  Column k's own sum
// and entry give dlarfg; w_c = a_kc + scal x^T a_c gives dlarf's update of
// the later columns, and for the earlier ones (their reflectors, not yet
// scaled) the entry v_c^T v_k = scal_c w_c of V^T V that T is made from, so
// no pass over V is spent on it.  A block with a zero reflector (a column that
// vanishes below its diagonal) takes V^T V from the scaled V instead: such
// panels have rows or columns that are exactly zero (single-layer networks,
// trivial legs), which Q keeps only where T agrees with V bit for bit; the
// leftovers of 1e-16 would otherwise be normalised to full columns by the next
// site's factorisation.  Columns that vanish only to rounding level are not
// covered: what such a fit converges to depends on rounding with either form of
// T, as it does in LAPACK.
//
// Bound by the instructions of a step, about 100 of them beside the tiles'
// own, which every wave issues for itself, and by their dependent chain (one
// barrier, two sums over the row groups, dlarfg).  After the barrier a lane
// reads the partials of NW / 4 waves and one MFMA adds the row groups' sums.
// Broadcasts folded into the tiles' FMAs, rows of R taken out of the tile
// instead of masked in each step, those sums on MFMA and T from registers took
// a 16-column block of 512 rows from 34900 to 28900 cycles.  A panel of one
// wave (NW = 1) needs neither LDS nor a barrier in a step.
template <int NW, int RT>
__device__ __forceinline__ void qm_factor(v4d (&a)[RT], int b, int nbb, QmShared<NW> &sh,
                                          double (*wred)[256], double *Ws,
                                          int tid = threadIdx.x) {
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15, b0 = 16 * b;
  double my_scal = 0.0, my_beta = 0.0, my_tau = 0.0;  // of column b0 + lc
  // The tiles may come from MFMAs, whose results the FMAs written as assembly
  // must not read for 19 wait states.  (Register by register: a tile as one
  // operand made the allocator keep a copy of each, 18 tiles then spilled.)
#pragma unroll
  for (int t = RT - 1; t >= 0; --t) {
    double x[4] = {a[t][0], a[t][1], a[t][2], a[t][3]};
    if (t > 0) asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
    else asm volatile("s_nop 15\n\ts_nop 3" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
    a[t] = v4d{x[0], x[1], x[2], x[3]};
  }
  // rows of R leave the tile as they are finished (zero instead, so that no
  // step has to mask them) and come back at the end
  double rsave[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    rsave[s] = a[0][s];
    if (16 * wave < b0) a[0][s] = 0.0;
  }
  static_for<0, 16>([&](auto KC) __attribute__((always_inline)) {
    constexpr int kc = decltype(KC)::value, pb = kc & 1;
    if (kc >= nbb) return;
    // this lane's first row relative to the block's, opaque so that every
    // step compares anew instead of keeping 64 lane masks in scalar registers
    int r0 = 16 * wave + lr - b0;
    asm volatile("" : "+v"(r0));
    const double rk = a[0][kc >> 2];  // in the lanes of row k: a_kc
    const bool in_k = r0 == (kc & 3);
    if (NW > 1 && in_k) sh.wq[pb][lc] = rk;
    if (in_k && lc >= kc) a[0][kc >> 2] = 0.0;
    double pp[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < RT; ++t) dot_bcast<kc>(pp, a[t]);
    const double pdot = sum_rows4((pp[0] + pp[1]) + (pp[2] + pp[3]));
    double pc, qc;
    if constexpr (NW > 1) {
      if (lr == 0) sh.wp[pb][lc][wave] = pdot;
      __syncthreads();
      double part = sh.wp[pb][lc][lr * (NW / 4)];
      qc = sh.wq[pb][lc];
#pragma unroll
      for (int i = 1; i < NW / 4; ++i) part += sh.wp[pb][lc][lr * (NW / 4) + i];
      pc = sum_rows4(part);
    } else {
      pc = pdot;
      qc = sum_rows4(in_k ? rk : 0.0);
    }
    const Reflector h = make_reflector(row_bcast<kc>(qc), row_bcast<kc>(pc));
    const double w = fma(h.scal, pc, qc);
    if (wave == 0 && lr == 0 && lc < kc) sh.G[kc][lc] = my_scal * w;
    if (lc == kc) {
      my_scal = h.scal;
      my_beta = h.beta;
      my_tau = h.tau;
    }
    // dlarf on the block's columns c > k: a_c -= tau v w_c, v = (1, scal x)
    const double wt = (lc > kc && lc < nbb) ? -(h.tau * w) : 0.0;
    const double cs = h.scal * wt;
    if (in_k) rsave[kc >> 2] = qc + wt;
#pragma unroll
    for (int t = 0; t < RT; ++t) axpy_bcast<kc>(a[t], cs);
  });
  asm volatile("s_nop 1");  // before an MFMA reads what they wrote
  // reflectors scaled in place, beta on the diagonal, R above it
  {
    const double f = lc < nbb && my_tau != 0.0 ? my_scal : 1.0;
    const int d0 = 16 * wave + lr - b0 - lc;  // first row minus the column's diagonal
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double x = a[0][s] * (d0 + 4 * s > 0 ? f : 1.0);
      a[0][s] = d0 + 4 * s < 0 ? rsave[s] : d0 + 4 * s == 0 && lc < nbb ? my_beta : x;
    }
#pragma unroll
    for (int t = 1; t < RT; ++t) a[t] *= f;
  }
  if (__ballot(lc < nbb && my_tau == 0.0) != 0) {  // the same in every wave
    v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int d = 16 * (wave + NW * t) + 4 * s + lr - b0 - lc;
        const double x = lc < nbb ? (d > 0 ? a[t][s] : (d == 0 ? 1.0 : 0.0)) : 0.0;
        acc[s & 1] = mfma16(x, x, acc[s & 1]);
      }
    acc[0] += acc[1];
    if constexpr (NW > 1) {
      qm_reduce<NW>(acc[0], wred, Ws, tid);
      if (wave == 0)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[0][s] = Ws[s * 64 + lane];
    }
    if (wave == 0)
#pragma unroll
      for (int s = 0; s < 4; ++s) sh.G[lc][4 * s + lr] = acc[0][s];
  }
  // T as in dlarft (forward, columnwise), by the wave that holds G: lane lc
  // keeps row lc, so that column i is a sum over the lane's own registers with
  // row i of G as DPP broadcasts (4 partial sums by column mod 4).  With a
  // row's columns spread over the lane rows, and so a cross-lane sum and an LDS
  // read in the chain of every column, T took 4700 cycles, a seventh of a
  // block's time.
  if (wave == 0) {
    wave_lds_order();
    double tr[16], g[16];
    static_for<0, 4>([&](auto UC) __attribute__((always_inline)) {
      constexpr int u = 4 * decltype(UC)::value;
#pragma unroll
      for (int i = u; i < u + 4; ++i) tr[i] = g[i] = 0.0;
      if (u >= nbb) return;
#pragma unroll
      for (int i = u; i < u + 4; ++i) g[i] = sh.G[i][lc];
#pragma unroll
      for (int i = u; i < u + 4; ++i) g[i] = lc < i && i < nbb ? g[i] : 0.0;
    });
    tr[0] = lc == 0 ? my_tau : 0.0;
    static_for<1, 16>([&](auto IC) __attribute__((always_inline)) {
      constexpr int i = decltype(IC)::value;
      if (i >= nbb) return;
      const double ti = row_bcast<i>(my_tau);
      double x[4] = {0.0, 0.0, 0.0, 0.0};
      static_for<0, (i + 3) / 4>([&](auto QC) __attribute__((always_inline)) {
        constexpr int q = 4 * decltype(QC)::value;  // columns >= i meet a zero tr
        fma_bcast4<q>(x, tr[q], tr[q + 1], tr[q + 2], tr[q + 3], g[i]);
      });
      const double xs = (x[0] + x[1]) + (x[2] + x[3]);
      tr[i] = lc < i ? -ti * xs : (lc == i ? ti : 0.0);
    });
    if (lr == 0)
#pragma unroll
      for (int k = 0; k < 16; ++k) sh.T[lc][k] = tr[k];
  }
}

// The panel of one item in one visit mode: m true rows, n true columns; entry
// (row, col) at row rs + (row / n2) ex + col cs of the site's slot.  Only a
// right-to-left inner site has a gap (ex) between the runs of its rows (l, y')
// (the physical index major, as in the QR of the transpose).  All offsets
// stay below 2^23 (bond caps <= 128, P <= 64), so 24-bit products form them:
// 64-bit offsets took a fifth of a 512 x 32 panel's instructions.
struct QrPanel {
  int m, n, rs, cs, n2, ex;
  __device__ __forceinline__ int row_off(int row, const DivN &d) const {
    const int o = __mul24(row, rs);
    return ex ? o + __mul24(d.quot(row), ex) : o;
  }
};
__device__ __forceinline__ QrPanel qr_panel(const QrArgs &q, int it) {
  const FitDims &dm = q.dims[(size_t)it * q.W + q.c];
  const int K = q.K, P = q.P, j = q.j;
  QrPanel p;
  p.n2 = 1;
  p.ex = 0;
  switch (q.mode) {
    case LR_INNER:
      p.m = dm.bl[j] * P; p.rs = K; p.n = dm.br[j]; p.cs = 1;
      break;
    case RL_INNER:
      p.m = P * dm.br[j]; p.rs = 1; p.n2 = dm.br[j]; p.ex = K - p.n2; p.n = dm.bl[j];
      p.cs = P * K;
      break;
    case LR_TOP:
      p.m = dm.p[j]; p.rs = K; p.n = dm.br[j]; p.cs = 1;
      break;
    default:  // RL_BOT
      p.m = dm.p[j]; p.rs = 1; p.n = dm.bl[j]; p.cs = K;
      break;
  }
  p.n = min(p.n, p.m);
  return p;
}

// -op(T) W as the update's MFMA B operands (register s: row 4s + lr, column
// lc), every wave for itself: no second pass through LDS.  w(q) is W[q][lc].
template <class F>
__device__ __forceinline__ v4d qm_coeff(const double (*T)[17], bool trans, F &&w, int lr, int lc) {
  v4d z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 4; ++s)
    z = mfma16(trans ? T[4 * s + lr][lc] : T[lc][4 * s + lr], w(4 * s + lr), z);
  return -z;
}

// LDS of a panel's factorisation in one workgroup.
template <int NW, int RT, int CT>
struct QmBuf {
  // a multiple of 32 rows, + 16: the stride is 16 (mod 32)
  static constexpr int VS = (16 * NW * RT + 31) / 32 * 32 + 16;
  double VT[16 * VS];  // V of the current block, column c at qm_col(c)
  double wred[NW][256];
  double Ws[256];
  QmShared<NW> sh[CT];
};

// QR of a panel held in registers by NW waves (the whole workgroup, or with
// NW = 1 its first wave alone): a[ct][t]
// register s of lane (lr, lc) is row 16 (wave + NW t) + 4 s + lr, column 16 ct
// + lc, zero outside the n columns and the true rows.  on_r() is called with R
// on and above a's diagonal; then a becomes Q.
template <int NW, int RT, int CT, class F>
__device__ __forceinline__ void qm_panel(v4d (&a)[CT][RT], int n, QmBuf<NW, RT, CT> &sm,
                                         F &&on_r, int tid = threadIdx.x) {
  static_assert((NW % 4 == 0 && NW >= CT) || (NW == 1 && CT == 1), "panel shape");
  constexpr int VS = QmBuf<NW, RT, CT>::VS;
  auto sync = [&]() __attribute__((always_inline)) {  // of the NW waves
    if constexpr (NW > 1) __syncthreads();
    else wave_lds_order();
  };
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15;
  double *VT = sm.VT, *Ws = sm.Ws;
  // Row tiles t > 0 start at row 16 * NW >= n, below every diagonal entry.
  auto rowof = [&](int t, int s) __attribute__((always_inline)) {
    return 16 * (wave + NW * t) + 4 * s + lr;
  };
  // entry (row of (t, s), b0 + lc) of V: 0 above the diagonal, 1 on it
  auto vent = [&](int b, int nbb, int t, int s) __attribute__((always_inline)) {
    const int row = rowof(t, s), pr = 16 * b + lc;
    return lc < nbb ? ((t > 0 || row > pr) ? a[b][t][s] : (row == pr ? 1.0 : 0.0)) : 0.0;
  };
  auto store_v = [&](int b, int nbb) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) VT[qm_col<VS>(lc) + rowof(t, s)] = vent(b, nbb, t, s);
    wave_lds_order();
  };
  // C += V z for a column tile, K = 16 (MFMA)
  auto update_tile = [&](v4d (&c)[RT], const v4d &z) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        c[t] = mfma16(VT[qm_col<VS>(4 * kk + lr) + 16 * (wave + NW * t) + lc], z[kk], c[t]);
  };
  // C -= V op(T) (V^T C) for the column tiles right of block b.
  auto apply_block = [&](int b, int nbb, bool trans) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      if (ct <= b || 16 * ct >= n) continue;
      v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[s & 1] = mfma16(vent(b, nbb, t, s), a[ct][t][s], acc[s & 1]);
      qm_reduce<NW>(acc[0] + acc[1], sm.wred, Ws, tid);  // W = V^T C
      update_tile(a[ct], qm_coeff(sm.sh[b].T, trans, [&](int q) { return Ws[cl_index(q, lc)]; }, lr, lc));
    }
  };

  // ---- factorisation (dgeqrf order) ----
  static_for<0, CT>([&](auto B) __attribute__((always_inline)) {
    constexpr int b = decltype(B)::value;
    if (16 * b >= n) return;
    const int nbb = min(16, n - 16 * b);
    qm_factor<NW, RT>(a[b], b, nbb, sm.sh[b], sm.wred, Ws, tid);
    if (b + 1 < CT && 16 * (b + 1) < n) {
      store_v(b, nbb);
      apply_block(b, nbb, true);
    }
  });

  on_r();

  // ---- Q = H_0 ... H_{n-1} [I; 0], backwards over the blocks (dorgqr) ----
  static_for<0, CT>([&](auto B) __attribute__((always_inline)) {
    constexpr int b = CT - 1 - decltype(B)::value, b0 = 16 * b;
    if (b0 >= n) return;
    const int nbb = min(16, n - b0);
    sync();  // the previous block's V is no longer read
    store_v(b, nbb);
    apply_block(b, nbb, false);
    sync();  // V of every wave (and T) visible
    // the block's own columns: E - V (T V_top^T), E the unit columns at rows b0..
    const v4d z = qm_coeff(sm.sh[b].T, false, [&](int q) { return VT[qm_col<VS>(q) + b0 + lc]; }, lr, lc);
    v4d c[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        c[t][s] = (t == 0 && rowof(0, s) == b0 + lc && lc < nbb) ? 1.0 : 0.0;
    update_tile(c, z);
#pragma unroll
    for (int t = 0; t < RT; ++t) a[b][t] = c[t];
  });
}

// Calls f(ct, t, s, byte offset) for every entry a lane holds, entries outside
// the panel at byte offset `out`.  Without a gap between the runs of rows the
// offsets are linear in the row and every entry costs four instructions; the
// gap's division, decided per entry, made them fifteen, 5000 cycles of a 512 x
// 32 panel's 92000.
template <int NW, int RT, int CT, class F>
__device__ __forceinline__ void qr_entries(const QrPanel &p, unsigned out, F &&f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane >> 4, lc = lane & 15, r0 = 16 * wave + lr;
  int lim[CT];  // row 16 NW t + 4 s + r0 of column tile ct is real below this
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) lim[ct] = 16 * ct + lc < p.n ? p.m - r0 : 0;
  const unsigned col = (unsigned)__mul24(lc, p.cs);
  if (p.ex == 0) {
    const unsigned o0 = (col + (unsigned)__mul24(r0, p.rs)) * 8u;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int c = 16 * NW * t + 4 * s;
        const unsigned o = o0 + (unsigned)(c * p.rs) * 8u;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          f(ct, t, s, c < lim[ct] ? o + (unsigned)(16 * ct * p.cs) * 8u : out);
      }
  } else {
    const DivN d(p.n2);
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int c = 16 * NW * t + 4 * s, row = c + r0;
        const unsigned o =
            (col + (unsigned)(__mul24(row, p.rs) + __mul24(d.quot(row), p.ex))) * 8u;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          f(ct, t, s, c < lim[ct] ? o + (unsigned)(16 * ct * p.cs) * 8u : out);
      }
  }
}

// One workgroup per panel of up to 16 NW RT rows and 16 CT columns.  Bound by
// the chain of column steps: one 512 x 32 panel 42.6 us at first, 34.8 with
// V^T V from the steps' sums and 24-bit offsets, 32.2 now; 768 x 48 (four to
// sixty-four of them) 120, 91, 71 us; 135 x 15 14.7, 12.0, 10.1 us (kernel
// trace).
template <int NW, int RT, int CT>
__global__ __launch_bounds__(NW * 64) void k_qrm(QrArgs q) {
  const int it = blockIdx.x;
  if (q.flag && !q.flag[it]) return;
  const QrPanel pn = qr_panel(q, it);
  const int K = q.K, n = pn.n;
  double *base = q.Y.at(it);
  __shared__ QmBuf<NW, RT, CT> sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane >> 4, lc = lane & 15;
  auto rowof = [&](int t, int s) { return 16 * (wave + NW * t) + 4 * s + lr; };

  // entries outside the panel load past the descriptor's end and read zero
  const unsigned ybytes = (unsigned)(K * q.P * K) * 8u;
  const __amdgpu_buffer_rsrc_t yrs = buf_rsrc(base, ybytes);
  v4d a[CT][RT];
  qr_entries<NW, RT, CT>(pn, ybytes, [&](int ct, int t, int s, unsigned o) __attribute__((
      always_inline)) { a[ct][t][s] = buf_ld(yrs, o); });

  qm_panel<NW, RT, CT>(a, n, sm, [&]() __attribute__((always_inline)) {
    if (!q.want_r) return;
    double *Rm = q.rbuf + (size_t)it * K * K;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int row = rowof(t, s), col = 16 * ct + lc;
          if (row < K && col < K)
            Rm[(size_t)row * K + col] =
                (t == 0 && row < n && col < n && col >= row) ? a[ct][0][s] : 0.0;
        }
  });

  // The store's offsets and masks are computed anew (opaque sizes) instead of
  // kept in registers from the load; a masked entry's store is dropped at the
  // descriptor's end.
  QrPanel po = pn;
  for (int *v : {&po.m, &po.n, &po.rs, &po.cs, &po.ex}) {
    *v = __builtin_amdgcn_readfirstlane(*v);
    asm volatile("" : "+s"(*v));
  }
  qr_entries<NW, RT, CT>(po, ybytes, [&](int ct, int t, int s, unsigned o) __attribute__((
      always_inline)) { buf_st_t<double>(yrs, o, a[ct][t][s]); });
}

// ---------------------------------------------------------------------------
// The same blocked QR with one column tile per workgroup, for panels that do
// not fit one workgroup's registers (D = 6: 2304 x 64; D = 4 above bond cap
// 48), a launch per block of 16 columns.  Launch b (k_qrb_factor): the
// workgroup of column tile c >= b applies block b - 1 to its tile, and the one
// of tile b then factorises it; the last launch (k_qrb_q) forms Q, the
// workgroup of tile c applying blocks c, c - 1, .. 0 to the unit columns, all
// tiles side by side.  Tiles pass between the launches through a global
// scratch in the accumulator layout (512 contiguous bytes per register), the
// reflectors in their own tile as in dgeqrf, T beside them; each workgroup
// reads a block's V twice (its products need it in both operand layouts, the
// second turned in LDS by the wave that owns the rows).
//
// Bound by the chain: 64 column steps of about 1 us (the VALU work of 2304
// rows on one CU), then one block application per launch.  One 2304 x 64
// panel takes 4 launches of 32 us and 43 us for Q, 171 us together; k_qrg, a
// 16-wave workgroup per panel that streams the trailing panel from L2 once
// for the dots and once for the update of every column, takes 2739 us, bound
// by one CU's L2 port.
// ---------------------------------------------------------------------------
constexpr int kQrbWaves = 8;
// scratch doubles of one panel: CT tiles of MT row tiles, then CT T factors
__host__ __device__ constexpr size_t qrb_words(int K, int P) {
  const size_t ct = (K + 15) / 16, mt = ((size_t)K * P + 15) / 16;
  return ct * (mt + 1) * 256;
}

struct QrbArgs {
  QrArgs q;
  int b;   // block of this launch
  int CT;  // column tiles of the bond cap
  int MT;  // row tiles of the bond cap
};

template <int RT>
struct QrbTile {
  static constexpr int NW = kQrbWaves;
  int wave, lane, lr, lc, mt;  // mt: row tiles of the true panel
  __device__ __forceinline__ QrbTile(int m) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lr = lane >> 4;
    lc = lane & 15;
    mt = (m + 15) / 16;
  }
  __device__ __forceinline__ int rtile(int t) const { return wave + NW * t; }
  __device__ __forceinline__ bool has(int t) const { return rtile(t) < mt; }
  // V of block b in row tile t: 0 above the diagonal, 1 on it
  __device__ __forceinline__ void load_v(const double *scr, int b, int nbb, int MT, int t,
                                         double (&v)[4]) const {
    const auto *p = gmem(scr) + ((size_t)b * MT + rtile(t)) * 256 + lane;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      v[s] = p[s * 64];
      if (t == 0) {  // the only row tiles that reach the diagonal
        const int d = 16 * (wave - b) + 4 * s + lr - lc;
        v[s] = d > 0 ? v[s] : (d == 0 ? 1.0 : 0.0);
      }
      if (lc >= nbb) v[s] = 0.0;
    }
  }
  // C += V z for the row tiles of this wave; tr: two 16 x 17 tiles of the
  // wave's own in LDS, used in turn
  __device__ __forceinline__ void update(v4d (&c)[RT], const double *scr, int b, int nbb, int MT,
                                         const v4d &z, double (*tr)[16][17]) const {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if (!has(t)) continue;
      double v[4];
      load_v(scr, b, nbb, MT, t, v);
      double (*x)[17] = tr[t & 1];
#pragma unroll
      for (int s = 0; s < 4; ++s) x[4 * s + lr][lc] = v[s];
      wave_lds_order();
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) c[t] = mfma16(x[lc][4 * kk + lr], z[kk], c[t]);
    }
    wave_lds_order();
  }
  // C -= V op(T) (V^T C)
  __device__ __forceinline__ void apply(v4d (&c)[RT], const double *scr, int b, int nbb, int MT,
                                        bool trans, const double *Tg, QmShared<NW> &sh,
                                        double (*wred)[256], double *Ws,
                                        double (*tr)[16][17]) const {
    if (threadIdx.x < 256) sh.T[threadIdx.x >> 4][threadIdx.x & 15] = gmem(Tg)[threadIdx.x];
    v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if (!has(t)) continue;
      double v[4];
      load_v(scr, b, nbb, MT, t, v);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[s & 1] = mfma16(v[s], c[t][s], acc[s & 1]);
    }
    qm_reduce<NW>(acc[0] + acc[1], wred, Ws);
    update(c, scr, b, nbb, MT,
           qm_coeff(sh.T, trans, [&](int q) { return Ws[cl_index(q, lc)]; }, lr, lc), tr);
    __syncthreads();  // T and Ws are refilled by the next block
  }
};

template <int RT>
__global__ __launch_bounds__(kQrbWaves * 64) void k_qrb_factor(QrbArgs g) {
  constexpr int NW = kQrbWaves;
  const QrArgs &q = g.q;
  const int it = blockIdx.x, b = g.b, c = b + blockIdx.y;
  if (q.flag && !q.flag[it]) return;
  const QrPanel pn = qr_panel(q, it);
  const int K = q.K, m = pn.m, n = pn.n;
  __shared__ QmShared<NW> sh;
  __shared__ double wred[NW][256], Ws[256];
  __shared__ double tr[NW][2][16][17];
  const QrbTile<RT> w(m);
  double *scr = q.scratch + (size_t)it * q.scratch_stride;
  double *Tg = scr + (size_t)g.CT * g.MT * 256;
  double *Rm = q.rbuf + (size_t)it * K * K;
  if (16 * c >= n) {  // columns past the panel: only R's zeros
    if (c == b && q.want_r)
      for (int i = threadIdx.x; i < K * 16; i += NW * 64)
        if (16 * c + i % 16 < K) gmem(Rm)[(i / 16) * K + 16 * c + i % 16] = 0.0;
    return;
  }
  v4d a[RT];
  if (b <= 1) {  // from the site's slot
    const unsigned ybytes = (unsigned)(K * q.P * K) * 8u;
    const __amdgpu_buffer_rsrc_t yrs = buf_rsrc(q.Y.at(it), ybytes);
    const DivN dn2(pn.n2);
    const int col = 16 * c + w.lc;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int row = 16 * w.rtile(t) + 4 * s + w.lr;
        const unsigned o = (unsigned)(pn.row_off(row, dn2) + __mul24(col, pn.cs));
        a[t][s] = buf_ld(yrs, row < m && col < n ? o * 8u : ybytes);
      }
  } else {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        a[t][s] = w.has(t)
                      ? gmem(scr)[((size_t)c * g.MT + w.rtile(t)) * 256 + s * 64 + w.lane]
                      : 0.0;
  }
  if (b > 0) w.apply(a, scr, b - 1, 16, g.MT, true, Tg + (b - 1) * 256, sh, wred, Ws, tr[w.wave]);
  const int nbb = min(16, n - 16 * b);
  if (c == b) {
    qm_factor<NW, RT>(a, b, nbb, sh, wred, Ws);
    if (w.wave == 0) {
      wave_lds_order();
#pragma unroll
      for (int u = 0; u < 4; ++u)
        gmem(Tg)[b * 256 + (4 * u + w.lr) * 16 + w.lc] = sh.T[4 * u + w.lr][w.lc];
    }
    if (q.want_r) {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int row = 16 * w.rtile(t) + 4 * s + w.lr, col = 16 * c + w.lc;
          if (row < K && col < K)
            gmem(Rm)[row * K + col] = (t == 0 && row < n && col < n && col >= row) ? a[0][s] : 0.0;
        }
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (!w.has(t)) continue;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      gmem(scr)[((size_t)c * g.MT + w.rtile(t)) * 256 + s * 64 + w.lane] = a[t][s];
  }
}

template <int RT>
__global__ __launch_bounds__(kQrbWaves * 64) void k_qrb_q(QrbArgs g) {
  constexpr int NW = kQrbWaves;
  const QrArgs &q = g.q;
  const int it = blockIdx.x, c = g.CT - 1 - (int)blockIdx.y;  // the longest chains first
  if (q.flag && !q.flag[it]) return;
  const QrPanel pn = qr_panel(q, it);
  const int K = q.K, m = pn.m, n = pn.n;
  if (16 * c >= n) return;
  __shared__ QmShared<NW> sh;
  __shared__ double wred[NW][256], Ws[256];
  __shared__ double tr[NW][2][16][17];
  const QrbTile<RT> w(m);
  const double *scr = q.scratch + (size_t)it * q.scratch_stride;
  const double *Tg = scr + (size_t)g.CT * g.MT * 256;
  const int nbb = min(16, n - 16 * c);
  v4d a[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int s = 0; s < 4; ++s)
      a[t][s] = (t == 0 && 16 * (w.wave - c) + 4 * s + w.lr == w.lc && w.lc < nbb) ? 1.0 : 0.0;
  // the block's own columns: E - V (T V_top^T)
  if (threadIdx.x < 256) sh.T[threadIdx.x >> 4][threadIdx.x & 15] = gmem(Tg)[c * 256 + threadIdx.x];
  __syncthreads();
  const v4d z = qm_coeff(sh.T, false, [&](int k) {  // V_top[lc][k]
    const double v = gmem(scr)[((size_t)c * g.MT + c) * 256 + cl_index(w.lc, k)];
    return k < nbb ? (w.lc > k ? v : (w.lc == k ? 1.0 : 0.0)) : 0.0;
  }, w.lr, w.lc);
  __syncthreads();  // T is refilled by the next block
  w.update(a, scr, c, nbb, g.MT, z, tr[w.wave]);
  for (int b = c - 1; b >= 0; --b)
    w.apply(a, scr, b, 16, g.MT, false, Tg + b * 256, sh, wred, Ws, tr[w.wave]);
  const unsigned ybytes = (unsigned)(K * q.P * K) * 8u;
  const __amdgpu_buffer_rsrc_t yrs = buf_rsrc(q.Y.at(it), ybytes);
  const DivN dn2(pn.n2);
  const int col = 16 * c + w.lc;
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int row = 16 * w.rtile(t) + 4 * s + w.lr;
      const unsigned o = (unsigned)(pn.row_off(row, dn2) + __mul24(col, pn.cs));
      buf_st_t<double>(yrs, row < m && col < n ? o * 8u : ybytes, a[t][s]);
    }
}

// ---------------------------------------------------------------------------
// Counter-based uniform numbers: SplitMix64 (Steele, Lea, Flood 2014).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t splitmix(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// One workgroup per (site, item): zero the slot, then fill the true
// (bl, p, br) tensor with 2*(h >> 11)*2^-52... values indexed by the compact
// C-order position, exactly as the oracle does.
__global__ __launch_bounds__(kThreads) void k_rand_init(
    FitDims *dims, int W, int c, int N, int K, int P, size_t S, Ptr Y,
    const uint64_t *slot, uint64_t seed, const int32_t *flag) {
  const int j = blockIdx.x, it = blockIdx.y;
  if (!flag[it]) return;
  const FitDims &dm = dims[(size_t)it * W + c];
  double *y = Y.at(it) + (size_t)j * S;
  for (size_t i = threadIdx.x; i < S; i += kThreads) y[i] = 0.0;
  __syncthreads();
  const int bl = dm.bl[j], p = dm.p[j], br = dm.br[j];
  const uint64_t h = splitmix(splitmix(splitmix(seed) ^ (slot[it] + c)) ^
                              (uint64_t)j);
  const int total = bl * p * br;
  for (int idx = threadIdx.x; idx < total; idx += kThreads) {
    const uint64_t v = splitmix(h ^ (uint64_t)idx);
    const double u = (double)(v >> 11) * 0x1p-52 - 1.0;
    const int y0 = idx / (p * br), rem = idx - y0 * p * br;
    const int a = rem / br, y1 = rem - a * br;
    size_t addr;
    if (j == 0) addr = (size_t)a * K + y1;               // [p][br]
    else if (j == N - 1) addr = (size_t)y0 * K + a;      // [bl][p]
    else addr = ((size_t)y0 * P + a) * K + y1;           // [bl][p][br]
    y[addr] = u;
  }
}

// ---------------------------------------------------------------------------
// Column absorptions of small shapes in one launch (D = 2, d = 2, bond caps up
// to 20): one workgroup of four waves per item runs every visit of columns
// col_hi .. col_lo - random start, right environments, the n_fit sweeps, the
// final centre and its norm - with the visit's operands in LDS.  Launched one
// by one these visits are three kernels of 4 to 8 us of which the arithmetic
// is a fraction (K = 8: 0.2 MFLOP), so the chain of launches bounded them:
// one message update of a 2x2 block at chi = 4 was 130 launches.
//
// A visit: four lanes per (yf, xb) pair contract F, X, ket and bra in registers
// (T1, T2, T3 are 4 x 4 each; a lane makes a row of T1, passes it round the
// quad and takes one column (lk, wbk) of the ket's output through the bra) and
// leave T3 in LDS as [(yf, l)][(xb, wb)]; the local update Yt = T3 G on MFMA
// lands in the QR's register layout (RL visits read T3's rows in the order
// (l, yf) of their panel); the QR is qm_panel, up to K = 8 by one wave, whose
// steps then need no barrier; and env' = Q^T T3 on MFMA is the next visit's F,
// in LDS, and goes to memory for the sweep back.  The end sites are the same
// with T[a][(xb, q)] in place of T3.  X, G, the site tensor (or an end site's
// message) of the next visit are fetched into registers before the QR.  An end
// visit's G is the environment just computed.
//
// All loops stop at the item's true bonds.  LDS at bond cap K: T3 (4 K)^2
// doubles and the QR's buffers, which leaves room up to K = 20.
//
// Bound by the chain of a visit: 4.8 us at K = 4 (a 2x2 block's 8 messages of
// one sweep 153 us, against 480 us of launches of which each waited for the
// one before), 12 us at K = 18.
// ---------------------------------------------------------------------------
struct SmallArgs {
  FitBatch f;
  int col_lo, col_hi, n_fit;
};

// QW waves factorise: 1 up to K = 8 (32 rows), else all four
template <int CT, int QW>
struct SmallShape {
  static constexpr int P = 4, NW = 4, NT = 64 * NW, RT = QW == 1 ? 2 : CT;
  static constexpr int QS = CT == 1 ? 16 : 48;  // row stride of Q and G: 16 (mod 32)
  typedef QmBuf<QW, RT, CT> Qm;
  // K P K / NT elements a thread
  static constexpr int NPF = QW == 1 ? 1 : CT == 1 ? 4 : 7;
  // row stride of T3: 18 (mod 32), conflict-free as the A operand of the local
  // update (16 rows, 4 k) and nearly so as the B operand of env'
  static __host__ __device__ int ld3(int K) { return P * K + (50 - P * K % 32) % 32; }
  static __host__ __device__ int fst(int K) { return P * K + 1; }
  static __host__ __device__ size_t words(int K) {
    const size_t qm = sizeof(Qm) / 8, q = (size_t)(P * K + 4) * QS + 64;
    return (size_t)P * K * ld3(K) + 64 + (size_t)P * K * QS + (size_t)K * fst(K) +
           (size_t)K * P * K + 64 + (qm > q ? qm : q);
  }
};

template <int CT, int QW>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(CT == 1 ? 2 : 1))) void k_absorb_small(SmallArgs g) {
  typedef SmallShape<CT, QW> Sh;
  constexpr int P = Sh::P, NT = Sh::NT, NW = Sh::NW, RT = Sh::RT, QS = Sh::QS, NPF = Sh::NPF;
  extern __shared__ double sm_raw[];
  __shared__ double As[64];  // ket, then bra: front view [s][wf, a][l, wb]
  __shared__ double red[NW];
  __shared__ FitDims dm;
  const FitBatch &f = g.f;
  const int K = f.K, N = f.N, W = f.W, KPK = K * P * K, it = blockIdx.x;
  const int LD = Sh::ld3(K), FS = Sh::fst(K);
  int tid = threadIdx.x;
  double *T3 = sm_raw;                     // [(yf, l)][(xb, wb)]
  double *Gs = T3 + P * K * LD + 64;       // [(xb, wb)][yb]
  double *Fs = Gs + P * K * QS;            // [yf][wf][xf]; an end site's message [a][q][a']
  double *Xs = Fs + K * FS;                // [xf][a][xb]; an end site's X [a'][xb]
  auto &qm = *reinterpret_cast<typename Sh::Qm *>(Xs + KPK + 64);
  double *Qs = Xs + KPK + 64;              // [(yf, l)][yb], after the QR is done with its LDS
  const DivN dK(K);
  const size_t S = f.S;
  double *store = f.store + (size_t)it * W * N * S;
  double *lenv = f.lenv + (size_t)it * N * S, *renv = f.renv + (size_t)it * N * S;
  auto zero_tiles = [&](v4d (&a)[CT][RT]) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int t = 0; t < RT; ++t) a[ct][t] = v4d{0.0, 0.0, 0.0, 0.0};
  };

  for (int col = g.col_hi; col >= g.col_lo; --col) {
    __syncthreads();  // the previous column's reads of dm and its stores
    {
      const int *src = reinterpret_cast<const int *>(f.dims + (size_t)it * W + col);
      int *dst = reinterpret_cast<int *>(&dm);
      for (int i = tid; i < (int)(sizeof(FitDims) / 4); i += NT) dst[i] = src[i];
    }
    __syncthreads();
    double *Y = store + (size_t)col * N * S;
    const double *X = col == W - 1 ? f.xin + (size_t)it * N * S : Y + (size_t)N * S;
    const double *MT = f.mt + ((size_t)it * W + col) * S, *MB = f.mb + ((size_t)it * W + col) * S;

    const uint64_t h0 = splitmix(splitmix(f.seed) ^ (f.slot[it] + col));
    if (dm.rnd)
      for (int i = tid; i < N * (int)S; i += NT) Y[i] = 0.0;

    // Visits of the column in order: with a random start, sites N - 1 .. 1 of it
    // brought to right-canonical form (v < 0); N - 1 right environments (site
    // N - 1 .. 1), then n_fit times left to right (0 .. N - 2) and right to
    // left (N - 1 .. 1), then the final centre at site 0.
    const int nv = (N - 1) * (1 + 2 * g.n_fit) + 1;
    auto visit = [&](int v, int &j, bool &rl, int &mode) __attribute__((always_inline)) {
      if (v < 0) {
        j = -v;
        rl = true;
        mode = 3;
        return;
      }
      if (v == nv - 1) {
        j = 0;
        rl = false;
        mode = 2;
        return;
      }
      const int sweep = v / (N - 1), k = v - sweep * (N - 1);
      rl = (sweep & 1) == 0;
      j = rl ? N - 1 - k : k;
      mode = sweep == 0 ? 0 : 1;  // 0 environment only, 1 fit, 2 final, 3 start
    };
    double xr[NPF], gr[NPF], mr[NPF], yr[NPF], ar = 0.0;
    auto fetch = [&](int v) __attribute__((always_inline)) {
      int j, mode;
      bool rl;
      visit(v, j, rl, mode);
      const bool end = j == 0 || j == N - 1;
      const double *x = X + (size_t)j * S;
      const double *gsrc = (rl ? lenv : renv) + (size_t)j * S;
      const double *msrc = rl ? MB : MT;
#pragma unroll
      for (int u = 0; u < NPF; ++u) {
        const int e = tid + NT * u;
        xr[u] = e < (end ? K * K : KPK) ? gmem(x)[e] : 0.0;
        gr[u] = mode > 0 && !end && e < KPK ? gmem(gsrc)[e] : 0.0;
        mr[u] = end && e < KPK ? gmem(msrc)[e] : 0.0;
        // environment-only visits read the site's current tensor
        yr[u] = mode == 0 && e < (end ? K * K : KPK) ? gmem(Y)[(size_t)j * S + e] : 0.0;
      }
      if (!end && tid < 64) {  // site tensors in the front view: ket, then bra
        const size_t site = (((size_t)it * f.H + (j - 1)) * W + col) * 32;
        const double *src = tid < 32      ? f.acan + site
                            : f.bra_one   ? f.bra_one
                                          : (f.abra ? f.abra : f.acan) + site;
        const int wb = tid & 1, l = (tid >> 1) & 1, a = (tid >> 2) & 1, wf = (tid >> 3) & 1,
                  s = (tid >> 4) & 1;
        ar = src[(((s * 2 + (rl ? wb : wf)) * 2 + l) * 2 + (rl ? wf : wb)) * 2 + a];
      }
    };
    const int v0 = dm.rnd ? 1 - N : 0;
    if (v0 == 0) fetch(0);
    for (int v = v0; v < nv; ++v) {
      // opaque: the lane's offsets are formed in each visit instead of held in
      // registers across all of them
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      const int lr = lane & 15, lq = lane >> 4;
      int j, mode;
      bool rl;
      visit(v, j, rl, mode);
      const bool end = j == 0 || j == N - 1;
      const SiteExt ex = site_ext(dm, j, N, rl);
      // end sites: rows a of the message site, back bonds of Y and X
      const int nyf = end ? 1 : ex.yf, nyb = ex.yb, nxf = ex.xf, nxb = ex.xb;
      const int M = end ? dm.p[j] : nyf * P, Nn = nxb * P;
      v4d a[CT][RT];
      int nat[RT][4];  // T3 row of panel row 16 (wave + NW t) + 4 s + lq
      const int n = min(nyb, M);
      if (mode == 3) {
        // counter-based random site (k_rand_init): its panel, rows (l, y') and
        // columns the left bond, times the R of the next site (in Xs); Q
        // replaces the site and R goes on to the one before.  Site 0 is not
        // made: the first visit that reads it has written it.
        const int p = dm.p[j], br = dm.br[j], bl = dm.bl[j];
        const uint64_t h = splitmix(h0 ^ (uint64_t)j);
        for (int i = tid; i < bl * p * br; i += NT)
          Fs[i] = (double)(splitmix(h ^ (uint64_t)i) >> 11) * 0x1p-52 - 1.0;  // U [bl][p][br]
        __syncthreads();
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int row = min(16 * (wave + QW * t) + 4 * s + lq, M - 1);
            const int l = row / br, y = row - l * br;
            nat[t][s] = end ? row : y * P + l;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
              const int c = 16 * ct + lr;
              double x = 0.0;
              if (wave < QW && 16 * (wave + QW * t) + 4 * s + lq < M && c < n) {
                const double *u = Fs + (c * p + l) * br;
                if (end) x = u[y];
                else
                  for (int k = y; k < br; ++k) x = fma(u[k], Xs[y * K + k], x);
              }
              a[ct][t][s] = x;
            }
          }
        __syncthreads();  // Xs is read
      } else {
        // an end visit's G is the environment the previous visit left in Fs
        if (end && mode > 0) {
          for (int i = tid; i < nyb * Nn; i += NT) {
            const int yb = i / Nn, n = i - yb * Nn;
            Gs[n * QS + yb] = Fs[yb * FS + (n & 3) * K + (n >> 2)];
          }
          __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < NPF; ++u) {
          const int e = tid + NT * u;
          if (end) {
            if (e < K * K) {
              const int i0 = dK.quot(e), i1 = e - i0 * K;
              Xs[rl ? i1 * K + i0 : e] = xr[u];
            }
            if (e < KPK) Fs[e] = mr[u];
          } else if (e < KPK) {
            const int q = dK.quot(e), i1 = e - q * K, a = q & 3, i0 = q >> 2;
            Xs[rl ? (i1 * P + a) * K + i0 : e] = xr[u];
            if (mode > 0) Gs[(i1 * P + a) * QS + i0] = gr[u];
          }
        }
        if (!end && tid < 64) As[tid] = ar;
        if (mode == 0) {  // the site as Q
#pragma unroll
          for (int u = 0; u < NPF; ++u) {
            const int e = tid + NT * u;
            if (e >= (end ? K * K : KPK)) continue;
            const int q = dK.quot(e), i1 = e - q * K;
            if (end) {  // Y [yb][a]
              if (i1 < M) Qs[i1 * QS + q] = yr[u];
            } else if (i1 < nyf) {  // Y [yb][l][yf]
              Qs[(i1 * P + (q & 3)) * QS + (q >> 2)] = yr[u];
            }
          }
        }
        __syncthreads();
        // ---- T3 --------------------------------------------------------------
        if (end) {  // T[a][xb][q] = sum_a' M[a][q][a'] X[a'][xb]
          const int na = dm.p[j];
          const int ap = col == W - 1 ? 1 : f.dims[(size_t)it * W + col + 1].p[j];
          for (int i = tid; i < na * nxb; i += NT) {
            const int a = i / nxb, xb = i - a * nxb;
            double t[P] = {0.0, 0.0, 0.0, 0.0};
            for (int k = 0; k < ap; ++k) {
              const double x = Xs[k * K + xb];
#pragma unroll
              for (int q = 0; q < P; ++q) t[q] = fma(Fs[(a * P + q) * K + k], x, t[q]);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) T3[a * LD + xb * P + q] = t[q];
          }
        } else {
          for (int i = tid; i < nyf * nxb * 4; i += NT) {
            const int q = i & 3, pr = i >> 2, yf = pr / nxb, xb = pr - yf * nxb;
            double t1[P][P];  // [wf][a]; this lane's row wf = q first
            double tq[P] = {0.0, 0.0, 0.0, 0.0};
            const double *pf = Fs + yf * FS + q * K, *px = Xs + xb;
#pragma unroll 4
            for (int k = nxf - 1; k >= 0; --k) {
              const double fv = pf[k];
#pragma unroll
              for (int a = 0; a < P; ++a) tq[a] = fma(fv, px[(k * P + a) * K], tq[a]);
            }
#pragma unroll
            for (int a = 0; a < P; ++a) {
              t1[0][a] = quad_bcast<0>(tq[a]);
              t1[1][a] = quad_bcast<1>(tq[a]);
              t1[2][a] = quad_bcast<2>(tq[a]);
              t1[3][a] = quad_bcast<3>(tq[a]);
            }
            double t3[P] = {0.0, 0.0, 0.0, 0.0};  // (lb, wbb) of column q = (lk, wbk)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              double t2[P] = {0.0, 0.0, 0.0, 0.0};  // (wfb, ab)
#pragma unroll
              for (int k = 0; k < P; ++k) {  // (wfk, ak)
                const double b = As[(s * P + k) * P + q];
#pragma unroll
                for (int m = 0; m < P; ++m)
                  t2[m] = fma(t1[(k >> 1) * 2 + (m >> 1)][(k & 1) * 2 + (m & 1)], b, t2[m]);
              }
#pragma unroll
              for (int k = 0; k < P; ++k)  // (wfb, ab)
#pragma unroll
                for (int n = 0; n < P; ++n)
                  t3[n] = fma(t2[k], As[32 + (s * P + k) * P + n], t3[n]);
            }
#pragma unroll
            for (int n = 0; n < P; ++n)  // l = (lk, lb), wb = (wbk, wbb)
              T3[(yf * P + (q >> 1) * 2 + (n >> 1)) * LD + xb * P + (q & 1) * 2 + (n & 1)] = t3[n];
          }
        }
        if (v + 1 < nv) fetch(v + 1);
        __syncthreads();
        if (mode != 0 && wave < QW) {
          // ---- Yt in the panel's register layout -------------------------------
          zero_tiles(a);
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            const int m0 = 16 * (wave + QW * t);
            auto natural = [&](int m) __attribute__((always_inline)) {
              if (end || !rl) return m;
              const int l = m / nyf;
              return (m - l * nyf) * P + l;  // rows (l, yf)
            };
#pragma unroll
            for (int s = 0; s < 4; ++s) nat[t][s] = natural(min(m0 + 4 * s + lq, M - 1));
            if (m0 >= M) continue;
            const double *pa = T3 + natural(min(m0 + lr, M - 1)) * LD + lq;
            const double *pb = Gs + lq * QS + lr;
            for (int k = 0; k < Nn; k += 4) {
              const double x = pa[k];
#pragma unroll
              for (int ct = 0; ct < CT; ++ct)
                a[ct][t] = mfma16(x, pb[k * QS + 16 * ct], a[ct][t]);
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
              for (int s = 0; s < 4; ++s)
                if (m0 + 4 * s + lq >= M || 16 * ct + lr >= (mode == 2 ? nyb : n)) a[ct][t][s] = 0.0;
          }
        }
        if (mode == 2) {  // the final centre, scaled to unit norm
          if (wave < QW) {
            double part = 0.0;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
              for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s) part = fma(a[ct][t][s], a[ct][t][s], part);
            part = wave_sum(part);
            if (lane == 0) red[wave] = part;
          }
          __syncthreads();
          double ss = red[0];
#pragma unroll
          for (int w = 1; w < QW; ++w) ss += red[w];
          const double nrm = sqrt(ss);
          const bool ok = nrm > 0.0 && isfinite(nrm);
          if (tid == 0) {
            f.nu[(size_t)it * W + col] = nrm;
            if (!ok) atomicOr(f.err, 1);
          }
          const double inv = ok ? 1.0 / nrm : 1.0;
          if (wave < QW) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
              for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                  const int row = 16 * (wave + QW * t) + 4 * s + lq, c = 16 * ct + lr;
                  if (row < M && c < nyb) Y[row * K + c] = a[ct][t][s] * inv;
                }
          }
          break;
        }
      }
      if (mode != 0 && wave < QW) {
        qm_panel<QW, RT, CT>(a, n, qm, [&]() __attribute__((always_inline)) {
          if (mode != 3) return;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              const int row = 16 * wave + 4 * s + lq, c = 16 * ct + lr;
              if (row < n && c < n) Xs[row * K + c] = c >= row ? a[ct][0][s] : 0.0;
            }
        }, tid);
        if constexpr (QW > 1) __syncthreads();  // the QR's LDS is free
        else wave_lds_order();
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int row = 16 * (wave + QW * t) + 4 * s + lq;
            if (row >= M) continue;
            const int r = nat[t][s];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
              const int c = 16 * ct + lr;
              Qs[r * QS + c] = a[ct][t][s];
              if (c >= n) continue;
              // LR: [row][yb]; RL: end [yb][a], inner [yb][l][yf]
              const size_t o = !rl ? (size_t)row * K + c
                                   : (end ? (size_t)c * K + row
                                          : (size_t)(c * P + (r & 3)) * K + (r >> 2));
              Y[(size_t)j * S + o] = a[ct][t][s];
            }
          }
      }
      if (v == -1) fetch(0);
      __syncthreads();
      if (mode == 3) continue;
      // ---- env'[yb][(xb, wb)] = sum_rows Q[row][yb] T3[row][(xb, wb)] ---------
      {
        const int tm = (nyb + 15) >> 4, tn = (Nn + 15) >> 4;
        const int jn = rl ? j - 1 : j + 1;
        double *E = (rl ? renv : lenv) + (size_t)jn * S;
        const bool keep = jn > 0 && jn < N - 1;  // read again by the sweep back
        for (int i = wave; i < tm * tn; i += NW) {
          const int m0 = (i / tn) << 4, n0 = (i % tn) << 4;
          const double *pa = Qs + lq * QS + m0 + lr, *pb = T3 + lq * LD + n0 + lr;
          v4d e = {0.0, 0.0, 0.0, 0.0};
          for (int k = 0; k < M; k += 4) {
            const bool in = k + lq < M;
            e = mfma16(in ? pa[k * QS] : 0.0, in ? pb[k * LD] : 0.0, e);
          }
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int m = m0 + 4 * s + lq, n = n0 + lr;
            if (m < nyb && n < Nn) {
              const int o = (n & 3) * K + (n >> 2);
              Fs[m * FS + o] = e[s];
              if (keep) E[m * P * K + o] = e[s];
            }
          }
        }
      }
      __syncthreads();
    }
  }
}

__global__ void k_set_unit(Ptr slot, size_t S) {
  double *s = slot.at(blockIdx.y);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < S;
       i += (size_t)gridDim.x * blockDim.x)
    s[i] = (i == 0) ? 1.0 : 0.0;
}

__global__ __launch_bounds__(kThreads) void k_copy_flagged(
    const double *src, size_t sstride, Ptr dst, size_t n, const int32_t *flag) {
  const int it = blockIdx.y;
  if (flag && !flag[it]) return;
  double *d = dst.at(it);
  const double *s = src + (size_t)it * sstride;
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n;
       i += (size_t)gridDim.x * kThreads)
    d[i] = s[i];
}

// Norm of the end slot (K*K doubles) per item; scale to unit norm.
// nu[it*W] receives the norm (nu already offset to the column).
__global__ __launch_bounds__(kThreads) void k_normalize(Ptr Y0, int K,
                                                        double *nu, int W,
                                                        int32_t *err) {
  const int it = blockIdx.x;
  double *y = Y0.at(it);
  const int n = K * K;
  double part = 0.0;
  for (int i = threadIdx.x; i < n; i += kThreads) part += y[i] * y[i];
  part = wave_sum(part);
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = part;
  __syncthreads();
  const double nrm = sqrt(red[0] + red[1] + red[2] + red[3]);
  const bool ok = nrm > 0.0 && isfinite(nrm);
  if (threadIdx.x == 0) {
    nu[(size_t)it * W] = nrm;
    if (!ok) atomicOr(err, 1);
  }
  if (ok) {
    const double inv = 1.0 / nrm;
    for (int i = threadIdx.x; i < n; i += kThreads) y[i] *= inv;
  }
}

// Copy one message site [a][q][b] from a slot with bond cap ks to a slot
// with bond cap kd (kd >= ks), optionally transposed to [b][q][a].  The
// destination slot is fully written (zero padding included).
__device__ __forceinline__ void copy_site(const double *src, double *dst,
                                          int ks, int kd, int P, bool tr,
                                          double scale, int tid, int nt) {
  const size_t S = (size_t)kd * P * kd;
  for (size_t i = tid; i < S; i += nt) {
    const int a = (int)(i / ((size_t)P * kd));
    const int rem = (int)(i - (size_t)a * P * kd);
    const int qq = rem / kd, b = rem - qq * kd;
    double v = 0.0;
    if (a < ks && b < ks)
      v = tr ? src[((size_t)b * P + qq) * ks + a] : src[((size_t)a * P + qq) * ks + b];
    dst[i] = scale * v;
  }
}

// blockIdx.x: site, blockIdx.y: which (0 top, 1 boundary, 2 bottom),
// blockIdx.z: item.
__global__ __launch_bounds__(kThreads) void k_gather(FitBatch f,
                                                     const GatherSrc *srcs) {
  const int site = blockIdx.x, which = blockIdx.y, it = blockIdx.z;
  const GatherSrc &g = srcs[it];
  const int K = f.K, P = f.P;
  const size_t S = f.S;
  int k, i;
  double *dst;
  if (which == 1) {
    if (site >= f.N) return;
    dst = f.xin + ((size_t)it * f.N + site) * S;
    if (site == 0 || site == f.N - 1) {
      for (size_t t = threadIdx.x; t < S; t += kThreads)
        dst[t] = (t == 0) ? 1.0 : 0.0;
      return;
    }
    k = 1;
    i = site - 1;
  } else {
    if (site >= f.W) return;
    k = which == 0 ? 0 : 2;
    i = site;
    dst = (which == 0 ? f.mt : f.mb) + ((size_t)it * f.W + site) * S;
  }
  const int seg = i < g.n[k][0] ? 0 : 1;
  const int loc = seg ? i - g.n[k][0] : i;
  const int n = g.n[k][seg];
  const bool rev = g.rev[k][seg] != 0;
  const int src_site = rev ? n - 1 - loc : loc;
  const size_t Ss = (size_t)g.ksrc * P * g.ksrc;
  copy_site(g.src[k][seg] + (size_t)src_site * Ss, dst, g.ksrc, K, P, rev, 1.0,
            threadIdx.x, kThreads);
}

// Final boundary (column 0) of each item -> message of H sites.
__global__ __launch_bounds__(kThreads) void k_extract(FitBatch f,
                                                      double *const *dst,
                                                      const int32_t *rev) {
  const int i = blockIdx.x, it = blockIdx.y;
  const int L = f.H;
  const double *Y = f.store + ((size_t)it * f.W * f.N) * f.S;  // column 0
  double scale = 1.0;
  if (i == 0) scale *= Y[0];                              // site 0 scalar
  if (i == L - 1) scale *= Y[(size_t)(f.N - 1) * f.S];    // site N-1 scalar
  const int out = rev[it] ? L - 1 - i : i;
  copy_site(Y + (size_t)(i + 1) * f.S, dst[it] + (size_t)out * f.S, f.K, f.K,
            f.P, rev[it] != 0, scale, threadIdx.x, kThreads);
}

__global__ __launch_bounds__(kThreads) void k_copy_jobs(const CopyJob *jobs,
                                                        int K, int P) {
  const CopyJob j = jobs[blockIdx.y];
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < j.n;
       i += (int64_t)gridDim.x * kThreads) {
    int64_t from = i;
    if (j.mode == 1) {
      const int64_t a = i / ((int64_t)P * K), rem = i - a * P * K;
      const int64_t qq = rem / K, b = rem - qq * K;
      from = (b * P + qq) * K + a;
    } else if (j.mode == 2) {
      if (i >= (int64_t)K * K) {
        j.dst[i] = 0.0;
        continue;
      }
      const int64_t a = i / K, b = i - a * K;
      from = b * K + a;
    }
    j.dst[i] = j.src[from];
  }
}

__global__ __launch_bounds__(kThreads) void k_dots(const double *const *a,
                                                   const double *const *b,
                                                   size_t n, double *out) {
  const int it = blockIdx.x;
  const double *x = a[it], *y = b[it];
  double part = 0.0;
  for (size_t i = threadIdx.x; i < n; i += kThreads) part += x[i] * y[i];
  part = wave_sum(part);
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = part;
  __syncthreads();
  if (threadIdx.x == 0) out[it] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ void k_ov_init(double *E, int K) {
  const int it = blockIdx.x;
  for (int i = threadIdx.x; i < K * K; i += blockDim.x)
    E[(size_t)it * K * K + i] = (i == 0) ? 1.0 : 0.0;
}
__global__ void k_ov_out(const double *E, int K, int items, double *out) {
  const int it = blockIdx.x * blockDim.x + threadIdx.x;
  if (it < items) out[it] = E[(size_t)it * K * K];
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static Shape shape_of(const FitBatch &f) { return Shape{f.K, f.P, f.D, f.d}; }
static size_t t1_stride(const FitBatch &f) { return (size_t)f.K * f.P * f.P * f.K; }
static size_t t2_stride(const FitBatch &f) {
  return (size_t)f.d * f.K * f.K * f.P * f.P;
}
static size_t a_site(const FitBatch &f) { return (size_t)f.d * f.P * f.P; }
static size_t a_stride(const FitBatch &f) { return (size_t)f.H * f.W * a_site(f); }

// Tile shape of the fused visit: the largest TY x TX pair set whose LDS
// footprint fits, or TY = 0 when none does (generic chain then).
static void visit_tiles(const FitBatch &f, int *TY, int *TX, size_t *bytes) {
  const size_t K = f.K, P = f.P;
  const int cand[][2] = {{2, 8}, {2, 4}, {4, 2}, {2, 2}, {1, 4}, {1, 2}, {1, 1}};
  for (auto &c : cand) {
    const size_t ty = c[0], tx = c[1];
    if ((int)ty > f.K) continue;
    size_t n = visit_lds(f.K, f.P, f.d, (int)ty, (int)tx);
    const size_t tiles = ((ty * P + 15) / 16) * ((K + 15) / 16);
    if (2 * tiles <= (size_t)kVisitWaves) n = std::max(n, tiles * 256);  // k-half sums
    if (n * 8 <= 150 * 1024 && tiles <= 4 * (size_t)kVisitWaves) {
      *TY = (int)ty;
      *TX = (int)tx;
      *bytes = n * 8;
      return;
    }
  }
  *TY = 0;
}

using VisitKernel = void (*)(VisitArgs);

template <class T, bool B16 = false>
static VisitKernel visit_kernel(int D) {
  switch (D) {
    case 2: return k_visit<2, T, B16>;
    case 3: return k_visit<3, T, B16>;
    case 4: return k_visit<4, T, B16>;
    case 5: return k_visit<5, T, B16>;
    case 6: return k_visit<6, T, B16>;
    default: return k_visit<0, T, B16>;
  }
}

// Tiles of the D = 4, d = 2 kernel: the first candidate whose LDS fits.
template <class T>
static bool visit4_tiles(const FitBatch &f, int *TY, int *TX, size_t *bytes) {
  if (f.D != 4 || f.d != 2 || f.K > 128) return false;
  const int cand[][2] = {{2, 4}, {4, 2}, {2, 2}, {1, 2}, {1, 1}};
  for (auto &c : cand) {
    if (c[0] > f.K) continue;
    const size_t n = visit4_lds<T>(f.K, c[0], c[1]) * sizeof(T);
    const size_t moved = (size_t)std::max(ceil4(f.K), ceil16(f.K)) * 16 * c[1];
    if (n <= 150 * 1024 && moved <= 8 * (size_t)kVisitThreads) {
      *TY = c[0];
      *TX = c[1];
      *bytes = n;
      return true;
    }
  }
  return false;
}

template <class T>
static VisitKernel visit4_kernel(int TY, int TX) {
  if (TY == 2 && TX == 4) return k_visit4<2, 4, T>;
  if (TY == 4 && TX == 2) return k_visit4<4, 2, T>;
  if (TY == 2 && TX == 2) return k_visit4<2, 2, T>;
  if (TY == 1 && TX == 2) return k_visit4<1, 2, T>;
  return k_visit4<1, 1, T>;
}

// NE = number of 16-wide local-update tiles the kernel is built for (>= 2).
static int visit4p_ne(int K) { return std::max(2, ceil16(K) / 16); }

// Pair-per-wave visit (K <= 64): 2 x 2 pairs, 4 x 1 at NE = 3.  A small
// batch takes 1 x 4 pairs: two or four times the workgroups, each walking a
// quarter of the columns xb.  At NE <= 2 that is a batch whose 2 x 2 grid would
// not give every CU a workgroup.  At NE = 3 (FP64) it is one of fewer than 128
// workgroups of 4 x 1 pairs; the two at 72 workgroups of K = 33 49 and 31 us, at
// 96 of K = 48 65 and 39.  Launches of up to 204 gain as well (140 of K = 40 76
// and 50, 204 of K = 48 89 and 83), 216 to 310 are about even and 360 of K = 33
// (84 and 98) and 480 of K = 48 (119 and 159) lose; the rule sees the whole
// batch, of which one launch may hold half, and leaves those as they are.
template <class T>
static bool visit4p_tiles(const FitBatch &f, int *TY, int *TX, size_t *bytes) {
  if (f.D != 4 || f.d != 2 || f.K > 64) return false;
  const int ne = visit4p_ne(f.K);
  const long sel = f.tile_items > 0 ? f.tile_items : f.items;
  const bool small = (ne <= 2 && sel * ((f.K + 1) / 2) < 256) ||
                     (ne == 3 && sizeof(T) == 8 && sel * ((f.K + 3) / 4) < 128);
  const int ty = small ? 1 : ne == 3 ? 4 : 2, tx = small ? 4 : ne == 3 ? 1 : 2;
  const size_t n = visit4p_lds<T>(f.K, ty, tx) * sizeof(T);
  if (n > 150 * 1024) return false;
  *TY = ty;
  *TX = tx;
  *bytes = n;
  return true;
}


template <class T>
static VisitKernel visit4p_kernel(int NE, int TY) {
  if (NE <= 2) return TY == 1 ? k_visit4p<1, 4, T, 2> : k_visit4p<2, 2, T, 2>;
  if constexpr (sizeof(T) == 8)
    if (NE == 3 && TY == 1) return k_visit4p<1, 4, T, 3>;
  if (NE == 3) return k_visit4p<4, 1, T, 3>;
  return k_visit4p<2, 2, T, 4>;
}

// BF16 contractions (precision 16) run in the generic fused visit and the
// environment update at bond caps <= 64, any D; T3 passes between them in
// FP32.  Elsewhere precision 16 leaves FP64 in place.
static bool visit_bf16(const FitBatch &f) {
  int TY, TX;
  size_t lds;
  if (f.prec != 16 || f.K > 64) return false;
  visit_tiles(f, &TY, &TX, &lds);
  return TY > 0;
}

// FP32 T3 and environment update: the FP32 contractions (precision 32) run
// where both the visit and the environment update have an FP32 form (every
// fused visit at K <= 64), and the BF16 ones (above) keep T3 in FP32 too.
// Elsewhere the precision option leaves FP64 in place.
static bool visit_f32(const FitBatch &f) {
  int TY, TX;
  size_t lds;
  if (f.prec == 16) return visit_bf16(f);
  if (f.prec != 32 || f.K > 64) return false;
  if (visit4_tiles<float>(f, &TY, &TX, &lds)) return true;
  visit_tiles(f, &TY, &TX, &lds);  // the generic fused visit
  return f.D != 4 && TY > 0;
}

// ---- algorithmic counts on the true extents (timing only) -----------------
// Floating-point operations and operand bytes of the split-layer
// contractions of one launch, summed over its items with each item's true
// bonds (f.hdims, present for the column absorptions).  Launches without
// them (the observables' line sandwiches) count at the bond cap.
enum : int { TC_T1 = 1, TC_KET = 2, TC_BRA = 4, TC_LOCAL = 8, TC_ENV = 16 };
struct Count {
  double flops = 0.0, bytes = 0.0;
};
static Count count_inner(const FitBatch &f, int c, int j, bool rl, int parts) {
  Count t;
  if (!timing_enabled()) return t;
  const double P = f.P, d = f.d;
  for (int i = 0; i < f.items; ++i) {
    double yf = f.K, yb = f.K, xf = f.K, xb = f.K;
    if (f.hdims) {
      const SiteExt e = site_ext(f.hdims[(size_t)i * f.W + c], j, f.N, rl);
      yf = e.yf, yb = e.yb, xf = e.xf, xb = e.xb;
    }
    double m = 0.0, b = 0.0;  // multiply-adds, doubles moved
    if (parts & TC_T1) m += yf * P * xf * P * xb, b += yf * P * xf + xf * P * xb;
    if (parts & TC_KET) m += yf * xb * d * P * P * P, b += d * P * P;
    if (parts & TC_BRA) m += yf * xb * d * P * P * P;
    if (parts & TC_LOCAL) m += yf * P * xb * P * yb, b += yb * P * xb + yf * P * yb;
    if (parts & TC_ENV) m += yb * P * xb * yf * P, b += yf * P * yb + yb * P * xb;
    t.flops += 2.0 * m;
    t.bytes += 8.0 * b;
  }
  return t;
}
// End site (0 in LR, N-1 in RL): the message site of the column as an MPO
// Mend[a][q][a'] against the X corner [a'][xe]; parts 1 chain, 2 local, 4 env.
static Count count_end(const FitBatch &f, int c, bool rl, int parts) {
  Count t;
  if (!timing_enabled()) return t;
  const double P = f.P;
  for (int i = 0; i < f.items; ++i) {
    double a = f.K, ap = f.K, xe = f.K, ye = f.K;
    if (f.hdims) {
      const FitDims &d = f.hdims[(size_t)i * f.W + c];
      const int j = rl ? f.N - 1 : 0;
      a = d.p[j];
      ap = c == f.W - 1 ? 1 : f.hdims[(size_t)i * f.W + c + 1].p[j];
      xe = rl ? d.xb[f.N - 2] : d.xb[0];
      ye = rl ? d.bl[f.N - 1] : d.br[0];
    }
    double m = 0.0, b = 0.0;
    if (parts & 1) m += a * P * ap * xe, b += a * P * ap + ap * xe;
    if (parts & 2) m += a * P * xe * ye, b += ye * P * xe + a * ye;
    if (parts & 4) m += ye * a * P * xe, b += a * ye + ye * P * xe;
    t.flops += 2.0 * m;
    t.bytes += 8.0 * b;
  }
  return t;
}
// Householder QR/LQ of the true panels: 4 m n^2 - 4 n^3 / 3 (R and Q).
static Count count_qr(const FitBatch &f, int c, int j, int mode) {
  Count t;
  if (!timing_enabled()) return t;
  for (int i = 0; i < f.items; ++i) {
    double m = (double)f.K * f.P, n = f.K;
    if (f.hdims) {
      const FitDims &d = f.hdims[(size_t)i * f.W + c];
      const bool lr = mode == LR_INNER || mode == LR_TOP;
      m = (double)(lr ? d.bl[j] : d.br[j]) * d.p[j];
      n = lr ? d.br[j] : d.bl[j];
    }
    t.flops += 4.0 * m * n * n - 4.0 * n * n * n / 3.0;
    t.bytes += 16.0 * m * n;
  }
  return t;
}

// The pair-per-wave visit of the other bond dimensions: its kernel, tile and
// LDS for this batch, or false (D = 4, other d, bond caps above 64 and the
// FP32 and BF16 contractions have kernels of their own).  The tile depends on
// the shape alone; only the xb split of D >= 5 above 32 rows looks at the
// batch, through the items the tiling is chosen for.
using VisitPKernel = void (*)(VisitPArgs);
struct VisitPChoice {
  VisitPKernel k = nullptr;
  int TY = 1, threads = 0, nsplit = 1;
  size_t lds = 0;
};
template <int D, int TY, int TX, int NE>
static VisitPChoice visitp_choice() {
  typedef VisitPShape<D, TY, TX, NE> Sh;
  static_assert(Sh::lds <= 160 * 1024, "LDS of one workgroup");
  return VisitPChoice{k_visitp<D, TY, TX, NE>, TY, Sh::NT, 1, Sh::lds};
}
template <int D>
static VisitPChoice visitp_small(int ne) {
  switch (ne) {
    case 1: return visitp_choice<D, 1, 4, 1>();
    case 2: return visitp_choice<D, 1, 4, 2>();
    case 3: return visitp_choice<D, 1, 4, 3>();
    default: return visitp_choice<D, 1, 4, 4>();
  }
}
template <int D>
static VisitPChoice visitp_large(int ne) {
  switch (ne) {
    case 1: return visitp_choice<D, 1, 4, 1>();
    case 2: return visitp_choice<D, 1, 4, 2>();
    case 3: return visitp_choice<D, 4, 1, 3>();
    default: return visitp_choice<D, 4, 1, 4>();
  }
}
static VisitPChoice visitp_kernel(int D, int ne) {
  switch (D) {
    case 2: return visitp_small<2>(ne);
    case 3: return visitp_small<3>(ne);
    case 5: return visitp_large<5>(ne);
    case 6: return visitp_large<6>(ne);
    default: return VisitPChoice{};
  }
}
static VisitPChoice visitp_tiles(const FitBatch &f) {
  if (f.d != 2 || f.K > 64) return VisitPChoice{};
  VisitPChoice c = visitp_kernel(f.D, (f.K + 15) / 16);
  if (!c.k) return c;
  // four yf a workgroup: a batch that would leave CUs without a workgroup
  // splits the xb range (partial Yt in the QR's scratch, P slots of which
  // the shapes above 32 rows have, summed by k_sum_parts)
  if (c.TY > 1 && f.t1) {
    const long sel = f.tile_items > 0 ? f.tile_items : f.items;
    const long wgs = sel * ((f.K + c.TY - 1) / c.TY);
    c.nsplit = (int)std::max<long>(1, std::min<long>(std::min(16, f.P), 256 / wgs));
  }
  return c;
}

static hipError_t launch_fused(const FitBatch &f, int c, int j, bool rl, Ptr X,
                               Ptr F, Ptr G, Ptr Y, bool do_local, int TY,
                               int TX, size_t lds, hipStream_t st) {
  static std::once_flag attr_once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [] {
    for (int D : {0, 2, 3, 4, 5, 6})
      for (VisitKernel kf : {visit_kernel<double>(D), visit_kernel<float>(D),
                             visit_kernel<float, true>(D)}) {
        hipError_t e = hipFuncSetAttribute((const void *)kf,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) attr_err = e;
      }
    for (auto t : {std::make_pair(2, 4), std::make_pair(4, 2), std::make_pair(2, 2),
                   std::make_pair(1, 2), std::make_pair(1, 1)})
      for (VisitKernel kf : {visit4_kernel<double>(t.first, t.second),
                             visit4_kernel<float>(t.first, t.second)}) {
        hipError_t e = hipFuncSetAttribute((const void *)kf,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) attr_err = e;
      }
    for (int D : {2, 3, 5, 6})
      for (int ne = 1; ne <= 4; ++ne) {
        hipError_t e = hipFuncSetAttribute((const void *)visitp_kernel(D, ne).k,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) attr_err = e;
      }
    for (int ne = 2; ne <= 4; ++ne)
      for (VisitKernel kf : {visit4p_kernel<double>(ne, 2), visit4p_kernel<float>(ne, 2),
                             visit4p_kernel<double>(ne, 1), visit4p_kernel<float>(ne, 1)}) {
        hipError_t e = hipFuncSetAttribute(
            (const void *)kf, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) attr_err = e;
      }
  });
  if (attr_err != hipSuccess) return attr_err;
  int TY4, TX4;
  size_t lds4;
  const bool b16 = visit_bf16(f), f32 = visit_f32(f);
  const bool spec = !b16 && (f32 ? visit4_tiles<float>(f, &TY4, &TX4, &lds4)
                                 : visit4_tiles<double>(f, &TY4, &TX4, &lds4));
  const size_t site_off = ((size_t)(j - 1) * f.W + c) * a_site(f);
  VisitArgs v;
  v.K = f.K; v.P = f.P; v.D = f.D; v.d = f.d; v.TY = TY; v.TX = TX;
  v.rl = rl ? 1 : 0;
  v.do_local = do_local ? 1 : 0;
  v.F = F; v.X = X; v.G = G; v.Y = Y;
  v.aket = f.acan + site_off;
  v.aket_stride = a_stride(f);
  v.abra = f.bra_one ? f.bra_one : (f.abra ? f.abra : f.acan) + site_off;
  v.abra_stride = f.bra_one ? 0 : a_stride(f);
  v.t3 = f.t3;
  v.t3_stride = t1_stride(f);
  v.dims = v.order = nullptr;
  v.W = f.W; v.c = c; v.j = j; v.N = f.N;
  const double it = f.items, K = f.K, P = f.P, d = f.d;
  double flops = it * (2 * K * K * K * P * P + 4 * d * K * K * P * P * P);
  double bytes = it * 8 * (2 * K * P * K + K * K * P * P + 2 * d * P * P);
  if (do_local) {
    flops += it * 2 * K * K * K * P * P;
    bytes += it * 8 * 2 * K * P * K;
  }
  const Count tc = count_inner(f, c, j, rl, TC_T1 | TC_KET | TC_BRA | (do_local ? TC_LOCAL : 0));
  Span sp(KC_VISIT, st, tc.flops, tc.bytes, flops, bytes);
  int TYp, TXp;
  size_t ldsp;
  const bool pairw = !b16 && (f32 ? visit4p_tiles<float>(f, &TYp, &TXp, &ldsp)
                                  : visit4p_tiles<double>(f, &TYp, &TXp, &ldsp));
  if (pairw) {  // one (yf, xb) pair per wave; skips the zero padding
    v.TY = TYp;
    v.TX = TXp;
    (f.bounded ? v.dims : v.order) = f.hdims ? f.dims : nullptr;
    const int ne = visit4p_ne(f.K);
    hipLaunchKernelGGL(f32 ? visit4p_kernel<float>(ne, TYp) : visit4p_kernel<double>(ne, TYp),
                       dim3((f.K + TYp - 1) / TYp, f.items), dim3(64 * TYp * TXp), ldsp, st, v);
  } else if (spec) {
    v.TY = TY4;
    v.TX = TX4;
    hipLaunchKernelGGL(f32 ? visit4_kernel<float>(TY4, TX4) : visit4_kernel<double>(TY4, TX4),
                       dim3((f.K + TY4 - 1) / TY4, f.items), dim3(kVisitThreads), lds4, st, v);
  } else if (const VisitPChoice vp = b16 || f32 ? VisitPChoice{} : visitp_tiles(f); vp.k) {
    v.dims = f.bounded && f.hdims ? f.dims : nullptr;
    VisitPArgs g{v, vp.nsplit, f.t1, t1_stride(f), f.hdims ? f.dims : nullptr};
    hipLaunchKernelGGL(vp.k, dim3((f.K + vp.TY - 1) / vp.TY * g.nsplit, f.items),
                       dim3(vp.threads), vp.lds, st, g);
    if (do_local && g.nsplit > 1)
      hipLaunchKernelGGL(k_sum_parts, dim3((f.K * f.P * f.K + kThreads - 1) / kThreads, f.items), dim3(kThreads), 0, st, Y,
                         (const double *)f.t1, t1_stride(f), g.nsplit, (size_t)f.K * f.P * f.K);
  } else {
    const VisitKernel kf = b16   ? visit_kernel<float, true>(f.D)
                           : f32 ? visit_kernel<float>(f.D)
                                 : visit_kernel<double>(f.D);
    hipLaunchKernelGGL(kf, dim3((f.K + TY - 1) / TY, f.items), dim3(kVisitThreads), lds, st, v);
  }
  return hipGetLastError();
}

bool visit_fused_fits(const FitBatch &f) {
  int TY, TX;
  size_t lds;
  visit_tiles(f, &TY, &TX, &lds);
  return TY > 0;
}

// Blocked MFMA QR (8 waves) for panels up to 768 x 48: row tiles per wave and
// column tiles from the bond cap K and the physical dimension P.
constexpr int kQmWavesUsed = 8;

bool qrm_fits(const FitBatch &f) {
  return f.K <= 48 && f.K * f.P <= 16 * kQmWavesUsed * 6;
}

bool qr_needs_scratch(const FitBatch &f) {
  if (qrm_fits(f)) return false;
  return (size_t)f.K * f.P * f.K > (size_t)kQrLds;
}

template <int NW, int RT, int CT>
void launch_qrm_as(int items, hipStream_t st, const QrArgs &q) {
  hipLaunchKernelGGL((k_qrm<NW, RT, CT>), dim3(items), dim3(NW * 64), 0, st, q);
}

template <int RT>
void launch_qrm_rt(int CT, int items, hipStream_t st, const QrArgs &q) {
  constexpr int NW = kQmWavesUsed;
  if (CT == 1) launch_qrm_as<NW, RT, 1>(items, st, q);
  else if (CT == 2) launch_qrm_as<NW, RT, 2>(items, st, q);
  else launch_qrm_as<NW, RT, 3>(items, st, q);
}

void launch_qrm(const FitBatch &f, hipStream_t st, const QrArgs &q) {
  const int m = f.K * f.P, CT = (f.K + 15) / 16;
  // Up to 256 x 16 four waves, one per SIMD: what every wave issues for itself
  // in a step is then issued once per SIMD (135 x 15: 10.1 us, with eight waves
  // 11.4).  Larger panels share their tiles' work over eight (512 x 32: 85600
  // cycles with four, 82200 with eight).
  if (CT == 1 && m <= 256) {
    if (m <= 64) launch_qrm_as<4, 1, 1>(f.items, st, q);
    else if (m <= 128) launch_qrm_as<4, 2, 1>(f.items, st, q);
    else launch_qrm_as<4, 4, 1>(f.items, st, q);
    return;
  }
  const int rt = (m + 16 * kQmWavesUsed - 1) / (16 * kQmWavesUsed);
  if (rt <= 1) launch_qrm_rt<1>(CT, f.items, st, q);
  else if (rt <= 2) launch_qrm_rt<2>(CT, f.items, st, q);
  else if (rt <= 4) launch_qrm_rt<4>(CT, f.items, st, q);
  else launch_qrm_rt<6>(CT, f.items, st, q);
}

// One column tile per workgroup, a launch per block and one for Q: panels of
// up to 3072 rows (24 row tiles a wave, all the registers hold) whose scratch
// is there.  CT + 1 launches instead of one, but each reads the panel once per
// 16 columns where k_qrg reads it per column.
template <int RT>
void launch_qrb_rt(QrbArgs g, int items, hipStream_t st) {
  for (g.b = 0; g.b < g.CT; ++g.b)
    hipLaunchKernelGGL((k_qrb_factor<RT>), dim3(items, g.b ? g.CT - g.b : 1),
                       dim3(kQrbWaves * 64), 0, st, g);
  hipLaunchKernelGGL((k_qrb_q<RT>), dim3(items, g.CT), dim3(kQrbWaves * 64), 0, st, g);
}

bool qrb_fits(const FitBatch &f) {
  return f.K * f.P <= 16 * kQrbWaves * 24 && f.K <= 16 * kQrbWaves &&
         qrb_words(f.K, f.P) <= t1_stride(f);
}

void launch_qrb(const FitBatch &f, hipStream_t st, const QrArgs &q) {
  QrbArgs g{q, 0, (f.K + 15) / 16, (f.K * f.P + 15) / 16};
  const int rt = (g.MT + kQrbWaves - 1) / kQrbWaves;
  if (rt <= 4) launch_qrb_rt<4>(g, f.items, st);
  else if (rt <= 8) launch_qrb_rt<8>(g, f.items, st);
  else if (rt <= 12) launch_qrb_rt<12>(g, f.items, st);
  else if (rt <= 18) launch_qrb_rt<18>(g, f.items, st);
  else launch_qrb_rt<24>(g, f.items, st);
}

hipError_t launch_inner_visit(const FitBatch &f, int c, int j, bool rl, Ptr X,
                              Ptr F, Ptr G, Ptr Y, hipStream_t st) {
  int TY, TX;
  size_t lds;
  visit_tiles(f, &TY, &TX, &lds);
  if (TY > 0) return launch_fused(f, c, j, rl, X, F, G, Y, true, TY, TX, lds, st);
  hipError_t e = launch_inner_chain_generic(f, c, j, rl, X, F, st);
  if (e != hipSuccess) return e;
  return launch_inner_local(f, c, j, rl, G, Y, st);
}

hipError_t launch_inner_chain(const FitBatch &f, int c, int j, bool rl, Ptr X,
                              Ptr F, hipStream_t st) {
  int TY, TX;
  size_t lds;
  visit_tiles(f, &TY, &TX, &lds);
  if (TY > 0)
    return launch_fused(f, c, j, rl, X, F, Ptr{}, Ptr{}, false, TY, TX, lds, st);
  return launch_inner_chain_generic(f, c, j, rl, X, F, st);
}

hipError_t launch_inner_chain_generic(const FitBatch &f, int c, int j, bool rl,
                                      Ptr X, Ptr F, hipStream_t st) {
  const Shape s = shape_of(f);
  const size_t t1s = t1_stride(f), t2s = t2_stride(f), t3s = t1s;
  const size_t site_off = ((size_t)(j - 1) * f.W + c) * a_site(f);
  const double *Ak = f.acan + site_off;
  const double *Ab = f.bra_one ? f.bra_one : (f.abra ? f.abra : f.acan) + site_off;
  const double it = f.items, K = f.K, P = f.P, d = f.d;
  OpK1 k1{f.K * f.P, f.P * f.K, f.K, nullptr, s, rl, X, F, f.t1, t1s};
  hipError_t e;
  {
    const Count tc = count_inner(f, c, j, rl, TC_T1);
    Span sp(KC_T1, st, tc.flops, tc.bytes, it * 2 * K * P * P * K * K,
            it * 8 * (2 * K * P * K + K * K * P * P));
    e = run_gemm<64, 64, 16>(k1, f.items, st);
  }
  if (e != hipSuccess) return e;
  OpK2 k2{f.K * f.P * f.K, f.d * f.P, f.P, nullptr, s, rl, f.t1, t1s, Ak,
          a_stride(f), f.t2, t2s};
  {
    const Count tc = count_inner(f, c, j, rl, TC_KET);
    Span sp(KC_KET, st, tc.flops, tc.bytes, it * 2 * K * P * K * d * P * P,
            it * 8 * (K * K * P * P + d * P * P + d * K * K * P * P));
    e = run_gemm<128, 32, 16>(k2, f.items, st);
  }
  if (e != hipSuccess) return e;
  OpK3 k3{f.K * f.K * f.P, f.P, f.d * f.P, nullptr, s, rl, f.t2, t2s, Ab,
          f.bra_one ? 0 : a_stride(f), f.t3, t3s};
  const Count tc = count_inner(f, c, j, rl, TC_BRA);
  Span sp(KC_BRA, st, tc.flops, tc.bytes, it * 2 * K * K * P * P * d * P,
          it * 8 * (d * K * K * P * P + d * P * P + K * K * P * P));
  return run_gemm<256, 16, 16>(k3, f.items, st);
}

hipError_t launch_inner_local(const FitBatch &f, int c, int j, bool rl, Ptr G, Ptr Y,
                              hipStream_t st) {
  OpK4 k4{f.K * f.P, f.K, f.K * f.P, nullptr, shape_of(f), rl, f.t3,
          t1_stride(f), G, Y};
  const double it = f.items, K = f.K, P = f.P;
  const Count tc = count_inner(f, c, j, rl, TC_LOCAL);
  Span sp(KC_LOCAL, st, tc.flops, tc.bytes, it * 2 * K * P * K * K * P,
          it * 8 * (K * K * P * P + 2 * K * P * K));
  return run_gemm<64, 32, 16>(k4, f.items, st);
}

hipError_t launch_inner_env(const FitBatch &f, int c, int j, bool rl, Ptr Y,
                            Ptr envOut, hipStream_t st) {
  const double it = f.items, K = f.K, P = f.P;
  const Count tc = count_inner(f, c, j, rl, TC_ENV);
  Span sp(KC_ENV, st, tc.flops, tc.bytes, it * 2 * K * K * P * K * P,
          it * 8 * (K * K * P * P + 2 * K * P * K));
  if (f.K <= 64) {
    EnvArgs e{f.K, f.P, rl ? 1 : 0, f.t3, t1_stride(f), Y, envOut,
              f.bounded && f.hdims ? f.dims : nullptr, f.W, c, j, f.N};
    const dim3 grid((f.K * f.P + 63) / 64, f.items);
    const int mt = (f.K + 15) / 16;
    // BF16 or FP32 only where the visit wrote FP32 T3
    if (visit_bf16(f)) {
      if (mt <= 1) hipLaunchKernelGGL((k_env<1, float, true>), grid, dim3(EnvShape<1>::kThreads), 0, st, e);
      else if (mt <= 2) hipLaunchKernelGGL((k_env<2, float, true>), grid, dim3(EnvShape<2>::kThreads), 0, st, e);
      else if (mt <= 3) hipLaunchKernelGGL((k_env<3, float, true>), grid, dim3(EnvShape<3>::kThreads), 0, st, e);
      else hipLaunchKernelGGL((k_env<4, float, true>), grid, dim3(EnvShape<4>::kThreads), 0, st, e);
      return hipGetLastError();
    }
    if (visit_f32(f)) {
      if (mt <= 1) hipLaunchKernelGGL((k_env<1, float>), grid, dim3(EnvShape<1>::kThreads), 0, st, e);
      else if (mt <= 2) hipLaunchKernelGGL((k_env<2, float>), grid, dim3(EnvShape<2>::kThreads), 0, st, e);
      else if (mt <= 3) hipLaunchKernelGGL((k_env<3, float>), grid, dim3(EnvShape<3>::kThreads), 0, st, e);
      else hipLaunchKernelGGL((k_env<4, float>), grid, dim3(EnvShape<4>::kThreads), 0, st, e);
      return hipGetLastError();
    }
    // The shape for small batches takes twice the workgroups and one fills a
    // CU: up to 128 workgroups of the other a launch it is the faster one (the
    // two in us: 120 of K = 17, D = 4 14.5 and 12.3; 120 of K = 40 33.6 and
    // 26.2; 128 of K = 64 54 and 39), beyond the slower one (136 of K = 32 21.0
    // and 24.0; 168 of K = 48 38.6 and 44.8; 224 of K = 64 69 and 77).  From 16
    // messages on a shape's batch is launched in two halves by default.
    const long sel = f.tile_items > 0 ? f.tile_items : f.items;
    const long wgs = sel * grid.x;
    if (mt > 1 && (sel < 16 ? wgs <= 128 : wgs < 256)) {
      const dim3 half((f.K * f.P + 31) / 32, f.items);
      if (mt <= 2) hipLaunchKernelGGL((k_env<2, double, false, false>), half, dim3(EnvShape<2, false>::kThreads), 0, st, e);
      else if (mt <= 3) hipLaunchKernelGGL((k_env<3, double, false, false>), half, dim3(EnvShape<3, false>::kThreads), 0, st, e);
      else hipLaunchKernelGGL((k_env<4, double, false, false>), half, dim3(EnvShape<4, false>::kThreads), 0, st, e);
      return hipGetLastError();
    }
    if (mt <= 1) hipLaunchKernelGGL((k_env<1, double>), grid, dim3(EnvShape<1>::kThreads), 0, st, e);
    else if (mt <= 2) hipLaunchKernelGGL((k_env<2, double>), grid, dim3(EnvShape<2>::kThreads), 0, st, e);
    else if (mt <= 3) hipLaunchKernelGGL((k_env<3, double>), grid, dim3(EnvShape<3>::kThreads), 0, st, e);
    else hipLaunchKernelGGL((k_env<4, double>), grid, dim3(EnvShape<4>::kThreads), 0, st, e);
    return hipGetLastError();
  }
  OpK5 k5{f.K, f.K * f.P, f.K * f.P, nullptr, shape_of(f), rl, f.t3,
          t1_stride(f), Y, envOut};
  return run_gemm<32, 64, 16>(k5, f.items, st);
}

hipError_t launch_end_chain(const FitBatch &f, int c, bool rl, Ptr Mend, Ptr Xe,
                            hipStream_t st) {
  OpE1 e1{f.K * f.P, f.K, f.K, nullptr, shape_of(f), rl, Mend, Xe, f.t3,
          t1_stride(f)};
  const double it = f.items, K = f.K, P = f.P;
  const Count tc = count_end(f, c, rl, 1);
  Span sp(KC_END, st, tc.flops, tc.bytes, it * 2 * K * P * K * K,
          it * 8 * (2 * K * P * K + K * K));
  return run_gemm<64, 32, 16>(e1, f.items, st);
}

hipError_t launch_end_local(const FitBatch &f, int c, bool rl, Ptr G, Ptr Ye,
                            hipStream_t st) {
  OpE2 e2{f.K, f.K, f.P * f.K, nullptr, shape_of(f), rl, f.t3, t1_stride(f),
          G, Ye};
  const double it = f.items, K = f.K, P = f.P;
  const Count tc = count_end(f, c, rl, 2);
  Span sp(KC_END, st, tc.flops, tc.bytes, it * 2 * K * K * P * K,
          it * 8 * (2 * K * P * K + K * K));
  // one 32x32 tile, K P long: split over eight (P >= 8) workgroups per tile
  // through the item's tmp slot (K P K doubles >= 8 K^2), which nothing
  // else holds at this point of a column
  if (f.P >= 8 && f.tmp) return run_gemm_splitk<32, 32, 64, 8>(e2, f.items, f.tmp, f.S, st);
  return run_gemm<32, 32, 64>(e2, f.items, st);
}

hipError_t launch_end_env(const FitBatch &f, int c, bool rl, Ptr Ye, Ptr envOut,
                          hipStream_t st) {
  OpE3 e3{f.K, f.P * f.K, f.K, nullptr, shape_of(f), rl, f.t3, t1_stride(f),
          Ye, envOut};
  const double it = f.items, K = f.K, P = f.P;
  const Count tc = count_end(f, c, rl, 4);
  Span sp(KC_END, st, tc.flops, tc.bytes, it * 2 * K * P * K * K,
          it * 8 * (2 * K * P * K + K * K));
  return run_gemm<32, 64, 16>(e3, f.items, st);
}

hipError_t launch_qr(const FitBatch &f, int c, int j, int mode, Ptr Y,
                     bool want_r, bool only_flagged, hipStream_t st) {
  QrArgs q{f.dims, f.W, c, j, mode, f.K, f.P, Y, f.rbuf, f.t1, t1_stride(f),
           only_flagged ? f.flag : nullptr, want_r ? 1 : 0};
  const size_t panel = (size_t)f.K * f.P * f.K;  // upper bound of m*n
  const double m = (double)f.K * f.P, n = f.K;
  const Count tc = count_qr(f, c, j, mode);
  Span sp(KC_QR, st, tc.flops, tc.bytes, f.items * (4.0 * m * n * n - 4.0 * n * n * n / 3.0),
          f.items * 16.0 * m * n);
  // The blocked MFMA kernel for panels up to 768 x 48 (every shape of the
  // D <= 4 workloads); otherwise the LDS kernel, or through the global scratch
  // a workgroup per column tile up to 3072 rows and the 16-wave kernel beyond
  // (up to 128 columns: every bond cap the context accepts).
  if (qrm_fits(f)) {
    launch_qrm(f, st, q);
  } else if (panel <= (size_t)kQrLds) {
    hipLaunchKernelGGL(k_qr, dim3(f.items), dim3(kThreads), 0, st, q);
  } else {
    if (!f.t1 || t1_stride(f) < panel)
      return hipErrorInvalidValue;  // global panel scratch missing or too small
    if (qrb_fits(f)) {
      launch_qrb(f, st, q);
      return hipGetLastError();
    }
    if (f.K > kQrgWaves * kQrgCols) return hipErrorInvalidValue;  // bond caps are <= 128
    hipLaunchKernelGGL(k_qrg, dim3(f.items), dim3(kQrgThreads), 0, st, q);
  }
  (void)panel;
  return hipGetLastError();
}

// One launch for every visit of columns col_hi .. col_lo where the shape fits
// k_absorb_small: D = 2, d = 2, FP64 and the LDS of one workgroup (bond caps up
// to 20), whatever the batch.  One item per CU from cap 17 on: a sweep of 8, 48,
// 224 and 960 messages at cap 20 takes 1.4, 2.6, 2.8 and 10.0 ms, launched one
// by one 3.5, 5.1, 14.5 and 56.6 ms; at cap 9 0.9, 1.2, 1.5 and 2.9 against 2.5,
// 2.9, 5.7 and 20.1.
static size_t small_lds(int K) {
  return 8 * (K <= 8    ? SmallShape<1, 1>::words(K)
              : K <= 16 ? SmallShape<1, 4>::words(K)
                        : SmallShape<2, 4>::words(K));
}
bool absorb_small_fits(const FitBatch &f) {
  return f.D == 2 && f.d == 2 && f.prec == 64 && f.K <= 32 && f.N >= 3 &&
         small_lds(f.K) + 4096 <= 160 * 1024;
}
// Counts of column c in k_absorb_small, true and at the bond cap: the
// contractions and QRs of every visit, and the bytes that the kernel itself
// loads and stores (T3, an end visit's G and the environment handed to the next
// visit stay in LDS).
static void count_small(const FitBatch &f, int c, int n_fit, Count *t, Count *pad) {
  if (!timing_enabled()) return;
  const int N = f.N;
  const double P = f.P, site = 2.0 * f.d * P * P;
  auto count = [&](const FitDims *d, const FitDims *next, bool rnd) {
    const double K = f.K;
    Count s;
    auto qr = [&](double m, double n) { s.flops += 4.0 * m * n * n - 4.0 * n * n * n / 3.0; };
    auto visit = [&](int j, bool rl, bool local, bool env) {
      double yf = K, yb = K, xf = K, xb = K, m = 0.0, b = 0.0;
      if (d) {
        const SiteExt e = site_ext(*d, j, N, rl);
        yf = e.yf, yb = e.yb, xf = e.xf, xb = e.xb;
      }
      const bool end = j == 0 || j == N - 1;
      if (end) {
        const double a = d ? d->p[j] : K, ap = d ? (c == f.W - 1 ? 1 : next->p[j]) : K;
        m += a * P * ap * xb + (local ? a * P * xb * yb : 0.0) +
             (env ? yb * a * P * xb : 0.0);
        b += a * P * ap + ap * xb + a * yb;  // message site, X, Y
        if (local && env) qr(d ? a : K * P, yb);
      } else {
        m += yf * P * xf * P * xb + 2.0 * yf * xb * f.d * P * P * P +
             (local ? 2.0 : 1.0) * yf * P * xb * P * yb;
        b += xf * P * xb + site + yf * P * yb;  // X, ket and bra, Y
        if (local) {
          b += yb * P * xb;  // G
          qr(yf * P, yb);
        }
      }
      const int jn = rl ? j - 1 : j + 1;
      if (env && jn > 0 && jn < N - 1) b += yb * P * xb;  // kept for the sweep back
      s.flops += 2.0 * m;
      s.bytes += 8.0 * b;
    };
    for (int j = N - 1; j >= 1; --j) visit(j, true, false, true);
    for (int k = 0; k < n_fit; ++k) {
      for (int j = 0; j < N - 1; ++j) visit(j, false, true, true);
      for (int j = N - 1; j >= 1; --j) visit(j, true, true, true);
    }
    visit(0, false, true, false);
    if (rnd)  // the start: each site made, factorised and stored
      for (int j = N - 1; j >= 1; --j) {
        const double m = d ? (double)d->p[j] * d->br[j] : K * P, n = d ? d->bl[j] : K;
        qr(m, n);
        s.bytes += 8.0 * m * n;
      }
    return s;
  };
  const Count cap = count(nullptr, nullptr, false), cap_rnd = count(nullptr, nullptr, true);
  for (int i = 0; i < f.items; ++i) {
    const FitDims *d = f.hdims ? f.hdims + (size_t)i * f.W + c : nullptr;
    const Count &y = d && d->rnd ? cap_rnd : cap, x = d ? count(d, d + 1, d->rnd) : y;
    t->flops += x.flops;
    t->bytes += x.bytes;
    pad->flops += y.flops;
    pad->bytes += y.bytes;
  }
}
hipError_t launch_absorb_small(const FitBatch &f, int col_hi, int col_lo, int n_fit,
                               hipStream_t st) {
  static std::once_flag once;
  static hipError_t attr = hipSuccess;
  std::call_once(once, [] {
    for (const void *k : {(const void *)k_absorb_small<1, 1>, (const void *)k_absorb_small<1, 4>,
                          (const void *)k_absorb_small<2, 4>}) {
      const hipError_t e =
          hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 156 * 1024);
      if (e != hipSuccess) attr = e;
    }
  });
  if (attr != hipSuccess) return attr;
  Count t, pad;
  for (int c = col_lo; c <= col_hi; ++c) count_small(f, c, n_fit, &t, &pad);
  Span sp(KC_VISIT, st, t.flops, t.bytes, pad.flops, pad.bytes);
  SmallArgs g{f, col_lo, col_hi, n_fit};
  const size_t lds = small_lds(f.K);
  const auto k = f.K <= 8    ? k_absorb_small<1, 1>
                 : f.K <= 16 ? k_absorb_small<1, 4>
                             : k_absorb_small<2, 4>;
  hipLaunchKernelGGL(k, dim3(f.items), dim3(256), lds, st, g);
  return hipGetLastError();
}

hipError_t launch_apply_l(const FitBatch &f, bool end_site, Ptr Y,
                          hipStream_t st) {
  const int rows = end_site ? f.K : f.K * f.P;
  OpApplyL op{rows, f.K, f.K, f.flag, shape_of(f), Y, f.rbuf, f.tmp, f.S};
  hipError_t e = run_gemm<64, 32, 16>(op, f.items, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_copy_flagged, dim3(64, f.items), dim3(kThreads), 0, st,
                     (const double *)f.tmp, f.S, Y, f.S, (const int32_t *)f.flag);
  return hipGetLastError();
}

hipError_t launch_rand_init(const FitBatch &f, int c, Ptr Ybase,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_rand_init, dim3(f.N, f.items), dim3(kThreads), 0, st,
                     f.dims, f.W, c, f.N, f.K, f.P, f.S, Ybase,
                     (const uint64_t *)f.slot, f.seed, (const int32_t *)f.flag);
  return hipGetLastError();
}

__global__ void k_zero_words(uint32_t *p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<size_t>(1024, (n + kThreads - 1) / kThreads);
  hipLaunchKernelGGL(k_zero_words, dim3(blocks), dim3(kThreads), 0, st, (uint32_t *)p, n);
  return hipGetLastError();
}

hipError_t launch_set_unit(const FitBatch &f, Ptr slot, hipStream_t st) {
  hipLaunchKernelGGL(k_set_unit, dim3(16, f.items), dim3(kThreads), 0, st,
                     slot, f.S);
  return hipGetLastError();
}

hipError_t launch_normalize(const FitBatch &f, int c, Ptr Y0, hipStream_t st) {
  hipLaunchKernelGGL(k_normalize, dim3(f.items), dim3(kThreads), 0, st, Y0,
                     f.K, f.nu + c, f.W, f.err);
  return hipGetLastError();
}

hipError_t launch_gather(const FitBatch &f, const GatherSrc *srcs,
                         hipStream_t st) {
  const int nx = f.N > f.W ? f.N : f.W;
  hipLaunchKernelGGL(k_gather, dim3(nx, 3, f.items), dim3(kThreads), 0, st, f,
                     srcs);
  return hipGetLastError();
}

hipError_t launch_extract(const FitBatch &f, double *const *dst,
                          const int32_t *rev, hipStream_t st) {
  hipLaunchKernelGGL(k_extract, dim3(f.H, f.items), dim3(kThreads), 0, st, f,
                     dst, rev);
  return hipGetLastError();
}

hipError_t launch_copy_jobs(const CopyJob *jobs, int njobs, int K, int P,
                            hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_jobs, dim3(8, njobs), dim3(kThreads), 0, st, jobs,
                     K, P);
  return hipGetLastError();
}

hipError_t launch_dots(int items, const double *const *a,
                       const double *const *b, size_t n, double *out,
                       hipStream_t st) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_dots, dim3(items), dim3(kThreads), 0, st, a, b, n, out);
  return hipGetLastError();
}

hipError_t launch_overlap(int items, int K, int P, int L,
                          const double *const *a, const double *const *b,
                          double *E, double *U, double *out, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  const size_t S = (size_t)K * P * K;
  hipLaunchKernelGGL(k_ov_init, dim3(items), dim3(64), 0, st, E, K);
  for (int i = 0; i < L; ++i) {
    OpOv1 o1{K, P * K, K, nullptr, K, E, a, (size_t)i * S, U, S};
    hipError_t e = run_gemm<32, 64, 16>(o1, items, st);
    if (e != hipSuccess) return e;
    OpOv2 o2{K, K, K * P, nullptr, K, P, U, S, b, (size_t)i * S, E};
    e = run_gemm<32, 32, 64>(o2, items, st);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_ov_out, dim3((items + 63) / 64), dim3(64), 0, st, E, K,
                     items, out);
  return hipGetLastError();
}

}  // namespace bbp
