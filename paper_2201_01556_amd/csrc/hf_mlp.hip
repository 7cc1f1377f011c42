// Learned pruning scorer: a 12 -> 64 -> 64 -> 1 perceptron (ReLU hidden
// units, sigmoid output) that scores block-pair flow problems by the
// probability that refining them improves the cut, so that low-scoring
// problems can be skipped.  It replaces the fixed pruning rule of the paper
// (section "Parallel Active Block Scheduling", paragraph "Implementation
// Details": skip pairs with a small cut) and is trained on outcomes of the
// plain run-everything schedule.
//
// Hand-written FP32 kernels (the 64 x 64 products on FP32 matrix instructions;
// the whole network has 5,057 parameters):
//   k_log1p        log1p(features) in float64
//   k_norm_stats   their column mean and population deviation in float64 (one
//                  wave per column, in chunks of samples)
//   k_norm_apply   z-scored float features
//   k_fwd_bwd      one workgroup per tile of 64 samples: forward pass with
//                  parameters and activations in LDS, mean binary
//                  cross-entropy on logits, backward pass, per-tile partial
//                  gradients (fixed summation order); without kGrad the
//                  forward pass only, sigmoid probabilities
//   k_reduce_adam  sum of the tile partials in tile order (deterministic),
//                  optional Adam step (Kingma and Ba)
//
// Parameter layout (row-major): W1 [64 x 12], b1 [64], W2 [64 x 64], b2 [64],
// W3 [64], b3.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "hf_host.h"

namespace hf {

constexpr int kIn = 12;
constexpr int kHid = 64;
constexpr int kTile = 64;  // samples per workgroup
constexpr int kMlpThreads = 512;
constexpr int oW1 = 0;
constexpr int ob1 = oW1 + kHid * kIn;    // 768
constexpr int oW2 = ob1 + kHid;          // 832
constexpr int ob2 = oW2 + kHid * kHid;   // 4928
constexpr int oW3 = ob2 + kHid;          // 4992
constexpr int ob3 = oW3 + kHid;          // 5056
constexpr int kParams = ob3 + 1;         // 5057
static_assert(kParams == FP_SCORER_PARAMS, "parameter count");
constexpr int kPart = (kParams + 1 + 3) & ~3;  // partial gradients, partial loss, 16-byte rows

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// one row of n values per feature column
__global__ void k_log1p(const int64_t* __restrict__ f, int n, double* __restrict__ lg) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n * kIn) lg[(size_t)(i % kIn) * n + i / kIn] = log1p((double)f[i]);
}

// One wave per feature column: mean, then the population deviation (two
// passes, float64); a deviation below 1e-9 counts as a constant column.  The
// order of the sums is fixed, so the twelve waves keep their serial chains;
// the logarithms, which were most of the time, come from k_log1p on the whole
// chip (12,000 samples: 289 -> 40 us for both kernels).
//
// The samples come in chunks of at most kFitChunk, so that the logarithms'
// buffer is bounded and k_log1p's indices fit 32 bits at any number of
// samples.  kFitChunk is a multiple of 64: every lane goes on with its own
// sums, which wait in acc (sum, squares per lane) between the chunks, and the
// results are those of one chunk.  pass: 1 the sums, 2 the squared
// differences, 3 both (all samples in one chunk).
constexpr int kFitChunk = 1 << 22;
static_assert(kFitChunk % 64 == 0 && (long long)kFitChunk * kIn < (1ll << 31), "chunk of samples");

__global__ void __launch_bounds__(kIn * 64) k_norm_stats(const double* __restrict__ lg, int n,
                                                         int total, int pass, int first, int last,
                                                         double* __restrict__ acc,
                                                         double* __restrict__ ms) {
  const int col = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double* row = lg + (size_t)col * n;
  double s = 0.0, mean = 0.0;
  if (pass & 1) {
    if (!first) s = acc[threadIdx.x];
#pragma unroll 16
    for (int i = lane; i < n; i += 64) s += row[i];
    acc[threadIdx.x] = s;
    mean = wave_sum_f64(s) / (double)total;
  } else {
    mean = wave_sum_f64(acc[threadIdx.x]) / (double)total;
  }
  if (!(pass & 2)) return;
  double* const squares = acc + kIn * 64;
  double q = first ? 0.0 : squares[threadIdx.x];
#pragma unroll 16
  for (int i = lane; i < n; i += 64) {
    const double d = row[i] - mean;
    q += d * d;
  }
  if (!last) {
    squares[threadIdx.x] = q;
    return;
  }
  const double sd = sqrt(wave_sum_f64(q) / (double)total);
  if (lane == 0) {
    ms[col] = mean;
    ms[kIn + col] = sd > 1e-9 ? sd : 1.0;
  }
}

__global__ void k_norm_apply(const int64_t* __restrict__ f, int n, const double* __restrict__ ms,
                             float* __restrict__ x) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)n * kIn) return;
  const int col = (int)(i % kIn);
  x[i] = (float)((log1p((double)f[i]) - ms[col]) / ms[kIn + col]);
}

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kLd = 72;  // row stride of the 64 x 64 LDS matrices: 16-byte rows, and both ways
                         // of reading an operand (along and across the rows) meet at most two
                         // lanes per bank

// One wave's 16 x (16 * N) outputs by matrix instructions: c[n] += sum over
// k of A(row, k) * B(16 n + col, k), k ascending.  An operand's element (i, k)
// lies at p[i * si + k * sk].  Lane l supplies element (l & 15, k0 + (l >> 4))
// of both operands of a 16 x 16 x 4 instruction and holds rows
// 4 (l >> 4) .. + 3 of column l & 15 of the result.  The instruction adds its
// four products one after another, each rounded like a fused multiply-add
// (checked against such a chain in k order: no bit differs).
template <int K, int N>
__device__ __forceinline__ void mm_16(const float* a, int sia, int ska, const float* b, int sib,
                                      int skb, f4 (&c)[N]) {
  const int r = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
  const float* ap = a + r * sia + q * ska;
  const float* bp = b + r * sib + q * skb;
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 4) {
    const float x = ap[k0 * ska];
#pragma unroll
    for (int n = 0; n < N; ++n)
      c[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, bp[n * 16 * sib + k0 * skb], c[n], 0, 0, 0);
  }
}

// Forward (and with kGrad the backward) pass over one tile of samples;
// with kGrad x holds the normalized samples, else they are computed here from
// the raw features f.  A tile is three 64 x 64 x 64 products (two of them
// backward) and a few sums between barriers, one workgroup per CU, so it is
// bound by latency and LDS reads: the products run on FP32 matrix
// instructions (eight waves of 16 units x 32 samples, operands read straight
// from one row-major copy of each matrix), the loss is one term per sample,
// and the short serial sums go to different waves.  Every sum keeps its order
// (k ascending, one accumulator); parameters, gradients and losses of 200
// training steps were those of the scalar form bit for bit.  The first form, in which a lane read its own row of W2 (64 lanes
// on one LDS bank) and one thread recomputed every sample's logit for the
// loss, took 70.8 us a step (12,000 samples, 188 tiles), 4 x 4 register tiles
// of vector multiply-adds 21.1, this one 11.9; 500 predictions 14.3 + 4.5
// (normalization), now 6.2 to 9.5.
template <bool kGrad>
__global__ void __launch_bounds__(kMlpThreads)
    k_fwd_bwd(const float* __restrict__ prm, const float* __restrict__ x,
              const int64_t* __restrict__ f, const double* __restrict__ ms,
              const float* __restrict__ y, int n, float inv_n, float* __restrict__ part,
              float* __restrict__ prob) {
  __shared__ __attribute__((aligned(16))) float W1[kHid * kIn];       // [unit][input]
  __shared__ __attribute__((aligned(16))) float X[kTile * kIn + 16];  // [sample][input]
  __shared__ __attribute__((aligned(16))) float W2[kHid * kLd];       // [unit][input]
  __shared__ __attribute__((aligned(16))) float H1[kTile * kLd];      // [sample][unit]
  __shared__ __attribute__((aligned(16))) float H2[kTile * kLd];      // [sample][unit]; then D1
  __shared__ __attribute__((aligned(16))) float D2[kGrad ? kTile * kLd : 4];  // dL/dz2
  __shared__ __attribute__((aligned(16))) float B1[kHid], B2[kHid], W3[kHid];
  __shared__ float DZ[kTile], LS[kTile];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6;
  const int s0 = blockIdx.x * kTile;
  const int ns = min(kTile, n - s0);
  const float b3 = prm[ob3];
  for (int i = tid; i < kHid * kHid / 4; i += kMlpThreads)
    *reinterpret_cast<float4*>(W2 + (i >> 4) * kLd + (i & 15) * 4) =
        *reinterpret_cast<const float4*>(prm + oW2 + i * 4);
  for (int i = tid; i < kHid * kIn; i += kMlpThreads) {
    W1[i] = prm[oW1 + i];
    float v = 0.f;
    if (i < ns * kIn) {
      if (kGrad) v = x[(size_t)s0 * kIn + i];
      else {
        const int col = i % kIn;
        v = (float)((log1p((double)f[(size_t)s0 * kIn + i]) - ms[col]) / ms[kIn + col]);
      }
    }
    X[i] = v;
  }
  if (tid < kHid) {
    B1[tid] = prm[ob1 + tid];
    B2[tid] = prm[ob2 + tid];
    W3[tid] = prm[oW3 + tid];
  } else if (tid < kHid + 16) {
    X[kTile * kIn + tid - kHid] = 0.f;  // read as inputs 12 .. 15 of the last sample
  }
  __syncthreads();
  const int u0 = (wid & 3) * 16;   // this wave's units
  const int m0 = (wid >> 2) * 32;  // its samples (or inputs)
  const int col = m0 + (lane & 15), row = u0 + (lane >> 4) * 4;
  f4 c[2];
  // c holds units row .. row + 3 of samples col and col + 16
  auto put_relu = [&](float* m) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int i = 0; i < 4; ++i) c[t][i] = c[t][i] > 0.f ? c[t][i] : 0.f;
      *reinterpret_cast<f4*>(m + (col + 16 * t) * kLd + row) = c[t];
    }
  };
  // layer 1
  c[0] = c[1] = *reinterpret_cast<const f4*>(B1 + row);
  mm_16<kIn>(W1 + u0 * kIn, kIn, 1, X + m0 * kIn, kIn, 1, c);
  put_relu(H1);
  __syncthreads();
  // layer 2
  c[0] = c[1] = *reinterpret_cast<const f4*>(B2 + row);
  mm_16<kHid>(W2 + u0 * kLd, kLd, 1, H1 + m0 * kLd, kLd, 1, c);
  put_relu(H2);
  __syncthreads();
  // output, dL/dz, loss term
  if (tid < kTile) {
    const int s = tid;
    float z = b3;
#pragma unroll
    for (int k = 0; k < kHid; k += 4) {
      const f4 h = *reinterpret_cast<const f4*>(H2 + s * kLd + k);
      const f4 w = *reinterpret_cast<const f4*>(W3 + k);
      z += w[0] * h[0];
      z += w[1] * h[1];
      z += w[2] * h[2];
      z += w[3] * h[3];
    }
    float dz = 0.f, term = 0.f;
    if (s < ns) {
      const float p = 1.f / (1.f + expf(-z));
      if (prob) prob[s0 + s] = p;
      if (kGrad) {
        const float yy = y[s0 + s];
        dz = (p - yy) * inv_n;
        // softplus(z) - y z (without overflow)
        const float sp = z > 0.f ? z + log1pf(expf(-z)) : log1pf(expf(z));
        term = sp - yy * z;
      }
    }
    DZ[s] = dz;
    LS[s] = term;
  }
  if (!kGrad) return;
  __syncthreads();
  float* out = part + (size_t)blockIdx.x * kPart;
  // dL/dz2 (c still holds H2)
  {
    const f4 w = *reinterpret_cast<const f4*>(W3 + row);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float dz = DZ[col + 16 * t];
#pragma unroll
      for (int i = 0; i < 4; ++i) c[t][i] = c[t][i] > 0.f ? dz * w[i] : 0.f;
      *reinterpret_cast<f4*>(D2 + (col + 16 * t) * kLd + row) = c[t];
    }
  }
  __syncthreads();
  // W2: units row .. row + 3, inputs col and col + 16, summed over the samples
  c[0] = c[1] = f4{0.f, 0.f, 0.f, 0.f};
  mm_16<kTile>(D2 + u0, 1, kLd, H1 + m0, 1, kLd, c);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) out[oW2 + (row + i) * kHid + col + 16 * t] = c[t][i];
  // dL/dz1 = (W2^T dz2) masked by layer 1: units row .. row + 3 of layer 1
  c[0] = c[1] = f4{0.f, 0.f, 0.f, 0.f};
  mm_16<kHid>(W2 + u0, 1, kLd, D2 + m0 * kLd, kLd, 1, c);
  // the sums over the samples of the output layer and of b2, and the loss,
  // in sample order, one wave each
  if (wid == 0) {
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < kTile; ++s) g += DZ[s] * H2[s * kLd + lane];
    out[oW3 + lane] = g;
  } else if (wid == 1) {
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < kTile; ++s) g += D2[s * kLd + lane];
    out[ob2 + lane] = g;
  } else if (tid == 128) {
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < kTile; ++s) g += DZ[s];
    out[ob3] = g;
  } else if (tid == 192) {
    float l = 0.f;
    for (int s = 0; s < ns; ++s) l += LS[s] * inv_n;
    out[kParams] = l;
  }
  __syncthreads();  // H2 is no longer needed
  float* const D1 = H2;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const f4 h = *reinterpret_cast<const f4*>(H1 + (col + 16 * t) * kLd + row);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[t][i] = h[i] > 0.f ? c[t][i] : 0.f;
    *reinterpret_cast<f4*>(D1 + (col + 16 * t) * kLd + row) = c[t];
  }
  __syncthreads();
  // W1 (16 units per wave; columns 12 .. 15 are not inputs), b1
  if (wid < 4) {
    f4 w1[1] = {f4{0.f, 0.f, 0.f, 0.f}};
    mm_16<kTile>(D1 + u0, 1, kLd, X, 1, kIn, w1);
    if ((lane & 15) < kIn)
#pragma unroll
      for (int i = 0; i < 4; ++i) out[oW1 + (row + i) * kIn + (lane & 15)] = w1[0][i];
  } else if (wid == 4) {
    float g = 0.f;
#pragma unroll 16
    for (int s = 0; s < kTile; ++s) g += D1[s * kLd + lane];
    out[ob1 + lane] = g;
  }
}

// Gradient = sum of the tile partials in tile order, 64 parameters per
// workgroup; with update, one Adam step (c1, c2 = bias corrections
// 1/(1 - beta^t)).  Bound by the latency of the partials' loads, since the
// order of the sum is fixed: the workgroup's waves bring the tiles to LDS side
// by side, kAhead loads in flight each, and one wave adds them in order (188
// tiles: 43.5 us with a thread walking its partials, 9.0 with 64 of them
// loaded ahead, now 4.6).
constexpr int kAdamWaves = 8;
constexpr int kAhead = 24;
constexpr int kAdamTiles = kAdamWaves * kAhead;  // tiles per pass through LDS
__global__ void __launch_bounds__(64 * kAdamWaves)
    k_reduce_adam(const float* __restrict__ part, int tiles, float* __restrict__ prm,
                  float* __restrict__ m, float* __restrict__ v, float* __restrict__ grad,
                  float* __restrict__ loss, int update, float lr, float b1, float b2, float eps,
                  float c1, float c2) {
  __shared__ float sums[kAdamTiles][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const bool mine = i <= kParams;
  float g = 0.f, m0 = 0.f, v0 = 0.f, p0 = 0.f;
  if (wid == 0 && update && i < kParams) {
    m0 = m[i];
    v0 = v[i];
    p0 = prm[i];
  }
  for (int t0 = 0; t0 < tiles; t0 += kAdamTiles) {
    const int nt = min(kAdamTiles, tiles - t0);
    float p[kAhead];
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int t = a * kAdamWaves + wid;
      p[a] = mine && t < nt ? part[(size_t)(t0 + t) * kPart + i] : 0.f;
    }
    __syncthreads();  // the previous tiles are summed
#pragma unroll
    for (int a = 0; a < kAhead; ++a) sums[a * kAdamWaves + wid][lane] = p[a];
    __syncthreads();
    if (wid == 0) {
#pragma unroll 16
      for (int t = 0; t < nt; ++t) g += sums[t][lane];
    }
  }
  if (wid != 0 || !mine) return;
  if (i == kParams) {
    if (loss) *loss = g;
    return;
  }
  if (grad) grad[i] = g;
  if (update) {
    // the rounding of each moment is written out: which product the compiler
    // would fuse into the sum depends on the code around it, and the last
    // bits of a step travel through all that follow
    const float mi = fmaf(1.f - b1, g, b1 * m0);
    const float vi = fmaf(g, (1.f - b2) * g, b2 * v0);
    m[i] = mi;
    v[i] = vi;
    prm[i] = p0 - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  }
}

}  // namespace hf

struct fp_scorer {
  int device = 0;
  void* mem = nullptr;  // params, m, v, grad, mean/std, loss
  float* prm = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  float* grad = nullptr;
  double* ms = nullptr;
  float* loss = nullptr;
  bool normalized = false;
  int step = 0;
};

namespace hf {

static size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

fp_status scorer_create_impl(const float* init, hipStream_t s, fp_scorer** out) {
  fp_scorer* sc = new (std::nothrow) fp_scorer();
  if (!sc) {
    set_error("host allocation failed");
    return FP_ERR_OOM;
  }
  for (int i = 0; i < kParams; ++i)
    if (!std::isfinite(init[i])) {
      delete sc;
      set_error("initial parameter %d is not finite", i);
      return FP_ERR_INVALID;
    }
  hipGetDevice(&sc->device);
  const size_t fp = al(kParams * sizeof(float));
  const size_t total = 4 * fp + al(2 * kIn * sizeof(double)) + al(sizeof(float));
  hipError_t he = hipMalloc(&sc->mem, total);
  if (he != hipSuccess) {
    delete sc;
    return hip_fail(he, "allocating the scorer");
  }
  char* p = static_cast<char*>(sc->mem);
  sc->prm = reinterpret_cast<float*>(p);
  sc->m = reinterpret_cast<float*>(p + fp);
  sc->v = reinterpret_cast<float*>(p + 2 * fp);
  sc->grad = reinterpret_cast<float*>(p + 3 * fp);
  sc->ms = reinterpret_cast<double*>(p + 4 * fp);
  sc->loss = reinterpret_cast<float*>(p + 4 * fp + al(2 * kIn * sizeof(double)));
  he = hipMemsetAsync(sc->mem, 0, total, s);
  if (he == hipSuccess)
    he = hipMemcpyAsync(sc->prm, init, kParams * sizeof(float), hipMemcpyHostToDevice, s);
  if (he == hipSuccess) he = hipStreamSynchronize(s);
  if (he != hipSuccess) {
    (void)hipFree(sc->mem);
    delete sc;
    return hip_fail(he, "initialising the scorer");
  }
  *out = sc;
  return FP_OK;
}

void scorer_destroy_impl(fp_scorer* sc) {
  if (sc->mem) (void)hipFree(sc->mem);
  delete sc;
}

// Device copies of features (and labels) with lifetime of the call.
struct Staged {
  void* mem = nullptr;
  const int64_t* f = nullptr;
  const float* y = nullptr;
  float* x = nullptr;
  float* part = nullptr;
  float* prob = nullptr;
  float* losses = nullptr;
  double* lg = nullptr;
  double* acc = nullptr;
  ~Staged() {
    if (mem) (void)hipFree(mem);
  }
};

// want_fit: the buffers of the feature statistics
static fp_status stage(const int64_t* f, const float* y, int n, int mem_kind, int tiles,
                       bool want_x, bool want_part, bool want_prob, int loss_slots, hipStream_t s,
                       Staged* st, bool want_fit = false) {
  const size_t fb = (size_t)n * kIn * sizeof(int64_t);
  const size_t yb = y ? (size_t)n * sizeof(float) : 0;
  const size_t xb = want_x ? (size_t)n * kIn * sizeof(float) : 0;
  size_t total = al(xb);
  if (mem_kind == 0) total += al(fb) + al(yb);
  if (want_part) total += al((size_t)tiles * kPart * sizeof(float));
  if (want_prob) total += al((size_t)n * sizeof(float));
  total += al((size_t)loss_slots * sizeof(float));
  const size_t lb = (size_t)std::min(n, kFitChunk) * kIn * sizeof(double);
  if (want_fit) total += al(lb) + al(2 * kIn * 64 * sizeof(double));
  hipError_t he = total ? hipMalloc(&st->mem, total) : hipSuccess;
  if (he != hipSuccess) {
    st->mem = nullptr;
    return hip_fail(he, "allocating scorer buffers");
  }
  char* p = static_cast<char*>(st->mem);
  if (want_x) st->x = reinterpret_cast<float*>(p);
  p += al(xb);
  if (mem_kind == 0) {
    int64_t* fd = reinterpret_cast<int64_t*>(p);
    p += al(fb);
    he = hipMemcpyAsync(fd, f, fb, hipMemcpyHostToDevice, s);
    st->f = fd;
    if (y) {
      float* yd = reinterpret_cast<float*>(p);
      p += al(yb);
      if (he == hipSuccess) he = hipMemcpyAsync(yd, y, yb, hipMemcpyHostToDevice, s);
      st->y = yd;
    }
    if (he != hipSuccess) return hip_fail(he, "copying scorer inputs");
  } else {
    st->f = f;
    st->y = y;
  }
  if (want_part) {
    st->part = reinterpret_cast<float*>(p);
    p += al((size_t)tiles * kPart * sizeof(float));
  }
  if (want_prob) {
    st->prob = reinterpret_cast<float*>(p);
    p += al((size_t)n * sizeof(float));
  }
  st->losses = reinterpret_cast<float*>(p);
  p += al((size_t)loss_slots * sizeof(float));
  if (want_fit) {
    st->lg = reinterpret_cast<double*>(p);
    st->acc = reinterpret_cast<double*>(p + al(lb));
  }
  return FP_OK;
}

fp_status scorer_fit_impl(fp_scorer* sc, const int64_t* f, int n, int mem_kind, hipStream_t s) {
  Staged st;
  fp_status r = stage(f, nullptr, n, mem_kind, 0, false, false, false, 0, s, &st, true);
  if (r) return r;
  const bool one = n <= kFitChunk;
  for (int pass = one ? 3 : 1; pass <= (one ? 3 : 2); ++pass)
    for (long long at = 0; at < n; at += kFitChunk) {
      const int m = (int)std::min<long long>(kFitChunk, n - at);
      k_log1p<<<(m * kIn + 255) / 256, 256, 0, s>>>(st.f + at * kIn, m, st.lg);
      k_norm_stats<<<1, kIn * 64, 0, s>>>(st.lg, m, n, pass, at == 0, at + m == n, st.acc, sc->ms);
    }
  hipError_t he = hipGetLastError();
  if (he == hipSuccess) he = hipStreamSynchronize(s);
  if (he != hipSuccess) return hip_fail(he, "feature statistics");
  sc->normalized = true;
  return FP_OK;
}

// Shared by gradient and training: normalized features, then `steps`
// forward / backward / reduce (+ Adam when update) rounds.
static fp_status run_steps(fp_scorer* sc, const int64_t* f, const float* y, int n, int mem_kind,
                           int steps, bool update, float lr, hipStream_t s, float* grad_host,
                           float* loss_host, float* losses_host) {
  if (!sc->normalized) {
    set_error("fit the feature normalization first");
    return FP_ERR_STATE;
  }
  const int tiles = (n + kTile - 1) / kTile;
  Staged st;
  fp_status r = stage(f, y, n, mem_kind, tiles, true, true, false, steps, s, &st);
  if (r) return r;
  k_norm_apply<<<(unsigned)(((size_t)n * kIn + 255) / 256), 256, 0, s>>>(st.f, n, sc->ms, st.x);
  const float inv_n = 1.f / (float)n;
  const double b1 = 0.9, b2 = 0.999;
  for (int t = 0; t < steps; ++t) {
    k_fwd_bwd<true><<<tiles, kMlpThreads, 0, s>>>(sc->prm, st.x, nullptr, nullptr, st.y, n,
                                                  inv_n, st.part, nullptr);
    const int step = sc->step + 1;
    const float c1 = (float)(1.0 / (1.0 - std::pow(b1, step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow(b2, step)));
    k_reduce_adam<<<(kParams + 64) / 64, 64 * kAdamWaves, 0, s>>>(
        st.part, tiles, sc->prm, sc->m, sc->v, sc->grad, st.losses + t, update ? 1 : 0, lr,
        (float)b1, (float)b2, 1e-8f, c1, c2);
    if (update) sc->step = step;
  }
  hipError_t he = hipGetLastError();
  if (he == hipSuccess && grad_host)
    he = hipMemcpyAsync(grad_host, sc->grad, kParams * sizeof(float), hipMemcpyDeviceToHost, s);
  if (he == hipSuccess && loss_host && steps > 0)
    he = hipMemcpyAsync(loss_host, st.losses + steps - 1, sizeof(float), hipMemcpyDeviceToHost, s);
  if (he == hipSuccess && losses_host && steps > 0)
    he = hipMemcpyAsync(losses_host, st.losses, (size_t)steps * sizeof(float),
                        hipMemcpyDeviceToHost, s);
  if (he == hipSuccess) he = hipStreamSynchronize(s);
  if (he != hipSuccess) return hip_fail(he, "scorer steps");
  return FP_OK;
}

fp_status scorer_gradient_impl(fp_scorer* sc, const int64_t* f, const float* y, int n,
                               int mem_kind, hipStream_t s, float* grad, float* loss) {
  return run_steps(sc, f, y, n, mem_kind, 1, false, 0.f, s, grad, loss, nullptr);
}

fp_status scorer_train_impl(fp_scorer* sc, const int64_t* f, const float* y, int n, int mem_kind,
                            int steps, float lr, hipStream_t s, float* losses) {
  return run_steps(sc, f, y, n, mem_kind, steps, true, lr, s, nullptr, nullptr, losses);
}

fp_status scorer_predict_impl(fp_scorer* sc, const int64_t* f, int n, int mem_kind,
                              hipStream_t s, float* prob) {
  if (!sc->normalized) {
    set_error("fit the feature normalization first");
    return FP_ERR_STATE;
  }
  const int tiles = (n + kTile - 1) / kTile;
  Staged st;
  fp_status r = stage(f, nullptr, n, mem_kind, tiles, false, false, mem_kind == 0, 0, s, &st);
  if (r) return r;
  float* out = mem_kind == 0 ? st.prob : prob;
  k_fwd_bwd<false><<<tiles, kMlpThreads, 0, s>>>(sc->prm, nullptr, st.f, sc->ms, nullptr, n, 0.f,
                                                 nullptr, out);
  hipError_t he = hipGetLastError();
  if (he == hipSuccess && mem_kind == 0)
    he = hipMemcpyAsync(prob, out, (size_t)n * sizeof(float), hipMemcpyDeviceToHost, s);
  if (he == hipSuccess) he = hipStreamSynchronize(s);
  if (he != hipSuccess) return hip_fail(he, "scorer prediction");
  return FP_OK;
}

fp_status scorer_get_impl(const fp_scorer* sc, float* params, double* mean_std) {
  hipError_t he = hipMemcpy(params, sc->prm, kParams * sizeof(float), hipMemcpyDeviceToHost);
  if (he == hipSuccess && mean_std)
    he = hipMemcpy(mean_std, sc->ms, 2 * kIn * sizeof(double), hipMemcpyDeviceToHost);
  if (he != hipSuccess) return hip_fail(he, "reading the scorer");
  return FP_OK;
}

fp_status scorer_set_impl(fp_scorer* sc, const float* params, const double* mean_std) {
  for (int i = 0; i < kParams; ++i)
    if (!std::isfinite(params[i])) {
      set_error("parameter %d is not finite", i);
      return FP_ERR_INVALID;
    }
  for (int i = 0; mean_std && i < 2 * kIn; ++i)
    if (!std::isfinite(mean_std[i]) || (i >= kIn && mean_std[i] <= 0.0)) {
      set_error("normalization entry %d is not usable", i);
      return FP_ERR_INVALID;
    }
  hipError_t he = hipMemcpy(sc->prm, params, kParams * sizeof(float), hipMemcpyHostToDevice);
  if (he == hipSuccess && mean_std) {
    he = hipMemcpy(sc->ms, mean_std, 2 * kIn * sizeof(double), hipMemcpyHostToDevice);
    sc->normalized = true;
  }
  if (he != hipSuccess) return hip_fail(he, "loading the scorer");
  return FP_OK;
}

}  // namespace hf
