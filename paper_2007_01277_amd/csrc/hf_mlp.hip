// hf_mlp.hip -- learned cost model of the fused-kernel tuner.
//
// A multilayer perceptron (three hidden layers of 64 ReLU units, linear output)
// predicts log2 of a fused launch's time from features of the two solo kernels
// and of the configuration (split, workgroup size, VGPR bound).  It is trained
// on the GPU by the kernels below (forward, mean-squared-error gradient, the
// two backward products, Adam), all deterministic: every output element is
// written by one lane that reduces in a fixed order, with no atomics.  The
// tuner ranks every candidate with it and profiles only the best k; the
// exhaustive search remains the fallback and the reference for its regret.
//
// Parameter layout (one flat fp32 vector): W1[d][64] b1[64] W2[64][64] b2[64]
// W3[64][64] b3[64] W4[64][1] b4[1], row-major W[in][out].
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <vector>

#include "hf_runtime.hpp"

namespace hf {

constexpr int kHid = 64;
constexpr int kFeat = HF_MLP_FEATURES;

// ------------------------------------------------------------------ kernels
// One training step of every member of an ensemble is two launches:
//   k_rows   everything that is local to a sample: the forward pass, the
//            squared error's derivative and the chain of dz back to layer 1;
//   k_grads  everything that sums over the samples: the gradient of each
//            parameter, and its Adam update.
// The second dimension of both grids is the member.  The sums keep one order:
// a dot product over a layer's inputs runs from the bias (or 0) through the
// inputs in order, a gradient through the samples in order, each in one lane
// with fused multiply-adds, so results do not depend on the launch shape.
//
// What bounds a step is not arithmetic (0.5 GFLOP at 1500 samples and five
// members) but the serial chain over the samples and the launches.  Thirteen
// launches per member and step with one lane walking memory per output took
// 7.2 ms per step of five members at 1500 samples and 42 features; the two
// launches take 18 + 22 us for all five members.

// Rows of one sample tile, in LDS: [kRows][64] activations or dz of each wave.
constexpr int kRows = 4;       // samples per wavefront (one float4 of a transposed row)
constexpr int kRowWaves = 4;   // wavefronts per workgroup
constexpr int kTile = 128;     // samples of one step of k_grads
constexpr int kPad = kHid + 1;  // row pitch of a weight matrix in LDS: a column
                                // and a row are both read without bank conflicts

struct MlpArgs {
  const float* X;   // [n][d] standardised samples
  const float* Xt;  // [d][ns] the same, transposed
  const float* y;   // [n]
  float* p;         // [members][np] parameters
  float* g;         // [members][np] gradients (k_grads without an update)
  float* m;         // [members][np] Adam's moments
  float* v;
  float* ws;        // [members][wstride] workspace, see the offsets below
  size_t wstride;
  int n, ns, d, np;  // ns: pitch of a row of samples (pitch())
  __host__ __device__ size_t o_ht(int l) const { return (size_t)l * kHid * ns; }          // [64][ns] layer l < 2's output
  __host__ __device__ size_t o_dz(int l) const { return (size_t)(3 + l) * kHid * ns; }    // [ns][64] its dz
  __host__ __device__ size_t o_h3() const { return (size_t)2 * kHid * ns; }               // [ns][64] layer 3's output
  __host__ __device__ size_t o_yh() const { return (size_t)6 * kHid * ns; }               // [ns] output
  __host__ __device__ size_t o_d4() const { return (size_t)6 * kHid * ns + ns; }          // [ns] its dz
  __host__ __device__ static size_t stride(int ns) { return (size_t)6 * kHid * ns + 2 * (size_t)ns; }
  // whole tiles of k_grads
  __host__ __device__ static int pitch(int n) { return (n + kTile - 1) / kTile * kTile; }
};

// acc[r] += sum_k in[r][k] * w[k*wk], k in order.  `in` are kRows rows of 64 in
// LDS (read as broadcasts), w this lane's column (wk = kPad) or row (wk = 1).
// The next four inputs are read while these four are used; the loop stays
// rolled, since every wavefront passes here only once per layer and straight-
// line code is then bound by instruction fetch (fully unrolled: 27 us per
// launch instead of 19).
__device__ __forceinline__ void dense64(const float* in, const float* w, int wk, float (&acc)[kRows]) {
  struct Step {
    float4 x[kRows];
    float w[4];
  };
  auto load = [&](int k, Step& q) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) q.x[r] = *reinterpret_cast<const float4*>(in + r * kHid + k);
#pragma unroll
    for (int c = 0; c < 4; ++c) q.w[c] = w[(k + c) * wk];
  };
  auto use = [&](const Step& q) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = __builtin_fmaf(q.x[r].x, q.w[0], acc[r]);
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = __builtin_fmaf(q.x[r].y, q.w[1], acc[r]);
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = __builtin_fmaf(q.x[r].z, q.w[2], acc[r]);
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = __builtin_fmaf(q.x[r].w, q.w[3], acc[r]);
  };
  Step q[3];
  load(0, q[0]);
  load(4, q[1]);
#pragma unroll 1
  for (int k = 0; k < kHid - 4; k += 12) {  // 60 inputs, then the last four
    load(k + 8, q[2]);
    __builtin_amdgcn_sched_barrier(0);
    use(q[0]);
    load(k + 12, q[0]);
    __builtin_amdgcn_sched_barrier(0);
    use(q[1]);
    load(min(k + 16, kHid - 4), q[1]);
    __builtin_amdgcn_sched_barrier(0);
    use(q[2]);
  }
  use(q[0]);
}

// Lane j of a wavefront holds output j of kRows samples.  The two 64x64
// matrices sit in LDS, shared by the workgroup's wavefronts; the samples' rows
// pass from layer to layer through LDS.  A wavefront past the last sample
// repeats it and stores nothing.  TRAIN: also the dz of every layer.
template <bool TRAIN>
__global__ void __launch_bounds__(64 * kRowWaves) k_rows(MlpArgs a) {
  __shared__ float w2[kHid * kPad], w3[kHid * kPad], w4[kHid];
  __shared__ __align__(16) float rows[kRowWaves][kRows * kHid];
  const int lane = (int)threadIdx.x & 63;
  const int wave = (int)uniform(threadIdx.x >> 6);
  const float* W1 = a.p + (size_t)blockIdx.y * a.np;
  const float* b1 = W1 + (size_t)a.d * kHid;
  const float* W2 = b1 + kHid;
  const float* b2 = W2 + kHid * kHid;
  const float* W3 = b2 + kHid;
  const float* b3 = W3 + kHid * kHid;
  const float* W4 = b3 + kHid;
  const float* b4 = W4 + kHid;
  float* ws = a.ws + (size_t)blockIdx.y * a.wstride;
  float* in = rows[wave];
  const int i0 = ((int)blockIdx.x * kRowWaves + wave) * kRows;

  // both matrices are requested before layer 1 and put into LDS after it
  constexpr int kLoads = kHid * kHid / (64 * kRowWaves);
  float q2[kLoads], q3[kLoads];
#pragma unroll
  for (int t = 0; t < kLoads; ++t) {
    q2[t] = W2[(int)threadIdx.x + 64 * kRowWaves * t];
    q3[t] = W3[(int)threadIdx.x + 64 * kRowWaves * t];
  }
  const float q4 = W4[lane], bias2 = b2[lane], bias3 = b3[lane], bias4 = b4[0];
  float acc[kRows], target[kRows];
  const float* x[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int i = min(i0 + r, a.n - 1);
    x[r] = a.X + (size_t)i * a.d;
    if (TRAIN) target[r] = a.y[i];
    acc[r] = b1[lane];
  }
#pragma unroll 8
  for (int k = 0; k < a.d; ++k) {
    const float w = W1[(size_t)k * kHid + lane];
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = __builtin_fmaf(x[r][k], w, acc[r]);
  }
#pragma unroll
  for (int t = 0; t < kLoads; ++t) {
    const int e = (int)threadIdx.x + 64 * kRowWaves * t;
    w2[(e >> 6) * kPad + (e & 63)] = q2[t];
    w3[(e >> 6) * kPad + (e & 63)] = q3[t];
  }
  if (wave == 0) w4[lane] = q4;

  float h[3][kRows];
  auto keep = [&](int l) {  // layer l's output: to LDS for the next layer, transposed to memory
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      h[l][r] = fmaxf(acc[r], 0.f);
      in[r * kHid + lane] = h[l][r];
    }
    if (TRAIN && l == 2) {
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        if (i0 + r < a.n) ws[a.o_h3() + (size_t)(i0 + r) * kHid + lane] = h[l][r];
    } else if (TRAIN && i0 < a.n)  // rows past n lie within the pitch and are not used
      *reinterpret_cast<float4*>(ws + a.o_ht(l) + (size_t)lane * a.ns + i0) =
          make_float4(h[l][0], h[l][1], h[l][2], h[l][3]);
    __syncthreads();
  };
  keep(0);
#pragma unroll
  for (int r = 0; r < kRows; ++r) acc[r] = bias2;
  dense64(in, w2 + lane, kPad, acc);
  __syncthreads();
  keep(1);
#pragma unroll
  for (int r = 0; r < kRows; ++r) acc[r] = bias3;
  dense64(in, w3 + lane, kPad, acc);
  __syncthreads();
  keep(2);
  // the output, the same in every lane
#pragma unroll
  for (int r = 0; r < kRows; ++r) acc[r] = bias4;
  dense64(in, w4, 1, acc);
  float d4[kRows];
  const float inv = 1.0f / (float)a.n;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int i = i0 + r;
    if (lane == 0 && i < a.n) ws[a.o_yh() + i] = acc[r];
    if (TRAIN) {
      const float e = acc[r] - target[r];
      d4[r] = 2.0f * e * inv;
      if (lane == 0 && i < a.n) ws[a.o_d4() + i] = d4[r];
    }
  }
  if constexpr (TRAIN) {
    auto send = [&](int l, float (&dz)[kRows]) {  // dz of layer l: to memory and to LDS
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        dz[r] = h[l][r] > 0.f ? dz[r] : 0.f;
        in[r * kHid + lane] = dz[r];
        if (i0 + r < a.n) ws[a.o_dz(l) + (size_t)(i0 + r) * kHid + lane] = dz[r];
      }
      __syncthreads();
    };
    float dz[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) dz[r] = __builtin_fmaf(d4[r], q4, 0.f);
    send(2, dz);
#pragma unroll
    for (int r = 0; r < kRows; ++r) dz[r] = 0.f;
    dense64(in, w3 + lane * kPad, 1, dz);
    send(1, dz);
#pragma unroll
    for (int r = 0; r < kRows; ++r) dz[r] = 0.f;
    dense64(in, w2 + lane * kPad, 1, dz);
    send(0, dz);
  }
}

// dW[k][j] = sum_i A[i][k] dZ[i][j] and db[j] = sum_i dZ[i][j], samples in
// order, then (UPDATE) Adam on the parameter.  A wavefront takes one row k of a
// layer (the bias is the row after the last, with A = 1), lane j the column; a
// workgroup's four rows share dZ, which passes through LDS in tiles of kTile
// samples, the next tile requested before this one is used.  The samples were
// written by other dies a moment ago, so a read takes about 1700 cycles to come
// back: a tile's chain covers that, and sharing divides the traffic by four.  A
// comes transposed, so four of its values are one (broadcast) LDS read.  (Two
// rows per wavefront, reading dZ from memory 32 samples ahead: 33-35 us per
// launch at 1500 samples and five members.)  The output layer has one column:
// its lanes are the rows, d4 is the broadcast value and the tiles are of h3; its
// bias, in the second wavefront, adds d4 alone.
struct AdamArgs {
  float lr, b1, b2, eps, bc1, bc2;  // bias corrections bc1 = 1 - b1^t, bc2 = 1 - b2^t
};

constexpr int kGradRows = 4;  // rows (wavefronts) per workgroup
__host__ __device__ constexpr int row_groups(int din) { return (din + kGradRows) / kGradRows; }  // din rows and the bias
__host__ __device__ constexpr int grad_jobs(int d) { return row_groups(d) + 2 * row_groups(kHid) + 1; }

template <bool UPDATE>
__global__ void __launch_bounds__(64 * kGradRows) k_grads(MlpArgs a, AdamArgs ad) {
  constexpr int kQ = kTile * kHid / 4 / (64 * kGradRows);  // float4 of a tile per lane
  static_assert(kTile <= 4 * 64 && kTile % 16 == 0, "a wavefront loads its row of A with one float4 per lane");
  __shared__ __align__(16) float D[2][kTile * kHid];
  __shared__ __align__(16) float A[2][kGradRows][kTile];
  const int lane = (int)threadIdx.x & 63;
  const int wave = (int)uniform(threadIdx.x >> 6);
  const float* ws = a.ws + (size_t)blockIdx.y * a.wstride;
  size_t off = (size_t)blockIdx.y * a.np;  // of this workgroup's layer
  const int j1 = row_groups(a.d), j2 = row_groups(kHid);
  int job = (int)blockIdx.x, din = a.d;
  const float *at = a.Xt, *dz = ws + a.o_dz(0);
  const bool last = job >= j1 + 2 * j2;
  if (last) {
    job = 0;
    off += (size_t)a.d * kHid + kHid + 2 * (kHid * kHid + kHid);
    dz = ws + a.o_h3();
  } else if (job >= j1) {
    const int l = 1 + (job - j1) / j2;
    job = (job - j1) % j2;
    din = kHid;
    off += (size_t)a.d * kHid + kHid + (size_t)(l - 1) * (kHid * kHid + kHid);
    at = ws + a.o_ht(l - 1);
    dz = ws + a.o_dz(l);
  }
  const int k = kGradRows * job + wave;
  const bool live = last ? wave < 2 : k <= din;
  const float* row = last ? ws + a.o_d4() : k < din ? at + (size_t)k * a.ns : nullptr;  // null: all ones

  f32x4 q[kQ], qa = {1.f, 1.f, 1.f, 1.f};
  auto request = [&](int t0) {  // the pitch holds whole tiles
    const f32x4* src = reinterpret_cast<const f32x4*>(dz + (size_t)t0 * kHid) + threadIdx.x;
#pragma unroll
    for (int t = 0; t < kQ; ++t) q[t] = src[64 * kGradRows * t];
    if (row && lane < kTile / 4) qa = reinterpret_cast<const f32x4*>(row + t0)[lane];
  };
  auto place = [&](int buf) {
    f32x4* dst = reinterpret_cast<f32x4*>(D[buf]) + threadIdx.x;
#pragma unroll
    for (int t = 0; t < kQ; ++t) dst[64 * kGradRows * t] = q[t];
    if (lane < kTile / 4) reinterpret_cast<f32x4*>(A[buf][wave])[lane] = qa;
  };
  float acc = 0.f;
  request(0);
  place(0);
  __syncthreads();
  int buf = 0;
  for (int t0 = 0; t0 < a.n; t0 += kTile, buf ^= 1) {
    const bool more = t0 + kTile < a.n;
    if (more) request(t0 + kTile);
    const int cnt = min(kTile, a.n - t0);
    const float* av = A[buf][wave];
    const float* dv = D[buf] + lane;
    if (last && wave == 1) {
      for (int i = 0; i < cnt; ++i) acc += av[i];
    } else {
      int i = 0;
#pragma unroll 2
      for (; i + 16 <= cnt; i += 16) {
#pragma unroll
        for (int u = 0; u < 16; u += 4) {
          const float4 x = *reinterpret_cast<const float4*>(av + i + u);
          acc = __builtin_fmaf(x.x, dv[(i + u) * kHid], acc);
          acc = __builtin_fmaf(x.y, dv[(i + u + 1) * kHid], acc);
          acc = __builtin_fmaf(x.z, dv[(i + u + 2) * kHid], acc);
          acc = __builtin_fmaf(x.w, dv[(i + u + 3) * kHid], acc);
        }
      }
      for (; i < cnt; ++i) acc = __builtin_fmaf(av[i], dv[i * kHid], acc);
    }
    if (more) place(buf ^ 1);
    __syncthreads();
  }
  auto put = [&](size_t t) {
    if constexpr (UPDATE) {
      const float mi = ad.b1 * a.m[t] + (1.f - ad.b1) * acc;
      const float vi = ad.b2 * a.v[t] + (1.f - ad.b2) * acc * acc;
      a.m[t] = mi;
      a.v[t] = vi;
      a.p[t] = a.p[t] - ad.lr * (mi / ad.bc1) / (sqrtf(vi / ad.bc2) + ad.eps);
    } else {
      a.g[t] = acc;
    }
  };
  if (!live) return;
  if (last && wave == 1) {
    if (lane == 0) put(off + kHid);
  } else {
    put(off + (size_t)k * kHid + lane);
  }
}

// Xt[k][i] = X[i][k]: lanes along the samples, so the stores are whole lines.
__global__ void __launch_bounds__(256) k_transpose(const float* __restrict__ X, int n, int ns, int d,
                                                   float* __restrict__ Xt) {
  const int i = (int)(blockIdx.x * 256 + threadIdx.x);
  if (i < n)
    for (int k = (int)blockIdx.y; k < d; k += (int)gridDim.y) Xt[(size_t)k * ns + i] = X[(size_t)i * d + k];
}

// loss[member] = (1/n) sum (yhat - y)^2.  One workgroup of 1024 lanes per
// member: strided partial sums, then a fixed LDS tree.
__global__ void __launch_bounds__(1024) k_loss(MlpArgs a, float* __restrict__ loss) {
  __shared__ float red[1024];
  const float* yhat = a.ws + (size_t)blockIdx.x * a.wstride + a.o_yh();
  float s = 0.f;
  const float inv = 1.0f / (float)a.n;
  for (int i = threadIdx.x; i < a.n; i += 1024) {
    const float e = yhat[i] - a.y[i];
    s = __builtin_fmaf(e, e, s);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[blockIdx.x] = red[0] * inv;
}

// ------------------------------------------------------------------ model state
// An ensemble of `members` networks of the same shape, trained side by side on
// the same standardised data from different initial weights; the prediction is
// the mean of the members' predictions.
struct MlpModel {
  int d = 0, np = 0, t = 0, members = 1;
  bool trained = false;
  float *p = nullptr, *m = nullptr, *v = nullptr;  // [members][np] parameters and Adam's moments
  float* g = nullptr;                              // [np] gradient of the first member
  // workspace: one allocation for cap_n samples and `slots` members at a time
  int cap_n = 0, slots = 0;
  float *arena = nullptr, *X = nullptr, *Xt = nullptr, *y = nullptr, *loss = nullptr, *ws = nullptr;
  std::vector<float> mu, sd;
  float ymu = 0.f, ysd = 1.f;
};

static MlpModel* g_model = nullptr;  // one model per process, on the device that created it
static int g_model_dev = -1;

static void mlp_free_ws(MlpModel* M) {
  if (M->arena) (void)hipFree(M->arena);
  M->arena = nullptr;
  M->cap_n = M->slots = 0;
}

void mlp_free() {
  if (!g_model) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  (void)hipSetDevice(g_model_dev);
  mlp_free_ws(g_model);
  if (g_model->p) (void)hipFree(g_model->p);  // with the moments and the gradient
  delete g_model;
  g_model = nullptr;
  (void)hipSetDevice(cur);
}

static int nparams(int d) { return d * kHid + kHid + 2 * (kHid * kHid + kHid) + kHid + 1; }

static int alloc_f(float** q, size_t n) {
  hipError_t e = hipMalloc(q, std::max<size_t>(n, 1) * sizeof(float));
  if (e != hipSuccess) {
    record_hip(e);
    return HF_ENOMEM;
  }
  return HF_OK;
}

// Members whose samples are in flight together: all of them, unless that takes
// more than 256 MiB of workspace.
static int slots_for(int members, int n) {
  const size_t one = MlpArgs::stride(MlpArgs::pitch(n)) * sizeof(float);
  return (int)std::max<size_t>(1, std::min<size_t>((size_t)members, (size_t(256) << 20) / one));
}

static int ensure_ws(MlpModel* M, int n) {
  if (n <= M->cap_n) return HF_OK;
  mlp_free_ws(M);
  const int c = std::max(n, 1024), slots = slots_for(M->members, c);
  const size_t ns = MlpArgs::pitch(c);
  const size_t fx = ((size_t)c * M->d + 63) / 64 * 64, fxt = ns * M->d, fy = ns, fl = 64;
  int rc;
  if ((rc = alloc_f(&M->arena, fx + fxt + fy + fl + (size_t)slots * MlpArgs::stride((int)ns))) != HF_OK) return rc;
  M->X = M->arena;
  M->Xt = M->X + fx;
  M->y = M->Xt + fxt;
  M->loss = M->y + fy;
  M->ws = M->loss + fl;
  M->cap_n = c;
  M->slots = slots;
  return HF_OK;
}

static int model(MlpModel** out) {
  if (!g_model) return HF_ENOMODEL;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return record_hip(e);
  if (dev != g_model_dev) return HF_EINVAL;  // the model lives on another device
  *out = g_model;
  return HF_OK;
}

#define HF_LAUNCH(...)                                  \
  do {                                                  \
    hipLaunchKernelGGL(__VA_ARGS__);                    \
    hipError_t e_ = hipGetLastError();                  \
    if (e_ != hipSuccess) return record_hip(e_);        \
  } while (0)

// Kernel arguments for members k .. on n samples (the pitch is that of n, not
// of the workspace's capacity, so that it only depends on the call).
static MlpArgs mlp_args(const MlpModel* M, int k, int n) {
  const int ns = MlpArgs::pitch(n);
  const size_t o = (size_t)k * M->np;
  return MlpArgs{M->X, M->Xt, M->y, M->p + o, M->g, M->m + o, M->v + o, M->ws, MlpArgs::stride(ns), n, ns, M->d, M->np};
}

// Outputs of `cnt` members (and, TRAIN, every dz) for the samples in M->X.
template <bool TRAIN>
static int rows(const MlpArgs& a, int cnt, hipStream_t st) {
  const int per = kRows * kRowWaves;
  HF_LAUNCH(k_rows<TRAIN>, dim3((a.n + per - 1) / per, cnt), dim3(64 * kRowWaves), 0, st, a);
  return HF_OK;
}

static int transpose(const MlpArgs& a, const MlpModel* M, hipStream_t st) {
  HF_LAUNCH(k_transpose, dim3((a.n + 255) / 256, std::min(a.d, 64)), dim3(256), 0, st, M->X, a.n, a.ns, a.d, M->Xt);
  return HF_OK;
}

static AdamArgs adam_args(int t, float lr) {
  const double b1 = 0.9, b2 = 0.999;
  return AdamArgs{lr, (float)b1, (float)b2, 1e-8f, (float)(1.0 - std::pow(b1, t)), (float)(1.0 - std::pow(b2, t))};
}

// One full-batch Adam step t of `cnt` members.
static int train_step(const MlpArgs& a, int cnt, int t, float lr, hipStream_t st) {
  int rc = rows<true>(a, cnt, st);
  if (rc != HF_OK) return rc;
  HF_LAUNCH(k_grads<true>, dim3(grad_jobs(a.d), cnt), dim3(64 * kGradRows), 0, st, a, adam_args(t, lr));
  return HF_OK;
}

static int losses(const MlpArgs& a, const MlpModel* M, int cnt, hipStream_t st) {
  HF_LAUNCH(k_loss, dim3(cnt), dim3(1024), 0, st, a, M->loss);
  return HF_OK;
}

static int upload(float* dst, const float* src, size_t n, hipStream_t st) {
  hipError_t e = hipMemcpyAsync(dst, src, n * sizeof(float), hipMemcpyHostToDevice, st);
  return e == hipSuccess ? HF_OK : record_hip(e);
}
static int download(float* dst, const float* src, size_t n, hipStream_t st) {
  hipError_t e = hipMemcpyAsync(dst, src, n * sizeof(float), hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return record_hip(e);
  e = hipStreamSynchronize(st);
  return e == hipSuccess ? HF_OK : record_hip(e);
}

// splitmix64 (Steele, Lea & Flood, OOPSLA 2014): seeded uniform doubles for the
// He-uniform initialisation.
static uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ------------------------------------------------------------------ features
struct SoloFeat {
  double t_ms = 0, bytes = 0, ops = 0;
  double t_blk[3] = {0, 0, 0};  // solo time at blocks 256, 512, 1024
  int kind = 0, vgprs = 0;
};

static void alg_work(const hf_task* t, double* bytes, double* ops) {
  const double n = (double)t->n, c = (double)t->c, h = (double)t->h, w = (double)t->w;
  switch (t->kind) {
    case HF_BN_STATS:
      *bytes = 4.0 * n * c * h * w + 8.0 * c;
      *ops = 4.0 * n * c * h * w;
      break;
    case HF_INT_MIX:
      *bytes = 8.0 * n;
      *ops = 8.0 * n * (double)t->p[0];
      break;
    case HF_IM2COL: {
      const double kh = t->p[0], kw = t->p[1], s = t->p[2], p = t->p[3];
      const double Ho = std::floor((h + 2 * p - kh) / s) + 1, Wo = std::floor((w + 2 * p - kw) / s) + 1;
      const double out = n * c * kh * kw * Ho * Wo;
      *bytes = 4.0 * n * c * h * w + 4.0 * out;
      *ops = 10.0 * out;
      break;
    }
    case HF_LDS_HIST:
      *bytes = n + 1024.0;
      *ops = 3.0 * n;
      break;
    case HF_UPSAMPLE: {
      const double s = t->p[0];
      const double out = n * c * h * w * s * s;
      *bytes = 4.0 * n * c * h * w + 4.0 * out;
      *ops = 20.0 * out;
      break;
    }
    case HF_MAXPOOL: {
      const double kh = t->p[0], kw = t->p[1], s = t->p[2], p = t->p[3];
      const double out = n * c * (std::floor((h + 2 * p - kh) / s) + 1) * (std::floor((w + 2 * p - kw) / s) + 1);
      *bytes = 4.0 * n * c * h * w + (t->out1 ? 8.0 : 4.0) * out;
      *ops = 4.0 * kh * kw * out;
      break;
    }
    case HF_SHA256D:
      *bytes = 32.0 * n;
      *ops = 3.0 * 64 * 24 * n;
      break;
    case HF_BLAKE2B:
      *bytes = 32.0 * n;
      *ops = 12.0 * 8 * 28 * n;
      break;
    case HF_ETHASH:
      *bytes = (64.0 * 128 + 32) * n;
      *ops = (64.0 * 40 / 8 + 80 * 55) * n;  // the walk, then the 80 SHA-512 rounds of the seed
      break;
  }
}

// Times the task alone at each block size (6 launches each, the first a warm
// up; the median of the other five).  `cost`, if given, accumulates the
// launches made and their summed time in milliseconds.
static int solo_feat(DeviceState* s, const hf_task* t, hipStream_t st, SoloFeat* f, FeatCost* cost) {
  f->kind = t->kind;
  alg_work(t, &f->bytes, &f->ops);
  double best = 1e30;
  const int blocks[] = {256, 512, 1024};
  for (int bi = 0; bi < 3; ++bi) {
    std::vector<float> ts;
    for (int r = 0; r < 6; ++r) {
      hipError_t e = hipEventRecord(s->ev_start, st);
      if (e != hipSuccess) return record_hip(e);
      int rc = launch_solo(s, t, blocks[bi], 0, 0, st);
      if (rc != HF_OK) return rc;
      if ((e = hipEventRecord(s->ev_stop, st)) != hipSuccess) return record_hip(e);
      if ((rc = wait_event(s->ev_stop)) != HF_OK) return rc;
      float ms = 0.f;
      if ((e = hipEventElapsedTime(&ms, s->ev_start, s->ev_stop)) != hipSuccess) return record_hip(e);
      if (cost) {
        cost->launches += 1;
        cost->ms += ms;
      }
      if (r > 0) ts.push_back(ms);  // the first launch warms up
    }
    std::sort(ts.begin(), ts.end());
    f->t_blk[bi] = std::max((double)ts[ts.size() / 2], 1e-4);
    best = std::min(best, f->t_blk[bi]);
  }
  f->t_ms = best;
  hf_kernel_info info;
  int rc = kernel_info(s, find_kernel(t->kind, -1, 1024, 0)->fn, 1024, &info);
  if (rc != HF_OK) return rc;
  f->vgprs = info.vgprs;
  return HF_OK;
}

// Features of one candidate (kFeat values), kernels in canonical order (the
// smaller kind first; the split fraction refers to that kernel):
//   per kernel (kPerKernel each): one-hot kind (HF_NUM_KINDS); log2 solo time
//   at blocks 256, 512, 1024; log2 algorithmic MB and mega-lane-ops; fractions
//   of the HBM and integer-ALU peaks the best solo run reached;
//   configuration (10): split fraction s = 64*split_waves/block; log2(block/512);
//   VGPR bound / 128 (1 when unbounded); resident waves per SIMD / 8;
//   log2(t_a(block)/s), log2(t_b(block)/(1-s)) and the log2 of their maximum,
//   with t_k(block) the solo time at the candidate's block size; the fused
//   instantiation's spill bytes per lane (log2(1 + bytes) / 8) and VGPRs / 128;
//   log2 of the sum of the best solo times (the last feature).
constexpr int kPerKernel = HF_NUM_KINDS + 7;
constexpr int kCfg = 2 * kPerKernel;
static_assert(kCfg + 10 == kFeat, "feature layout and HF_MLP_FEATURES disagree");

static void fill_features(const SoloFeat& fa0, const SoloFeat& fb0, const hf_config& c,
                          const hf_kernel_info& fused, float* x) {
  const int waves_per_simd = fused.waves_per_simd;
  auto l2 = [](double v) { return (float)std::log2(std::max(v, 1e-30)); };
  // canonical order: the kernel of the smaller kind first, with the split
  // fraction mirrored, so (a, b, s) and (b, a, 1 - s) -- the same fused kernel
  // -- get the same features
  const bool swap = fa0.kind > fb0.kind;
  const SoloFeat& fa = swap ? fb0 : fa0;
  const SoloFeat& fb = swap ? fa0 : fb0;
  const SoloFeat* f[2] = {&fa, &fb};
  for (int k = 0; k < 2; ++k) {
    float* o = x + kPerKernel * k;
    for (int i = 0; i < HF_NUM_KINDS; ++i) o[i] = (f[k]->kind == i) ? 1.f : 0.f;
    float* q = o + HF_NUM_KINDS;
    q[0] = l2(f[k]->t_blk[0]);
    q[1] = l2(f[k]->t_blk[1]);
    q[2] = l2(f[k]->t_blk[2]);
    q[3] = l2(f[k]->bytes / 1e6 + 1e-3);
    q[4] = l2(f[k]->ops / 1e6 + 1e-3);
    q[5] = (float)(f[k]->bytes / (f[k]->t_ms * 1e-3) / 8e12);
    q[6] = (float)(f[k]->ops / (f[k]->t_ms * 1e-3) / 39.3216e12);
  }
  const int bi = c.block == 256 ? 0 : (c.block == 512 ? 1 : 2);
  const double W = c.block / 64.0;
  const double s = swap ? 1.0 - c.split_waves / W : c.split_waves / W;
  float* g = x + kCfg;
  g[0] = (float)s;
  g[1] = l2(c.block / 512.0);
  g[2] = c.vgpr_cap == 0 ? 1.f : c.vgpr_cap / 128.f;
  g[3] = waves_per_simd / 8.f;
  const double ta = fa.t_blk[bi] / s, tb = fb.t_blk[bi] / (1.0 - s);
  g[4] = l2(ta);
  g[5] = l2(tb);
  g[6] = l2(std::max(ta, tb));
  g[7] = (float)(std::log2(1.0 + std::max(0, fused.spill_bytes)) / 8.0);
  g[8] = fused.vgprs / 128.f;
  g[9] = l2(fa.t_ms + fb.t_ms);
}

int featurize(DeviceState* s, const hf_pair* pr, const hf_config* cfg, int n, hipStream_t st, float* X,
              FeatCost* cost) {
  SoloFeat fa, fb;
  int rc;
  if ((rc = solo_feat(s, &pr->a, st, &fa, cost)) != HF_OK) return rc;
  if ((rc = solo_feat(s, &pr->b, st, &fb, cost)) != HF_OK) return rc;
  for (int i = 0; i < n; ++i) {
    hf_kernel_info info;
    if ((rc = hf_fused_info(pr->a.kind, pr->b.kind, cfg[i].block, cfg[i].vgpr_cap, &info)) != HF_OK) return rc;
    fill_features(fa, fb, cfg[i], info, X + (size_t)i * kFeat);
  }
  return HF_OK;
}

// Standardise raw features / predictions with the model's statistics.
static void standardise(const MlpModel* M, const float* X, int n, std::vector<float>* out) {
  out->resize((size_t)n * M->d);
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < M->d; ++k)
      (*out)[(size_t)i * M->d + k] = (X[(size_t)i * M->d + k] - M->mu[k]) / M->sd[k];
}

// Mean of the members' predictions, in the units of the training targets.
static int predict(MlpModel* M, const float* X, int n, float* y, hipStream_t st) {
  int rc;
  if ((rc = ensure_ws(M, n)) != HF_OK) return rc;
  std::vector<float> xs;
  standardise(M, X, n, &xs);
  if ((rc = upload(M->X, xs.data(), xs.size(), st)) != HF_OK) return rc;
  std::vector<double> acc(n, 0.0);
  std::vector<float> yk((size_t)M->slots * n);
  for (int k = 0; k < M->members; k += M->slots) {
    const int cnt = std::min(M->slots, M->members - k);
    const MlpArgs a = mlp_args(M, k, n);
    if ((rc = rows<false>(a, cnt, st)) != HF_OK) return rc;
    hipError_t e = hipMemcpy2DAsync(yk.data(), n * sizeof(float), a.ws + a.o_yh(), a.wstride * sizeof(float),
                                    n * sizeof(float), cnt, hipMemcpyDeviceToHost, st);
    if (e != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess) return record_hip(e);
    for (int j = 0; j < cnt; ++j)
      for (int i = 0; i < n; ++i) acc[i] += yk[(size_t)j * n + i];
  }
  for (int i = 0; i < n; ++i) y[i] = (float)(acc[i] / M->members) * M->ysd + M->ymu;
  return HF_OK;
}

int mlp_rank(DeviceState* s, const hf_pair* pr, const std::vector<hf_config>& cands, hipStream_t st,
             std::vector<int>* order, FeatCost* cost) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if (!M->trained || M->d != kFeat) return HF_ENOMODEL;
  const int n = (int)cands.size();
  std::vector<float> X((size_t)n * kFeat), y(n);
  if ((rc = featurize(s, pr, cands.data(), n, st, X.data(), cost)) != HF_OK) return rc;
  if ((rc = predict(M, X.data(), n, y.data(), st)) != HF_OK) return rc;
  order->resize(n);
  std::iota(order->begin(), order->end(), 0);
  std::stable_sort(order->begin(), order->end(), [&](int a, int b) { return y[a] < y[b]; });
  return HF_OK;
}

}  // namespace hf

using namespace hf;

extern "C" {

int hf_mlp_init_ensemble(int d_in, uint64_t seed, int members) {
  if (d_in < 1 || d_in > 4096 || members < 1 || members > HF_MLP_MAX_MEMBERS) return HF_EINVAL;
  int rc;
  DeviceState* s = device_state(&rc);
  if (!s) return rc;
  mlp_free();
  MlpModel* M = new MlpModel();
  M->d = d_in;
  M->np = nparams(d_in);
  M->members = members;
  const size_t all = (size_t)members * M->np;
  if ((rc = alloc_f(&M->p, 3 * all + M->np)) != HF_OK) {
    delete M;
    return rc;
  }
  M->m = M->p + all;
  M->v = M->m + all;
  M->g = M->v + all;
  // He-uniform weights U(-sqrt(6/fan_in), +sqrt(6/fan_in)), zero biases;
  // member k draws from the splitmix64 stream seeded with seed + k
  std::vector<float> host(all, 0.f);
  const int dims[5] = {d_in, kHid, kHid, kHid, 1};
  for (int k = 0; k < members; ++k) {
    uint64_t st = seed + (uint64_t)k;
    size_t o = (size_t)k * M->np;
    for (int l = 0; l < 4; ++l) {
      const double lim = std::sqrt(6.0 / dims[l]);
      for (int i = 0; i < dims[l] * dims[l + 1]; ++i) {
        const double u = (double)(splitmix64(st) >> 11) * (1.0 / 9007199254740992.0);
        host[o++] = (float)((2.0 * u - 1.0) * lim);
      }
      o += dims[l + 1];
    }
  }
  M->mu.assign(d_in, 0.f);
  M->sd.assign(d_in, 1.f);
  g_model = M;
  g_model_dev = s->device;
  hipError_t e = hipMemcpy(M->p, host.data(), host.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e != hipSuccess) return record_hip(e);
  if ((e = hipMemset(M->m, 0, 2 * all * sizeof(float))) != hipSuccess) return record_hip(e);  // both moments
  return HF_OK;
}

int hf_mlp_init(int d_in, uint64_t seed) { return hf_mlp_init_ensemble(d_in, seed, 1); }

int hf_mlp_members(void) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  return rc != HF_OK ? rc : M->members;
}

int hf_mlp_num_params(void) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  return rc != HF_OK ? rc : M->np;
}

int hf_mlp_get_params(float* host, int64_t n) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if (!host || n != M->np) return HF_EINVAL;
  return download(host, M->p, M->np, nullptr);
}

int hf_mlp_set_params(const float* host, int64_t n) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if (!host || n != M->np) return HF_EINVAL;
  if ((rc = upload(M->p, host, M->np, nullptr)) != HF_OK) return rc;
  hipError_t e = hipStreamSynchronize(nullptr);
  return e == hipSuccess ? HF_OK : record_hip(e);
}

int hf_mlp_grad(const float* X, const float* y, int n, float* loss_out, float* grad_out) {
  if (!X || !y || n < 1 || !loss_out || !grad_out) return HF_EINVAL;
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if ((rc = ensure_ws(M, n)) != HF_OK) return rc;
  const MlpArgs a = mlp_args(M, 0, n);
  if ((rc = upload(M->X, X, (size_t)n * M->d, nullptr)) || (rc = upload(M->y, y, n, nullptr)) ||
      (rc = transpose(a, M, nullptr)) || (rc = rows<true>(a, 1, nullptr)))
    return rc;
  HF_LAUNCH(k_grads<false>, dim3(grad_jobs(a.d), 1), dim3(64 * kGradRows), 0, nullptr, a, AdamArgs{});
  if ((rc = losses(a, M, 1, nullptr)) != HF_OK) return rc;
  if ((rc = download(loss_out, M->loss, 1, nullptr)) != HF_OK) return rc;
  return download(grad_out, M->g, M->np, nullptr);
}

int hf_mlp_step(const float* X, const float* y, int n, float lr, float* loss_out) {
  if (!X || !y || n < 1 || lr <= 0.f) return HF_EINVAL;
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if ((rc = ensure_ws(M, n)) != HF_OK) return rc;
  const MlpArgs a = mlp_args(M, 0, n);
  if ((rc = upload(M->X, X, (size_t)n * M->d, nullptr)) || (rc = upload(M->y, y, n, nullptr)) ||
      (rc = transpose(a, M, nullptr)) || (rc = train_step(a, 1, M->t + 1, lr, nullptr)))
    return rc;
  M->t += 1;
  if ((rc = losses(a, M, 1, nullptr)) != HF_OK) return rc;
  return loss_out ? download(loss_out, M->loss, 1, nullptr) : HF_OK;
}

int hf_mlp_adam_reset(void) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  M->t = 0;
  hipError_t e;
  if ((e = hipMemset(M->m, 0, M->np * sizeof(float))) != hipSuccess) return record_hip(e);
  if ((e = hipMemset(M->v, 0, M->np * sizeof(float))) != hipSuccess) return record_hip(e);
  return HF_OK;
}

int hf_mlp_train(const float* X, const float* y, int n, int d, int epochs, float lr, float* loss_out) {
  if (!X || !y || n < 2 || epochs < 1 || lr <= 0.f) return HF_EINVAL;
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if (d != M->d) return HF_EINVAL;
  // feature and target standardisation from the training set (double sums)
  for (int k = 0; k < d; ++k) {
    double s = 0, q = 0;
    for (int i = 0; i < n; ++i) s += X[(size_t)i * d + k];
    const double mu = s / n;
    for (int i = 0; i < n; ++i) q += (X[(size_t)i * d + k] - mu) * (X[(size_t)i * d + k] - mu);
    const double sd = std::sqrt(q / n);
    M->mu[k] = (float)mu;
    M->sd[k] = sd > 1e-6 ? (float)sd : 1.f;
  }
  {
    double s = 0, q = 0;
    for (int i = 0; i < n; ++i) s += y[i];
    const double mu = s / n;
    for (int i = 0; i < n; ++i) q += (y[i] - mu) * (y[i] - mu);
    M->ymu = (float)mu;
    M->ysd = std::sqrt(q / n) > 1e-6 ? (float)std::sqrt(q / n) : 1.f;
  }
  std::vector<float> xs, ys(n);
  standardise(M, X, n, &xs);
  for (int i = 0; i < n; ++i) ys[i] = (y[i] - M->ymu) / M->ysd;
  if ((rc = ensure_ws(M, n)) != HF_OK) return rc;
  if ((rc = upload(M->X, xs.data(), xs.size(), nullptr)) || (rc = upload(M->y, ys.data(), n, nullptr))) return rc;
  if ((rc = transpose(mlp_args(M, 0, n), M, nullptr)) != HF_OK) return rc;
  // every member from its own initial weights, on the same data
  double lsum = 0.0;
  M->t = 0;
  const size_t all = (size_t)M->members * M->np;
  hipError_t e = hipMemsetAsync(M->m, 0, 2 * all * sizeof(float), nullptr);  // both moments
  if (e != hipSuccess) return record_hip(e);
  for (int k = 0; k < M->members; k += M->slots) {
    const int cnt = std::min(M->slots, M->members - k);
    const MlpArgs a = mlp_args(M, k, n);
    for (int ep = 1; ep <= epochs; ++ep)
      if ((rc = train_step(a, cnt, ep, lr, nullptr)) != HF_OK) return rc;
    // loss of the members' final parameters
    float l[HF_MLP_MAX_MEMBERS];
    if ((rc = rows<false>(a, cnt, nullptr)) || (rc = losses(a, M, cnt, nullptr)) ||
        (rc = download(l, M->loss, cnt, nullptr)))
      return rc;
    for (int j = 0; j < cnt; ++j) lsum += l[j];
  }
  M->t = epochs;
  if (loss_out) *loss_out = (float)(lsum / M->members);
  M->trained = true;
  return HF_OK;
}

int hf_mlp_predict(const float* X, int n, float* y_out) {
  if (!X || n < 1 || !y_out) return HF_EINVAL;
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  return predict(M, X, n, y_out, nullptr);
}

int hf_mlp_save(const char* path) {
  MlpModel* M = nullptr;
  int rc = model(&M);
  if (rc != HF_OK) return rc;
  if (!path) return HF_EINVAL;
  const size_t all = (size_t)M->members * M->np;
  std::vector<float> p(all);
  if ((rc = download(p.data(), M->p, all, nullptr)) != HF_OK) return rc;
  FILE* f = std::fopen(path, "wb");
  if (!f) return HF_EINVAL;
  const char magic[8] = {'H', 'F', 'M', 'L', 'P', '2', 0, 0};
  const int32_t hdr[4] = {M->d, M->np, M->trained ? 1 : 0, M->members};
  bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(hdr, 4, 4, f) == 4 &&
            std::fwrite(&M->ymu, 4, 1, f) == 1 && std::fwrite(&M->ysd, 4, 1, f) == 1 &&
            std::fwrite(M->mu.data(), 4, M->d, f) == (size_t)M->d &&
            std::fwrite(M->sd.data(), 4, M->d, f) == (size_t)M->d &&
            std::fwrite(p.data(), 4, all, f) == all;
  ok = (std::fclose(f) == 0) && ok;
  return ok ? HF_OK : HF_EINVAL;
}

int hf_mlp_load(const char* path) {
  if (!path) return HF_EINVAL;
  FILE* f = std::fopen(path, "rb");
  if (!f) return HF_EINVAL;
  char magic[8];
  int32_t hdr[4];
  bool ok = std::fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "HFMLP2", 6) == 0 &&
            std::fread(hdr, 4, 4, f) == 4 && hdr[0] >= 1 && hdr[0] <= 4096 && hdr[1] == nparams(hdr[0]) &&
            hdr[3] >= 1 && hdr[3] <= HF_MLP_MAX_MEMBERS;
  if (!ok) {
    std::fclose(f);
    return HF_EINVAL;
  }
  float ymu = 0, ysd = 1;
  const size_t all = (size_t)hdr[3] * hdr[1];
  std::vector<float> mu(hdr[0]), sd(hdr[0]), p(all);
  ok = std::fread(&ymu, 4, 1, f) == 1 && std::fread(&ysd, 4, 1, f) == 1 &&
       std::fread(mu.data(), 4, hdr[0], f) == (size_t)hdr[0] && std::fread(sd.data(), 4, hdr[0], f) == (size_t)hdr[0] &&
       std::fread(p.data(), 4, all, f) == all;
  std::fclose(f);
  if (!ok) return HF_EINVAL;
  int rc = hf_mlp_init_ensemble(hdr[0], 0, hdr[3]);
  if (rc != HF_OK) return rc;
  if ((rc = upload(g_model->p, p.data(), all, nullptr)) != HF_OK) return rc;
  hipError_t e = hipStreamSynchronize(nullptr);
  if (e != hipSuccess) return record_hip(e);
  g_model->mu = mu;
  g_model->sd = sd;
  g_model->ymu = ymu;
  g_model->ysd = ysd;
  g_model->trained = hdr[2] != 0;
  return HF_OK;
}

int hf_featurize(const hf_pair* pr, const hf_config* cfg, int n, void* stream, float* X_out) {
  if (!pr || !cfg || n < 1 || !X_out) return HF_EINVAL;
  int rc;
  for (int i = 0; i < n; ++i)
    if ((rc = hf_validate_fused(pr, &cfg[i])) != HF_OK) return rc;
  DeviceState* s = device_state(&rc);
  if (!s) return rc;
  return featurize(s, pr, cfg, n, static_cast<hipStream_t>(stream), X_out, nullptr);
}

}  // extern "C"
