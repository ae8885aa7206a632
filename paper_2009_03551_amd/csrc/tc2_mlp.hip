// Block-skip network of the TC2 solver: a multilayer perceptron 8 -> 64 -> 64 -> 1
// (ReLU) giving the logit that a candidate output block falls under the drop
// threshold.  Forward, gradient (mean binary cross-entropy on logits) and Adam
// kernels written for gfx950, and the C-ABI entry points that train and
// evaluate it on the device.
//
// Parameter layout (MLP_NP = 4801 floats): W1 (64 x 8 row-major), b1 (64),
// W2 (64 x 64 row-major, W2[j][k] maps input k to output j), b2 (64), w3 (64), b3.
#include "tc2_device.h"
#include "../../include/tc2.h"

#include <cfloat>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

namespace tc2 {

constexpr int OFF_W1 = 0, OFF_B1 = 512, OFF_W2 = 576, OFF_B2 = 4672, OFF_W3 = 4736, OFF_B3 = 4800;
static_assert(MLP_NP == OFF_B3 + 1, "parameter layout");

// One thread per sample: logits of rows of x (n x 8).
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ th,
                                                     const float* __restrict__ x, long long n,
                                                     float* __restrict__ out) {
  __shared__ float s[MLP_NP];
  for (int p = threadIdx.x; p < MLP_NP; p += blockDim.x) s[p] = th[p];
  __syncthreads();
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float xi[MLP_NF];
#pragma unroll
  for (int f = 0; f < MLP_NF; ++f) xi[f] = x[i * MLP_NF + f];
  float h1[MLP_NH];
#pragma unroll
  for (int j = 0; j < MLP_NH; ++j) {
    float a = s[OFF_B1 + j];
#pragma unroll
    for (int f = 0; f < MLP_NF; ++f) a += s[OFF_W1 + j * MLP_NF + f] * xi[f];
    h1[j] = fmaxf(a, 0.f);
  }
  float z = s[OFF_B3];
  for (int j = 0; j < MLP_NH; ++j) {
    float a = s[OFF_B2 + j];
#pragma unroll
    for (int k = 0; k < MLP_NH; ++k) a += s[OFF_W2 + j * MLP_NH + k] * h1[k];
    z += s[OFF_W3 + j] * fmaxf(a, 0.f);
  }
  out[i] = z;
}

// Gradient of the mean loss softplus(z) - y z over samples [0, n) with weight
// inv_n.  A block takes 256 samples, a wave 16 at a time, as FP32 matrix
// products (16x16x4 MFMA) with the units along the rows and the samples along
// the columns: lane (g, c) = (lane / 16, lane % 16) then holds units 16 t + 4 g
// + r of sample c, which is the second operand of the next product as it
// stands, its steps taken in the order (t, r).  The products over samples read the same
// values, stored per sample in LDS, with the units along both sides; their
// sums stay in registers for the wave's samples, the waves are added in a
// fixed order.  gpart (gridDim x MLP_NP), lpart and, where given, bad (gridDim: a value
// of the block or a parameter is not finite) receive the block's results.
//
// Bound by latency: at 65536 samples 69 us, of which 11 are matrix time (216
// MFMAs per 16 samples); straight code runs only twice per wave.  One thread per
// sample, adding its 4800 products to the same LDS words by atomics, took 2890 us.
constexpr int GT = 512, GW = GT / 64;  // threads and waves of a block
constexpr int GS = 256;                // samples of a block
constexpr int LDW = MLP_NH + 4;        // padded rows: 16-byte reads without bank conflicts
typedef float f4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(GT) void k_mlp_grad(const float* __restrict__ th,
                                                 const float* __restrict__ x,
                                                 const float* __restrict__ y, long long n,
                                                 double inv_n, float* __restrict__ gpart,
                                                 double* __restrict__ lpart, int* __restrict__ bad) {
  constexpr int NTL = MLP_NH / 16;              // tiles of units
  struct Tiles {
    f4 w2[MLP_NH * LDW / 4];                    // W2[j][k]
    f4 w2t[MLP_NH * LDW / 4];                   // W2[j][k] at (k, j)
    f4 tr[GW][2][16 * LDW / 4];                 // per wave: two 16 x 64 (sample, unit)
  };
  __shared__ union {
    Tiles m;
    float sums[GW / 2][MLP_NP];                 // after the last product
  } sh;
  __shared__ double sl[GW];
  __shared__ int sbad;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  if (threadIdx.x == 0) sbad = 0;
  for (int p = threadIdx.x; p < MLP_NH * MLP_NH; p += GT) {
    const int j = p / MLP_NH, k = p % MLP_NH;
    const float v = th[OFF_W2 + p];
    ((float*)sh.m.w2)[j * LDW + k] = v;
    ((float*)sh.m.w2t)[k * LDW + j] = v;
  }
  float w1[NTL][2];
  f4 b1[NTL], b2[NTL], w3[NTL];
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
#pragma unroll
    for (int s = 0; s < 2; ++s) w1[t][s] = th[OFF_W1 + (16 * t + c) * MLP_NF + 4 * s + g];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b1[t][r] = th[OFF_B1 + 16 * t + 4 * g + r];
      b2[t][r] = th[OFF_B2 + 16 * t + 4 * g + r];
      w3[t][r] = th[OFF_W3 + 16 * t + 4 * g + r];
    }
  }
  const float b3 = th[OFF_B3];
  __syncthreads();
  if (bad) {
    bool inf = false;
    for (int p = threadIdx.x; p < MLP_NP; p += GT) inf = inf || !(fabsf(th[p]) <= FLT_MAX);
    if (inf) sbad = 1;
  }

  const f4 zero = {0.f, 0.f, 0.f, 0.f};
  f4 gw2[NTL][NTL], gw1[NTL], gb2[NTL], gw3[NTL];  // gw1: features 0..7, then b1
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    gw1[t] = gb2[t] = gw3[t] = zero;
#pragma unroll
    for (int u = 0; u < NTL; ++u) gw2[t][u] = zero;
  }
  float gb3 = 0.f;
  double loss = 0.0;
  f4* const th1 = sh.m.tr[wave][0];
  f4* const td = sh.m.tr[wave][1];
  auto wave_sync = [] {  // LDS of this wave alone: order its accesses
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto mfma32 = [](f4& d, float a, float b) { d = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, d, 0, 0, 0); };
  auto relu = [](f4 v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
    return v;
  };
  // v (units x samples) = m (units x units, rows of LDW) times u
  auto times = [&](const f4* m, const f4* u, f4* v) {
    int at = (c * LDW + 4 * g) / 4;
    asm volatile("" : "+v"(at));  // the weights are read anew: held over the samples they would spill
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int q = 0; q < NTL; ++q) {
        const f4 a = m[at + (16 * q * LDW + 16 * t) / 4];
#pragma unroll
        for (int r = 0; r < 4; ++r) mfma32(v[q], a[r], u[t][r]);
      }
  };
  for (int i0 = wave * 16; i0 < GS; i0 += GW * 16) {
    const long long first = (long long)blockIdx.x * GS + i0, i = first + c;
    if (first >= n) break;
    const bool live = i < n;  // the samples beyond the last are zeros, without weight
    float xs[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) xs[s] = live ? x[i * MLP_NF + 4 * s + g] : 0.f;
    const float yi = live ? y[i] : 0.f;
    if (bad && !(fabsf(xs[0]) <= FLT_MAX && fabsf(xs[1]) <= FLT_MAX && fabsf(yi) <= FLT_MAX)) sbad = 1;
    f4 h1[NTL], h2[NTL];
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      h1[t] = b1[t];
      mfma32(h1[t], w1[t][0], xs[0]);
      mfma32(h1[t], w1[t][1], xs[1]);
      h1[t] = relu(h1[t]);
      h2[t] = b2[t];
    }
    times(sh.m.w2, h1, h2);
    float z = 0.f;
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      h2[t] = relu(h2[t]);
#pragma unroll
      for (int r = 0; r < 4; ++r) z += w3[t][r] * h2[t][r];
    }
    z += __shfl_xor(z, 16, 64);
    z += __shfl_xor(z, 32, 64);
    z += b3;
    float dz = 0.f;
    if (live) {
      // softplus(z) - y z, evaluated without overflow
      if (g == 0) loss += (double)(fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - yi * z) * inv_n;
      dz = (float)((1.0 / (1.0 + exp(-(double)z)) - yi) * inv_n);
      if (g == 0) gb3 += dz;
    }
    // d2: gradient at layer 2 before the activation, d1 at layer 1
    f4 d2[NTL], d1[NTL];
    bool odd = dz != dz;  // 0 times a value beyond the FP32 range must add nothing
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      d1[t] = zero;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d2[t][r] = h2[t][r] > 0.f ? dz * w3[t][r] : 0.f;
        gb2[t][r] += d2[t][r];
        gw3[t][r] += live ? dz * h2[t][r] : 0.f;
        odd = odd || !(h1[t][r] <= FLT_MAX);
      }
    }
    times(sh.m.w2t, d2, d1);
    wave_sync();
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      th1[(c * LDW + 16 * t + 4 * g) / 4] = h1[t];
      td[(c * LDW + 16 * t + 4 * g) / 4] = d2[t];
#pragma unroll
      for (int r = 0; r < 4; ++r) d1[t][r] = h1[t][r] > 0.f ? d1[t][r] : 0.f;
    }
    wave_sync();
    auto unit = [&](const f4* m, int s, int k) { return ((const float*)m)[s * LDW + k]; };
    if (__ballot(odd) == 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float a[NTL], b[NTL];
#pragma unroll
        for (int t = 0; t < NTL; ++t) {
          a[t] = unit(td, 4 * s + g, 16 * t + c);
          b[t] = unit(th1, 4 * s + g, 16 * t + c);
        }
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
          for (int u = 0; u < NTL; ++u) mfma32(gw2[t][u], a[t], b[u]);
      }
    } else {
      for (int s = 0; s < 16; ++s)
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
          for (int u = 0; u < NTL; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float a = unit(td, s, 16 * t + 4 * g + r), b = unit(th1, s, 16 * u + c);
              if (a != 0.f && b > 0.f) gw2[t][u][r] += a * b;
            }
    }
    wave_sync();
#pragma unroll
    for (int t = 0; t < NTL; ++t) td[(c * LDW + 16 * t + 4 * g) / 4] = d1[t];
    wave_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const long long is = first + 4 * s + g;
      const float b = is < n ? (c < MLP_NF ? x[is * MLP_NF + c] : (c == MLP_NF ? 1.f : 0.f)) : 0.f;
#pragma unroll
      for (int t = 0; t < NTL; ++t) mfma32(gw1[t], unit(td, 4 * s + g, 16 * t + c), b);
    }
  }

  // sums over the samples of a wave, then over the waves
  auto over = [](double v, int lanes) {
    for (int o = lanes / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
  auto overf = [](float v) {
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
  loss = over(loss, 16);
  gb3 = overf(gb3);
#pragma unroll
  for (int t = 0; t < NTL; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      gb2[t][r] = overf(gb2[t][r]);
      gw3[t][r] = overf(gw3[t][r]);
    }
  if (lane == 0) sl[wave] = loss;
  // each value of the wave with its place in the block's sums
  auto each = [&](auto&& f) {
#pragma unroll
    for (int t = 0; t < NTL; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = 16 * t + 4 * g + r;
#pragma unroll
        for (int u = 0; u < NTL; ++u) gw2[t][u][r] = f(OFF_W2 + j * MLP_NH + 16 * u + c, gw2[t][u][r]);
        if (c < MLP_NF) gw1[t][r] = f(OFF_W1 + j * MLP_NF + c, gw1[t][r]);
        if (c == MLP_NF) gw1[t][r] = f(OFF_B1 + j, gw1[t][r]);
        if (c == 0) gb2[t][r] = f(OFF_B2 + j, gb2[t][r]);
        if (c == 0) gw3[t][r] = f(OFF_W3 + j, gw3[t][r]);
      }
    if (lane == 0) gb3 = f(OFF_B3, gb3);
  };
  float* sg = sh.sums[wave % (GW / 2)];
  __syncthreads();  // all waves are through with W2 and their tiles
  if (wave >= GW / 2) each([&](int p, float v) { return sg[p] = v; });
  __syncthreads();
  if (wave < GW / 2) {
    each([&](int p, float v) { return v + sg[p]; });
    each([&](int p, float v) { return sg[p] = v; });
  }
  __syncthreads();
  for (int p = threadIdx.x; p < MLP_NP; p += GT) {
    float v = sh.sums[0][p];
#pragma unroll
    for (int w = 1; w < GW / 2; ++w) v += sh.sums[w][p];
    gpart[(size_t)blockIdx.x * MLP_NP + p] = v;
  }
  if (threadIdx.x == 0) {
    double l = 0.0;
    for (int w = 0; w < GW; ++w) l += sl[w];
    lpart[blockIdx.x] = l;
    if (bad) bad[blockIdx.x] = sbad;
  }
}

// Sum of the block partials, in FP64: 64 parameters per block, 16 rows of
// partials apart, then the 16 sums in order (6.4 us for the 4.9 MB of 65536
// samples).  The last block adds the losses and the flags.
__global__ __launch_bounds__(1024) void k_mlp_sum(const float* gpart, const double* lpart,
                                                  const int* bad, int nblk, float* grad,
                                                  double* loss, int* any_bad) {
  __shared__ double sh[16][64];
  __shared__ int sbad;
  const int row = threadIdx.x >> 6, col = threadIdx.x & 63;
  const bool last = blockIdx.x == gridDim.x - 1;
  const int p = blockIdx.x * 64 + col;
  if (threadIdx.x == 0) sbad = 0;
  __syncthreads();
  double acc = 0.0;
  if (!last) {
    if (p < MLP_NP)
      for (int b = row; b < nblk; b += 16) acc += gpart[(size_t)b * MLP_NP + p];
  } else {
    for (int b = threadIdx.x; b < nblk; b += 1024) {
      acc += lpart[b];
      if (bad && bad[b]) sbad = 1;
    }
  }
  sh[row][col] = acc;
  __syncthreads();
  if (row != 0) return;
  acc = 0.0;
  for (int r = 0; r < 16; ++r) acc += sh[r][col];
  if (!last) {
    if (p < MLP_NP) grad[p] = (float)acc;
  } else {
    acc = wave_sum(acc);
    if (col == 0) {
      *loss = acc;
      if (any_bad) *any_bad = sbad;
    }
  }
}
constexpr int SUM_BLOCKS = (MLP_NP + 63) / 64 + 1;

// Adam (Kingma & Ba) with bias correction, step t >= 1.
__global__ void k_adam(float* th, float* m, float* v, const float* g, float lr, float b1,
                       float b2, float eps, int t) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= MLP_NP) return;
  const float gp = g[p];
  const float mp = b1 * m[p] + (1.f - b1) * gp;
  const float vp = b2 * v[p] + (1.f - b2) * gp * gp;
  m[p] = mp;
  v[p] = vp;
  const float mh = mp / (1.f - powf(b1, (float)t));
  const float vh = vp / (1.f - powf(b2, (float)t));
  th[p] -= lr * mh / (sqrtf(vh) + eps);
}

// Scratch of tc2_mlp_grad_noalloc: the per-block gradient partials (float,
// TC2_MLP_NOALLOC_MAX_N / GS blocks of MLP_NP) followed by the per-block loss
// partials (double).  Every device the library runs on holds its own copy
// until the process ends.
constexpr int NA_BLOCKS = TC2_MLP_NOALLOC_MAX_N / GS;
static_assert(TC2_MLP_NOALLOC_MAX_N % GS == 0, "whole blocks");
constexpr size_t NA_GPART = (size_t)NA_BLOCKS * MLP_NP * sizeof(float);
constexpr size_t NA_LPART_OFF = (NA_GPART + 255) / 256 * 256;
constexpr size_t NA_BYTES = NA_LPART_OFF + (size_t)NA_BLOCKS * sizeof(double);
static __device__ __align__(256) unsigned char scratch[NA_BYTES];

}  // namespace tc2

using namespace tc2;

namespace {

struct DevMem {
  void* p = nullptr;
  ~DevMem() {
    tc2::dev_free(p);
  }
  hipError_t alloc(size_t n) { return tc2::dev_malloc(&p, n < 256 ? 256 : n); }
  template <typename T> T* as() const { return (T*)p; }
};

#define MLPCHK(x)                                                        \
  do {                                                                   \
    hipError_t e_ = (x);                                                 \
    if (e_ != hipSuccess) return e_ == hipErrorOutOfMemory ? TC2_ENOMEM : TC2_EDEVICE; \
  } while (0)

tc2_status use_device(int device) {
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return TC2_EDEVICE;
  if (device < 0 || device >= ndev) return TC2_EDEVICE;
  if (hipSetDevice(device) != hipSuccess) return TC2_EDEVICE;
  return TC2_OK;
}

bool finite_all(const float* p, long long n) {
  for (long long i = 0; i < n; ++i)
    if (!std::isfinite(p[i])) return false;
  return true;
}

// gradient and loss of the mean loss over rows [0, n) of the device data
// (bad and any_bad: the flags of values that are not finite, or both null)
tc2_status grad_dev(hipStream_t st, const float* th, const float* x, const float* y, long long n,
                    float* gpart, double* lpart, float* grad, double* loss, int* bad = nullptr,
                    int* any_bad = nullptr) {
  const int nblk = (int)((n + GS - 1) / GS);
  hipLaunchKernelGGL(k_mlp_grad, dim3(nblk), dim3(GT), 0, st, th, x, y, n, 1.0 / (double)n, gpart,
                     lpart, bad);
  hipLaunchKernelGGL(k_mlp_sum, dim3(SUM_BLOCKS), dim3(1024), 0, st, gpart, lpart, bad, nblk, grad,
                     loss, any_bad);
  MLPCHK(hipGetLastError());
  return TC2_OK;
}

// Device address of `scratch` on each device, looked up once per device with
// that device current (the array's host-side name is not a device address).
constexpr int NA_MAX_DEVICES = 64;
std::mutex na_lock;
void* na_ptr[NA_MAX_DEVICES] = {};

tc2_status scratch_of(int device, void** out) {
  if (device < 0 || device >= NA_MAX_DEVICES) return TC2_EDEVICE;
  std::lock_guard<std::mutex> g(na_lock);
  if (!na_ptr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TC2_EDEVICE;
    na_ptr[device] = p;
  }
  *out = na_ptr[device];
  return TC2_OK;
}

}  // namespace

extern "C" {

tc2_status tc2_mlp_grad_noalloc(const float* theta, const float* x, const float* y, int64_t n,
                                void* hip_stream, float* grad, double* loss) {
  if (!theta || !x || !y || !grad || !loss || n <= 0) return TC2_EINVAL;
  if (n > TC2_MLP_NOALLOC_MAX_N) return TC2_EINVAL;
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return TC2_EDEVICE;
  void* base = nullptr;
  if (tc2_status s = scratch_of(device, &base); s != TC2_OK) return s;
  float* gpart = (float*)base;
  double* lpart = (double*)((unsigned char*)base + NA_LPART_OFF);
  // every partial the sum reads is written by the gradient kernel first: no
  // clearing is needed
  return grad_dev((hipStream_t)hip_stream, theta, x, y, n, gpart, lpart, grad, loss);
}

tc2_status tc2_mlp_forward(const float* theta, const float* x, int64_t n, int32_t device,
                           float* logits) {
  if (!theta || (n > 0 && (!x || !logits)) || n < 0) return TC2_EINVAL;
  if (!finite_all(theta, MLP_NP) || !finite_all(x, n * MLP_NF)) return TC2_ENAN;
  tc2_status s = use_device(device);
  if (s != TC2_OK) return s;
  if (n == 0) return TC2_OK;
  const ServiceStream svc;
  if (!svc.st) return TC2_EDEVICE;
  MemScope scope;  // waits for the stream at the end of the call
  scope.open(svc.st);
  DevMem dth, dx, dout;
  MLPCHK(dth.alloc(MLP_NP * 4));
  MLPCHK(dx.alloc((size_t)n * MLP_NF * 4));
  MLPCHK(dout.alloc((size_t)n * 4));
  MLPCHK(hipMemcpyAsync(dth.p, theta, MLP_NP * 4, hipMemcpyHostToDevice, svc.st));
  MLPCHK(hipMemcpyAsync(dx.p, x, (size_t)n * MLP_NF * 4, hipMemcpyHostToDevice, svc.st));
  hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, svc.st,
                     dth.as<float>(), dx.as<float>(), (long long)n, dout.as<float>());
  MLPCHK(hipGetLastError());
  MLPCHK(hipMemcpyWithStream(logits, dout.p, (size_t)n * 4, hipMemcpyDeviceToHost, svc.st));
  return TC2_OK;
}

tc2_status tc2_mlp_grad(const float* theta, const float* x, const float* y, int64_t n,
                        int32_t device, float* grad, double* loss) {
  if (!theta || !x || !y || !grad || !loss || n <= 0) return TC2_EINVAL;
  if (tc2_status s = use_device(device); s != TC2_OK)
    return finite_all(theta, MLP_NP) && finite_all(x, n * MLP_NF) && finite_all(y, n) ? s : TC2_ENAN;
  // one allocation: inputs, partials, and the results in one piece; the
  // kernels look for values that are not finite as they read them
  struct Result {
    double loss;
    int bad, pad;
    float grad[MLP_NP];
  } res;
  const long long nblk = (n + GS - 1) / GS;
  size_t size = 0;
  auto place = [&](size_t bytes) {
    const size_t at = size;
    size = (size + bytes + 255) / 256 * 256;
    return at;
  };
  const size_t at_th = place(MLP_NP * 4), at_x = place((size_t)n * MLP_NF * 4),
               at_y = place((size_t)n * 4), at_g = place((size_t)nblk * MLP_NP * 4),
               at_l = place((size_t)nblk * 8), at_b = place((size_t)nblk * 4),
               at_r = place(sizeof(Result));
  const ServiceStream svc;
  if (!svc.st) return TC2_EDEVICE;
  MemScope scope;  // waits for the stream at the end of the call
  scope.open(svc.st);
  DevMem mem;
  MLPCHK(mem.alloc(size));
  char* base = mem.as<char>();
  MLPCHK(hipMemcpyAsync(base + at_th, theta, MLP_NP * 4, hipMemcpyHostToDevice, svc.st));
  MLPCHK(hipMemcpyAsync(base + at_x, x, (size_t)n * MLP_NF * 4, hipMemcpyHostToDevice, svc.st));
  MLPCHK(hipMemcpyAsync(base + at_y, y, (size_t)n * 4, hipMemcpyHostToDevice, svc.st));
  Result* dr = (Result*)(base + at_r);
  if (tc2_status s = grad_dev(svc.st, (float*)(base + at_th), (float*)(base + at_x), (float*)(base + at_y), n,
                              (float*)(base + at_g), (double*)(base + at_l), dr->grad, &dr->loss,
                              (int*)(base + at_b), &dr->bad);
      s != TC2_OK)
    return s;
  MLPCHK(hipMemcpyWithStream(&res, dr, sizeof(Result), hipMemcpyDeviceToHost, svc.st));
  if (res.bad) return TC2_ENAN;
  memcpy(grad, res.grad, sizeof(res.grad));
  *loss = res.loss;
  return TC2_OK;
}

tc2_status tc2_mlp_train(const float* x, const float* y, int64_t n, const tc2_mlp_train_opts* o,
                         float* theta, double* loss_per_epoch) {
  if (!x || !y || !o || !theta || n <= 0) return TC2_EINVAL;
  if (o->epochs < 1 || o->batch < 1 || !(o->lr > 0.f) || !(o->beta1 >= 0.f && o->beta1 < 1.f) ||
      !(o->beta2 >= 0.f && o->beta2 < 1.f) || !(o->adam_eps > 0.f))
    return TC2_EINVAL;
  if (!finite_all(theta, MLP_NP) || !finite_all(x, n * MLP_NF) || !finite_all(y, n)) return TC2_ENAN;
  tc2_status s = use_device(o->device);
  if (s != TC2_OK) return s;
  const long long B = std::min<long long>(o->batch, n);
  const int nblk = (int)((B + GS - 1) / GS);
  const ServiceStream svc;
  if (!svc.st) return TC2_EDEVICE;
  MemScope scope;  // waits for the stream at the end of the call
  scope.open(svc.st);
  DevMem dth, dm, dv, dx, dy, gpart, lpart, dg, dl;
  MLPCHK(dth.alloc(MLP_NP * 4));
  MLPCHK(dm.alloc(MLP_NP * 4));
  MLPCHK(dv.alloc(MLP_NP * 4));
  MLPCHK(dx.alloc((size_t)n * MLP_NF * 4));
  MLPCHK(dy.alloc((size_t)n * 4));
  MLPCHK(gpart.alloc((size_t)nblk * MLP_NP * 4));
  MLPCHK(lpart.alloc((size_t)nblk * 8));
  MLPCHK(dg.alloc(MLP_NP * 4));
  MLPCHK(dl.alloc(8));
  MLPCHK(hipMemcpyAsync(dth.p, theta, MLP_NP * 4, hipMemcpyHostToDevice, svc.st));
  MLPCHK(hipMemsetAsync(dm.p, 0, MLP_NP * 4, svc.st));
  MLPCHK(hipMemsetAsync(dv.p, 0, MLP_NP * 4, svc.st));
  MLPCHK(hipMemcpyAsync(dx.p, x, (size_t)n * MLP_NF * 4, hipMemcpyHostToDevice, svc.st));
  MLPCHK(hipMemcpyAsync(dy.p, y, (size_t)n * 4, hipMemcpyHostToDevice, svc.st));
  int t = 0;
  for (int ep = 0; ep < o->epochs; ++ep) {
    double ep_loss = 0.0;
    for (long long b0 = 0; b0 < n; b0 += B) {
      const long long nb = std::min<long long>(B, n - b0);
      s = grad_dev(svc.st, dth.as<float>(), dx.as<float>() + b0 * MLP_NF, dy.as<float>() + b0, nb,
                   gpart.as<float>(), lpart.as<double>(), dg.as<float>(), dl.as<double>());
      if (s != TC2_OK) return s;
      ++t;
      hipLaunchKernelGGL(k_adam, dim3((MLP_NP + 255) / 256), dim3(256), 0, svc.st, dth.as<float>(),
                         dm.as<float>(), dv.as<float>(), dg.as<float>(), o->lr, o->beta1, o->beta2,
                         o->adam_eps, t);
      MLPCHK(hipGetLastError());
      double bl = 0.0;
      MLPCHK(hipMemcpyWithStream(&bl, dl.p, 8, hipMemcpyDeviceToHost, svc.st));
      ep_loss += bl * (double)nb / (double)n;
    }
    if (loss_per_epoch) loss_per_epoch[ep] = ep_loss;
  }
  MLPCHK(hipMemcpyWithStream(theta, dth.p, MLP_NP * 4, hipMemcpyDeviceToHost, svc.st));
  return TC2_OK;
}

}  // extern "C"
