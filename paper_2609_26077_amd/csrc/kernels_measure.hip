// Error measurement (Appendix E.2: relative error against an fp64 product)
// and the standalone e4m3 codec.
//
// reference_f64_kernel: C_ref = A B in binary64 from fp32 operands, on the
//   fp64 matrix cores.
//   Measurement infrastructure: not on the timed path.
// error partials / totals: per product, sum (C - C_ref)^2 and sum C_ref^2 in
//   binary64 by a fixed grid of workgroups (each a fixed-order strided sum and
//   a fixed LDS tree), then one workgroup per product adds the partials in
//   index order.  No atomics, so results are identical run to run.
// The allocation-free form of the reduction keeps its partials in `scratch`,
//   a static device array of this file (one copy per device).
#include <hip/hip_runtime.h>

#include <mutex>

#include "device.h"
#include "internal.h"

namespace fmm {

namespace {

// C_ref on the fp64 matrix cores (v_mfma_f64_16x16x4_f64: lane l holds A row
// l % 16 and B column l % 16 at contracted position l / 16; register e of the
// result is row 4 e + l / 16, column l % 16).
//
// A workgroup of 2 x 2 waves owns a 64 x 64 tile, each wave TI x TI MFMA
// tiles, so one 4-byte LDS read a lane feeds TI matrix instructions of 64
// cycles.  The operands are staged in fp32, double-buffered in steps of 16
// positions (a row of A every 20 floats and a position of B every 80, so that
// the 16 x 4 reads fall on distinct banks), and widened on the way to the
// matrix core, which is exact.  Bound by the fp64 matrix rate: 59.9 TFLOP/s at
// 8192^3 (18.4 ms) and 58.6 at 4096^3, where the vendor library's fp64 product
// reaches 61.9; an LDS-tiled fma kernel (64 x 64, 4 x 4
// per thread) took 32.7 and 4.23 ms, and 441 us for two 2048 x 1024 x 1536
// products (now 239).
// 128 x 128 tiles (4 x 4 MFMA tiles a wave): 53.9 and 53.7, and 1.4 to 3 times
// slower where they are too few to fill the chip; steps of 32: the same.
constexpr int TI = 2, RT = 32 * TI, RK = 16;

typedef double v4d __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256, 4) void reference_f64_kernel(const float *__restrict__ A,
                                                               const float *__restrict__ B,
                                                               double *__restrict__ C, int64_t M,
                                                               int64_t K, int64_t N, int tiles_n) {
  constexpr int SA = RK + 4, SB = RT + 16;
  constexpr int NA = RT * RK / 256, NSTEP_B = 256 / RT;   // loads per thread and side; B positions per pass
  __shared__ float la[2][RT * SA], lb[2][RK * SB];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = (wave >> 1) * 16 * TI, wn = (wave & 1) * 16 * TI;
  const int c16 = lane & 15, q4 = lane >> 4;
  const int64_t bt = blockIdx.z;
  const int64_t m0 = (int64_t)(blockIdx.x / tiles_n) * RT, n0 = (int64_t)(blockIdx.x % tiles_n) * RT;
  // rows of A and columns of B past the end repeat the last one (their
  // outputs are not stored); positions past K read as zero
  const int ak = t % RK, ar = t / RK, bc = t % RT, bk = t / RT;
  const float *Ab = A + bt * M * K, *Bb = B + bt * K * N + min(n0 + bc, N - 1);
  float sa[NA], sb[NA];
  auto load = [&](int64_t k0) {
    const bool whole = k0 + RK <= K;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int64_t row = min(m0 + ar + (256 / RK) * i, M - 1);
      sa[i] = whole || k0 + ak < K ? Ab[row * K + k0 + ak] : 0.0f;
      const int64_t kb = k0 + bk + NSTEP_B * i;
      sb[i] = whole || kb < K ? Bb[kb * N] : 0.0f;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      la[buf][(ar + (256 / RK) * i) * SA + ak] = sa[i];
      lb[buf][(bk + NSTEP_B * i) * SB + bc] = sb[i];
    }
  };
  v4d acc[TI][TI];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TI; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
  if (K > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  int buf = 0;
  for (int64_t k0 = 0; k0 < K; k0 += RK, buf ^= 1) {
    const bool more = k0 + RK < K;
    if (more) load(k0 + RK);
    const float *pa = la[buf] + (wm + c16) * SA + q4, *pb = lb[buf] + q4 * SB + wn + c16;
#pragma unroll
    for (int kk = 0; kk < RK; kk += 4) {
      double a[TI], b[TI];
#pragma unroll
      for (int i = 0; i < TI; ++i) a[i] = (double)pa[16 * i * SA + kk];
#pragma unroll
      for (int j = 0; j < TI; ++j) b[j] = (double)pb[kk * SB + 16 * j];
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // (the other buffer was last read before the barrier that ended the previous step)
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  double *Cb = C + bt * M * N;
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TI; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t gm = m0 + wm + 16 * i + 4 * e + q4, gn = n0 + wn + 16 * j + c16;
        if (gm < M && gn < N) Cb[gm * N + gn] = acc[i][j][e];
      }
}

constexpr int kRedThreads = 256;
constexpr int kRedBlocks = 512;   // partials per product

// Partials of the allocation-free reduction: kStaticErrorBatch products of
// kRedBlocks (err2, ref2) pairs, 8 MiB.  Every partial is written before it
// is read, so nothing needs clearing between calls.
static __device__ __align__(256) double scratch[kStaticErrorBatch * kRedBlocks * 2];

__device__ __forceinline__ void tree_sum2(double *s0, double *s1, int t) {
  for (int w = kRedThreads / 2; w > 0; w >>= 1) {
    if (t < w) {
      s0[t] += s0[t + w];
      s1[t] += s1[t + w];
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kRedThreads) void error_partials_kernel(const float *__restrict__ C,
                                                                     const double *__restrict__ Cref,
                                                                     double *__restrict__ part,
                                                                     int64_t MN) {
  __shared__ double s0[kRedThreads], s1[kRedThreads];
  const int t = threadIdx.x;
  const int64_t bt = blockIdx.y;
  const float *c = C + bt * MN;
  const double *r = Cref + bt * MN;
  double e2 = 0.0, r2 = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kRedThreads + t; i < MN; i += (int64_t)kRedBlocks * kRedThreads) {
    const double ref = r[i];
    const double d = (double)c[i] - ref;
    e2 = fma(d, d, e2);
    r2 = fma(ref, ref, r2);
  }
  s0[t] = e2;
  s1[t] = r2;
  __syncthreads();
  tree_sum2(s0, s1, t);
  if (t == 0) {
    part[(bt * kRedBlocks + blockIdx.x) * 2] = s0[0];
    part[(bt * kRedBlocks + blockIdx.x) * 2 + 1] = s1[0];
  }
}

__global__ __launch_bounds__(kRedThreads) void error_totals_kernel(const double *__restrict__ part,
                                                                   double *__restrict__ out) {
  __shared__ double s0[kRedThreads], s1[kRedThreads];
  const int t = threadIdx.x;
  const int64_t bt = blockIdx.x;
  double e2 = 0.0, r2 = 0.0;
  for (int i = t; i < kRedBlocks; i += kRedThreads) {
    e2 += part[(bt * kRedBlocks + i) * 2];
    r2 += part[(bt * kRedBlocks + i) * 2 + 1];
  }
  s0[t] = e2;
  s1[t] = r2;
  __syncthreads();
  tree_sum2(s0, s1, t);
  if (t == 0) {
    out[2 * bt] = s0[0];
    out[2 * bt + 1] = s1[0];
  }
}

__global__ __launch_bounds__(256) void e4m3_quantize_kernel(const float *__restrict__ in,
                                                            uint8_t *__restrict__ out, int64_t n) {
  const int64_t i4 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i4 + 3 < n) {
    const float4 v = *reinterpret_cast<const float4 *>(in + i4);
    *reinterpret_cast<uint32_t *>(out + i4) = dev::e4m3_pack4(v.x, v.y, v.z, v.w);
  } else if (i4 < n) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; i4 + k < n; ++k) v[k] = in[i4 + k];
    const uint32_t w = dev::e4m3_pack4(v[0], v[1], v[2], v[3]);
    for (int k = 0; i4 + k < n; ++k) out[i4 + k] = (uint8_t)(w >> (8 * k));
  }
}

// The cast of the power-of-two scale rules: codes of in[i] / s, s = 2^e,
// through the routine the encoder applies to every block with an E8M0 scale.
__global__ __launch_bounds__(256) void e4m3_quantize_pow2_kernel(const float *__restrict__ in,
                                                                 uint8_t *__restrict__ out, int64_t n,
                                                                 float s) {
  const int64_t i4 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i4 + 3 < n) {
    const float4 v = *reinterpret_cast<const float4 *>(in + i4);
    *reinterpret_cast<uint32_t *>(out + i4) = dev::e4m3_pack4_pow2(v.x, v.y, v.z, v.w, s);
  } else if (i4 < n) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; i4 + k < n; ++k) v[k] = in[i4 + k];
    const uint32_t w = dev::e4m3_pack4_pow2(v[0], v[1], v[2], v[3], s);
    for (int k = 0; i4 + k < n; ++k) out[i4 + k] = (uint8_t)(w >> (8 * k));
  }
}

}  // namespace

int launch_reference_f64(int64_t batch, int64_t M, int64_t K, int64_t N, const float *A,
                         const float *B, double *Cref, void *stream) {
  if (batch == 0 || M == 0 || N == 0) return hipSuccess;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int64_t tm = (M + RT - 1) / RT, tn = (N + RT - 1) / RT;
  hipLaunchKernelGGL(reference_f64_kernel, dim3((unsigned)(tm * tn), 1, (unsigned)batch), dim3(256),
                     0, st, A, B, Cref, M, K, N, (int)tn);
  return hipGetLastError();
}

size_t error_stats_scratch_bytes(int64_t batch, int64_t, int64_t) {
  return (size_t)batch * kRedBlocks * 2 * sizeof(double);
}

int launch_error_stats(int64_t batch, int64_t M, int64_t N, const float *C, const double *Cref,
                       double *out, void *scratch, void *stream) {
  if (batch == 0) return hipSuccess;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  double *part = reinterpret_cast<double *>(scratch);
  hipLaunchKernelGGL(error_partials_kernel, dim3(kRedBlocks, (unsigned)batch), dim3(kRedThreads), 0,
                     st, C, Cref, part, M * N);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(error_totals_kernel, dim3((unsigned)batch), dim3(kRedThreads), 0, st, part, out);
  return hipGetLastError();
}

// The device address of `scratch` on the current device, looked up once per
// device (each device holds its own copy of the array at its own address).
// In host code the array's name is only a stand-in for the symbol, never an
// address a kernel may be given.
int static_error_scratch(void **ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

int launch_e4m3_quantize(const float *in, uint8_t *out, int64_t n, void *stream) {
  if (n == 0) return hipSuccess;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int64_t groups = (n + 3) / 4;
  hipLaunchKernelGGL(e4m3_quantize_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st,
                     in, out, n);
  return hipGetLastError();
}

int launch_e4m3_quantize_pow2(const float *in, uint8_t *out, int64_t n, int e, void *stream) {
  if (n == 0) return hipSuccess;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int64_t groups = (n + 3) / 4;
  const uint32_t sbits = (uint32_t)(e + 127) << 23;   // 2^e, e in [-126, 127]
  float s;
  __builtin_memcpy(&s, &sbits, 4);
  hipLaunchKernelGGL(e4m3_quantize_pow2_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st,
                     in, out, n, s);
  return hipGetLastError();
}

}  // namespace fmm
