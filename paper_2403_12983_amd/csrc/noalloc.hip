// osscar_gram_static: the quadratic form of one small layer, H = X^T X + lambda I and G = H W (Section 3, dense-layer
// paragraph), in one call that allocates nothing.  It is osscar_gram (one chunk plus finalize) for callers that cannot
// allocate device memory: there is no context and no workspace argument; what osscar_gram keeps in the caller's workspace
// during the Gram phase -- the float64 accumulator of H, the partial tiles of cut contractions and a few scalars -- lives in a
// fixed device array of this file instead.
#include "../../include/osscar.h"
#include "internal.h"

#include <algorithm>
#include <mutex>

using namespace osscar;

namespace {

constexpr int64_t ST_MAX = OSSCAR_STATIC_MAX_DIM;      // largest d1 and m
constexpr int64_t ST_ROWS = 1 << 20;                     // calibration rows per launch (the kernel's row index is 32 bits wide)
constexpr size_t ST_H64 = (size_t)ST_MAX * ST_MAX * 8, ST_PART = (size_t)ST_MAX * (8192 + 4 * ST_MAX);      // accumulator, partial tiles
constexpr size_t ST_SMALL = 64 * 1024;                 // scalars and the partial sums of the reductions
constexpr size_t ST_BYTES = ST_H64 + ST_PART + ST_SMALL;
static_assert(ST_BYTES == OSSCAR_STATIC_SCRATCH_BYTES, "the header states the size of the array");

// One copy per GPU, at its own address on each, for as long as the process lives.  In host code this name is only a
// handle for hipGetSymbolAddress: the device address is looked up once per device below and everything else uses that.
static __device__ __align__(256) unsigned char scratch[ST_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

hipError_t scratch_of_current_device(unsigned char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = reinterpret_cast<unsigned char*>(g_scratch_ptr[dev]);
  return hipSuccess;
}

__global__ void st_fill_f64_kernel(double* p, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
// out = (lambda, c0 = <W, G>): DOT_WGS workgroups leave a sum each, the last one to finish adds them in order.  (done: zero before the launch.)
constexpr int DOT_WGS = 64;
__device__ __forceinline__ double dot_block_sum(double v, double* sh) {      // valid in thread 0
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}
__global__ __launch_bounds__(256) void st_dot_kernel(const void* __restrict__ W, int w_bf16, int64_t ldw, const float* __restrict__ G, int d1, int m,
                                                     const double* __restrict__ ridge, double* partial, int* done, double* __restrict__ out) {
  __shared__ double sh[4];
  __shared__ int last;
  double v = 0;
  for (int i = blockIdx.x; i < d1; i += DOT_WGS)
    for (int j = threadIdx.x; j < m; j += 256) {
      const float w = w_bf16 ? __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(W)[(int64_t)i * ldw + j] << 16)
                             : reinterpret_cast<const float*>(W)[(int64_t)i * ldw + j];
      v += (double)w * (double)G[(int64_t)i * m + j];
    }
  const double t = dot_block_sum(v, sh);
  if (threadIdx.x == 0) {
    __hip_atomic_store(partial + blockIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == DOT_WGS - 1;
  }
  __syncthreads();
  if (!last || threadIdx.x >= 64) return;
  double x = __hip_atomic_load(partial + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
  if (threadIdx.x == 0) { out[0] = *ridge; out[1] = x; }
}

osscar_status refuse(osscar_status st, const char* msg) { set_contextless_error(msg); return st; }

}  // namespace

extern "C" osscar_status osscar_gram_static(const void* X_dev, int64_t n, int64_t ldx, int32_t x_dtype, const void* W_dev, int64_t ldw,
                                            int32_t w_dtype, int64_t d1, int64_t m, double lambda_abs, double lambda_rel, float* H_dev,
                                            float* G_dev, double* scalars_dev, void* hip_stream) {
  if (d1 < 1 || m < 1 || n < 0) return refuse(OSSCAR_EINVAL, "osscar_gram_static: d1 and m must be positive and n >= 0");
  if (d1 > ST_MAX || m > ST_MAX)
    return refuse(OSSCAR_ENOMEM, "osscar_gram_static: d1 and m may not exceed OSSCAR_STATIC_MAX_DIM (1024): the fixed scratch array "
                                 "is sized for that; larger layers go through osscar_gram with a caller-provided workspace");
  if ((x_dtype != OSSCAR_F32 && x_dtype != OSSCAR_BF16) || (w_dtype != OSSCAR_F32 && w_dtype != OSSCAR_BF16))
    return refuse(OSSCAR_EINVAL, "osscar_gram_static: unknown dtype");
  if (!W_dev || !H_dev || !G_dev || !scalars_dev || (n > 0 && !X_dev) || ldx < d1 || ldw < m)
    return refuse(OSSCAR_EINVAL, "osscar_gram_static: NULL pointer or leading dimension below the row length");
  unsigned char* base = nullptr;
  if (scratch_of_current_device(&base) != hipSuccess) return refuse(OSSCAR_EHIP, "osscar_gram_static: hipGetSymbolAddress failed");
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  double* H64 = reinterpret_cast<double*>(base);
  // the partial tiles of cut contractions take what the accumulator leaves in front of the scalars
  const size_t h_bytes = ((size_t)d1 * d1 * 8 + 255) / 256 * 256;
  size_t part_bytes = ST_H64 + ST_PART - h_bytes;
  double* part = reinterpret_cast<double*>(base + h_bytes);
  double* scal = reinterpret_cast<double*>(base + ST_H64 + ST_PART);      // 64 scalars, then 2048 partial sums
  double* partial = scal + 64;
  int* done = reinterpret_cast<int*>(scal + 32);
  const int D = (int)d1, M = (int)m;
  const bool xbf = x_dtype == OSSCAR_BF16;
  // the array keeps the last call's contents; everything in it is written before it is read
  hipError_t e = hipSuccess;
  const size_t esz = xbf ? 2 : 4;
  if (n == 0) hipLaunchKernelGGL(st_fill_f64_kernel, dim3((unsigned)std::min<int64_t>((d1 * d1 + 1023) / 1024, 4096)), dim3(256), 0, s, H64, d1 * d1, 0.0);
  for (int64_t r0 = 0; r0 < n && e == hipSuccess; r0 += ST_ROWS) {
    Gemm64 g{};      // H64 (+)= X^T X on the lower triangle, float64 sums on the matrix cores
    g.M = D; g.N = D; g.K = (int)std::min<int64_t>(ST_ROWS, n - r0); g.lower = 1;
    g.A = g.B = reinterpret_cast<const char*>(X_dev) + (size_t)r0 * ldx * esz; g.lda = g.ldb = ldx; g.a_kind = g.b_kind = xbf ? OPK_K_BF16 : OPK_K_F32;
    g.Cin = r0 ? H64 : nullptr; g.ldcin = D; g.C = H64; g.ldc = D; g.c_is_f64 = 1; g.alpha = 1.0; g.beta = 1.0; g.ws = part; g.ws_bytes = part_bytes;
    e = launch_gemm64_logged(g, s);
  }
  // The call's time is the chain of its launches (nine of them took 52 us for 4096 rows of 288 columns, six take 41): the ridge is formed where H is,
  // W is read as it comes, and one launch forms c0 = Tr(W^T G) and the two results.
  if (e == hipSuccess) e = launch_finalize_ridge(H64, H_dev, D, lambda_abs, lambda_rel, scal + 1, s, done);
  bool wbf = w_dtype == OSSCAR_BF16;
  {      // W where G goes: a float32 copy of it, in front of the partial tiles
    const char *w = reinterpret_cast<const char*>(W_dev), *g = reinterpret_cast<const char*>(G_dev);
    if (w < g + (size_t)d1 * m * 4 && g < w + ((size_t)(d1 - 1) * ldw + m) * (wbf ? 2 : 4)) {
      const size_t copy_bytes = ((size_t)d1 * m * 4 + 255) / 256 * 256;
      if (e == hipSuccess) e = launch_convert_to_f32(W_dev, wbf, d1, m, ldw, reinterpret_cast<float*>(part), s);
      W_dev = part; ldw = m; wbf = false;
      part = reinterpret_cast<double*>(base + h_bytes + copy_bytes); part_bytes -= copy_bytes;
    }
  }
  if (e == hipSuccess) {
    Gemm64 g{};      // G = H W (H is symmetric: its rows serve as the columns that the product contracts)
    g.M = D; g.N = M; g.K = D; g.A = H_dev; g.lda = D; g.a_kind = OPK_K_F32; g.B = W_dev; g.ldb = ldw; g.b_kind = wbf ? OPK_K_BF16 : OPK_K_F32;
    g.C = G_dev; g.ldc = M; g.alpha = 1.0; g.ws = part; g.ws_bytes = part_bytes;
    e = launch_gemm64_logged(g, s);
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(st_dot_kernel, dim3(DOT_WGS), dim3(256), 0, s, W_dev, wbf ? 1 : 0, ldw, G_dev, D, M, scal + 1, partial, done, scalars_dev);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return refuse(OSSCAR_EHIP, hipGetErrorString(e));
  return OSSCAR_OK;
}
