// GPTQ rounding for HIGGS (Sec. 3.5): the nearest-point step of Alg. 1
// replaced by the GPTQ error-feedback rounding, in the rotated space, with the
// same output format (codes + fp16 group scales).
//
// Factor: H = X'^T X' over the rotated calibration activations X' (samples x
// in, as higgs_rht_activations writes them), damped by damp * mean(diag H) on
// the diagonal (the usual GPTQ damping), then Hinv = H^-1 and its Cholesky
// factor Hinv = U^T U, all in fp64 (rocBLAS syrk, rocSOLVER potrf / potri /
// potrf). rocSOLVER leaves a column-major lower factor L with Hinv = L L^T;
// read row-major, that buffer is exactly U = L^T.
//
// Quantize: the rotated weights W' and group norms (one kernel), then per
// block of 64 columns the block kernel (rounding, in-block error feedback,
// codes; E takes the block's place in W') and one fp64 GEMM: after block b the
// errors of the last 2^k blocks, 2^k the largest power of two dividing b + 1,
// update the next 2^k blocks' columns. 4096 x 4096, (2,256): 8.3 -> 2.9 ms (64
// block kernels of 24 us, and 1.3 ms of products, of which the one over half
// the row takes 0.7; with one product of all later columns per block they took
// 2.6 ms, bound by reading and writing W' for an inner dimension of 64).

#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <cstdio>
#include <mutex>

#include "internal.h"

namespace higgs {
namespace {

// One rocBLAS handle per (thread, device); rocSOLVER uses the same handle.
rocblas_handle blas_handle(char* msg, int msg_len) {
  struct Slot {
    int device = -1;
    rocblas_handle h = nullptr;
  };
  thread_local Slot slots[16];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) {
    std::snprintf(msg, size_t(msg_len), "no usable HIP device");
    return nullptr;
  }
  Slot& s = slots[dev];
  if (s.h == nullptr) {
    if (rocblas_create_handle(&s.h) != rocblas_status_success) {
      std::snprintf(msg, size_t(msg_len), "rocblas_create_handle failed");
      s.h = nullptr;
      return nullptr;
    }
    s.device = dev;
  }
  return s.h;
}

int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }

}  // namespace

int64_t gptq_factor_workspace_bytes(int64_t samples, int64_t in) {
  return align256(samples * in * 8) + 256;  // fp64 activations + the info word
}

int64_t gptq_quantize_workspace_bytes(int64_t out, int64_t in, int g) {
  return align256(out * in * 8) + align256(out * (in / g) * 8);  // W' / E, group norms
}

int gptq_factor(const float* x_rot, int64_t samples, int64_t in, double damp, double* factor,
                void* workspace, hipStream_t stream, char* msg, int msg_len) {
  rocblas_handle h = blas_handle(msg, msg_len);
  if (!h) return HIGGS_ERR_DEVICE;
  if (rocblas_set_stream(h, stream) != rocblas_status_success) {
    std::snprintf(msg, size_t(msg_len), "rocblas_set_stream failed");
    return HIGGS_ERR_DEVICE;
  }
  double* x64 = static_cast<double*>(workspace);
  rocblas_int* info =
      reinterpret_cast<rocblas_int*>(static_cast<char*>(workspace) + align256(samples * in * 8));
  if (launch_to_f64(x_rot, samples * in, x64, stream) != hipSuccess) {
    std::snprintf(msg, size_t(msg_len), "activation conversion launch failed");
    return HIGGS_ERR_DEVICE;
  }
  // row-major X' [samples][in] is column-major in x samples: H = A A^T
  const double one = 1.0, zero = 0.0;
  const rocblas_int n = rocblas_int(in), k = rocblas_int(samples);
  if (rocblas_dsyrk(h, rocblas_fill_lower, rocblas_operation_none, n, k, &one, x64, n, &zero,
                    factor, n) != rocblas_status_success) {
    std::snprintf(msg, size_t(msg_len), "rocblas_dsyrk failed");
    return HIGGS_ERR_DEVICE;
  }
  if (launch_damp_diag(factor, in, damp, stream) != hipSuccess) {
    std::snprintf(msg, size_t(msg_len), "damping launch failed");
    return HIGGS_ERR_DEVICE;
  }
  const char* steps[3] = {"Cholesky factorisation of H", "inversion of H",
                          "Cholesky factorisation of H^-1"};
  for (int step = 0; step < 3; ++step) {
    const rocblas_status st =
        step == 1 ? rocsolver_dpotri(h, rocblas_fill_lower, n, factor, n, info)
                  : rocsolver_dpotrf(h, rocblas_fill_lower, n, factor, n, info);
    if (st != rocblas_status_success) {
      std::snprintf(msg, size_t(msg_len), "rocSOLVER failed in the %s", steps[step]);
      return HIGGS_ERR_DEVICE;
    }
    rocblas_int host_info = 0;
    if (hipMemcpyAsync(&host_info, info, sizeof(host_info), hipMemcpyDeviceToHost, stream) !=
            hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess) {
      std::snprintf(msg, size_t(msg_len), "reading the factorisation status failed");
      return HIGGS_ERR_DEVICE;
    }
    if (host_info != 0) {
      std::snprintf(msg, size_t(msg_len),
                    "%s failed at column %d: the damped Hessian is not positive definite",
                    steps[step], int(host_info));
      return HIGGS_ERR_INVALID_ARG;
    }
  }
  return HIGGS_OK;
}

int gptq_quantize(const void* w, higgs_dtype dtype, int64_t out, int64_t in, const float* grid,
                  int p, int n, int g, uint64_t seed, const double* factor, uint8_t* codes,
                  uint16_t* scales, void* workspace, hipStream_t stream, char* msg, int msg_len) {
  rocblas_handle h = blas_handle(msg, msg_len);
  if (!h) return HIGGS_ERR_DEVICE;
  if (rocblas_set_stream(h, stream) != rocblas_status_success) {
    std::snprintf(msg, size_t(msg_len), "rocblas_set_stream failed");
    return HIGGS_ERR_DEVICE;
  }
  char* ws = static_cast<char*>(workspace);
  double* wr = reinterpret_cast<double*>(ws);
  double* norms = reinterpret_cast<double*>(ws + align256(out * in * 8));
  if (launch_gptq_prepare(w, dtype, out, in, g, seed, wr, norms, scales, stream) != hipSuccess) {
    std::snprintf(msg, size_t(msg_len), "rotation launch failed");
    return HIGGS_ERR_DEVICE;
  }
  // Blocks of 64 columns left to right. After block b, with 2^k the largest
  // power of two that divides b + 1, the errors of the last 2^k blocks update
  // the next 2^k blocks of columns (fewer at the row's end) in one matrix
  // product: every block's errors reach every later column, each product's
  // inner dimension is as long as what it updates, and W' is read and written
  // log2(in / 64) times in all instead of half of in / 64 times.
  const double minus_one = -1.0, one = 1.0;
  const int64_t nb = in / 64;
  for (int64_t b = 0; b < nb; ++b) {
    if (launch_gptq_block(wr, norms, factor, grid, p, n, out, in, g, 64 * b, codes, stream) !=
        hipSuccess) {
      std::snprintf(msg, size_t(msg_len), "block launch failed at column %lld",
                    (long long)(64 * b));
      return HIGGS_ERR_DEVICE;
    }
    const int64_t len = (b + 1) & -(b + 1);            // blocks whose errors are applied
    const int64_t c0 = 64 * (b + 1 - len);             // their first column
    const int64_t c1 = 64 * (b + 1);                   // the first column updated
    const int64_t cols = std::min(64 * len, in - c1);  // columns updated
    if (cols <= 0) break;
    // column-major views: W'^T[c1:c1+cols, :] (cols x out, ld in) -=
    //   U[c0:c1, c1:c1+cols]^T (cols x K, ld in) * E^T[c0:c1, :] (K x out, ld in)
    if (rocblas_dgemm(h, rocblas_operation_none, rocblas_operation_none, rocblas_int(cols),
                      rocblas_int(out), rocblas_int(c1 - c0), &minus_one, factor + c0 * in + c1,
                      rocblas_int(in), wr + c0, rocblas_int(in), &one, wr + c1,
                      rocblas_int(in)) != rocblas_status_success) {
      std::snprintf(msg, size_t(msg_len), "rocblas_dgemm failed at column %lld", (long long)c1);
      return HIGGS_ERR_DEVICE;
    }
  }
  return HIGGS_OK;
}

}  // namespace higgs
