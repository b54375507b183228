// kernels_ntt.hip -- the transform multiply: kernels and launchers.
#include "internal.hpp"
#include "dev_mul_ntt.hpp"

namespace bi {

// one work-group per product of a uniform batch; 16 waves per CU at every size
template <class Z>
__global__ __launch_bounds__(Z::T, 4) void k_mul_ntt(uint32_t* out, const uint32_t* a, int na, const uint32_t* b,
                                                     int nb, int nout) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int64_t inst = blockIdx.x;
  ntt::wg_mul_ntt<Z>(out + inst * (int64_t)nout, a + inst * (int64_t)na, na, b + inst * (int64_t)nb, nb, nout,
                     reinterpret_cast<int32_t*>(smem));
}

template <int T, int Q, int R1, int R2>
static int launch_ntt_size(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb,
                           int64_t batch, int nout, hipStream_t s) {
  typedef ntt::Size<T, Q, R1, R2> Z;
  BI_HIP(hipFuncSetAttribute((const void*)k_mul_ntt<Z>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)Z::LDS_BYTES));
  hipLaunchKernelGGL(k_mul_ntt<Z>, dim3((unsigned)batch), dim3(T), Z::LDS_BYTES, s, out, a, (int)na, b, (int)nb,
                     nout);
  BI_LAUNCH_CHECK();
  return BIGINT_OK;
}

template <int T, int R1, int R2>
static int launch_ntt_t(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb,
                        int64_t batch, int nout, int q, hipStream_t s) {
  switch (q) {
    case 5: return launch_ntt_size<T, 5, R1, R2>(out, a, na, b, nb, batch, nout, s);
    case 6: return launch_ntt_size<T, 6, R1, R2>(out, a, na, b, nb, batch, nout, s);
    case 7: return launch_ntt_size<T, 7, R1, R2>(out, a, na, b, nb, batch, nout, s);
    default: return launch_ntt_size<T, 8, R1, R2>(out, a, na, b, nb, batch, nout, s);
  }
}

// smallest transform of at least na + nb points: M = 4 q T, T = 64 .. 1024,
// q = 5 .. 8
bool ntt_size(int64_t na, int64_t nb, int* T, int* q) {
  if (na + nb > 32768) return false;
  for (int t = 64; t <= 1024; t *= 2)
    for (int k = 5; k <= 8; ++k)
      if (4 * (int64_t)k * t >= na + nb) {
        *T = t;
        *q = k;
        return true;
      }
  return false;
}

int launch_mul_ntt(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb, int64_t batch,
                   int nout, hipStream_t s) {
  int T, q;
  if (!ntt_size(na, nb, &T, &q)) return BIGINT_EUNSUPPORTED;
  switch (T) {
    case 64: return launch_ntt_t<64, 4, 16>(out, a, na, b, nb, batch, nout, q, s);
    case 128: return launch_ntt_t<128, 8, 16>(out, a, na, b, nb, batch, nout, q, s);
    case 256: return launch_ntt_t<256, 16, 16>(out, a, na, b, nb, batch, nout, q, s);
    case 512: return launch_ntt_t<512, 32, 16>(out, a, na, b, nb, batch, nout, q, s);
    default: return launch_ntt_t<1024, 32, 32>(out, a, na, b, nb, batch, nout, q, s);
  }
}

}  // namespace bi
