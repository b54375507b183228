// kernels_ntt.hip -- the transform multiply: kernels and launchers.
#include <algorithm>
#include <cmath>

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

// the three primes side by side (3T threads), for batches that leave waves idle
template <class Z>
__global__ __launch_bounds__(3 * Z::T) void k_mul_ntt3(uint32_t* out, const uint32_t* a, int na, const uint32_t* b,
                                                       int nb, int nout) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int64_t inst = blockIdx.x;
  ntt::wg_mul_ntt3<Z>(out + inst * (int64_t)nout, a + inst * (int64_t)na, na, b + inst * (int64_t)nb, nb, nout,
                      reinterpret_cast<int32_t*>(smem));
}

// The work-groups of one launch: HIP takes fewer than 2^32 work-items, which
// 5.6 million products side by side (768 threads each) exceed; larger batches
// go in several launches.
static int64_t max_groups(int threads) { return 0xffffffffll / threads; }

template <int T, int Q, int R1, int R2>
static int launch_ntt3_size(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb,
                            int64_t batch, int nout, hipStream_t s) {
  typedef ntt::Size<T, Q, R1, R2> Z;
  constexpr size_t lds = ntt::ntt3_lds_bytes<Z>();
  BI_HIP(hipFuncSetAttribute((const void*)k_mul_ntt3<Z>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  for (int64_t first = 0, step = max_groups(3 * T); first < batch; first += step) {
    hipLaunchKernelGGL(k_mul_ntt3<Z>, dim3((unsigned)std::min(step, batch - first)), dim3(3 * T), lds, s,
                       out + first * nout, a + first * na, (int)na, b + first * nb, (int)nb, nout);
    BI_LAUNCH_CHECK();
  }
  return BIGINT_OK;
}

template <int T, int Q, int R1, int R2>
static int launch_ntt_size(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb,
                           int64_t batch, int nout, hipStream_t s) {
  typedef ntt::Size<T, Q, R1, R2> Z;
  BI_HIP(hipFuncSetAttribute((const void*)k_mul_ntt<Z>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)Z::LDS_BYTES));
  for (int64_t first = 0, step = max_groups(T); first < batch; first += step) {
    hipLaunchKernelGGL(k_mul_ntt<Z>, dim3((unsigned)std::min(step, batch - first)), dim3(T), Z::LDS_BYTES, s,
                       out + first * nout, a + first * na, (int)na, b + first * nb, (int)nb, nout);
    BI_LAUNCH_CHECK();
  }
  return BIGINT_OK;
}

// ---- few large products: every prime and factor of a product its own work-group ------
template <class Z>
__global__ __launch_bounds__(Z::T) void k_ntt_quarter(int32_t* y, const uint32_t* a, int na, const uint32_t* b,
                                                      int nb) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int64_t inst = blockIdx.y;
  const int pr = blockIdx.x >> 2, node = blockIdx.x & 3;
  ntt::wg_ntt_quarter<Z>(y + (inst * 12 + blockIdx.x) * Z::M, a + inst * na, na, b + inst * nb, nb, pr, node,
                         reinterpret_cast<int32_t*>(smem));
}

// 1024 points of every factor per work-group of two waves
__global__ __launch_bounds__(128) void k_ntt_join(uint32_t* out, int nout, const int32_t* y, int m,
                                                  uint64_t* strip) {
  const int64_t inst = blockIdx.y;
  ntt::join_strip(out + inst * nout, nout, y + inst * 12 * m, m, (int)(blockIdx.x * 128 + threadIdx.x),
                  strip + inst * (8 * m / ntt::kStripLimbs));
}

// four strips per work-group
__global__ __launch_bounds__(256) void k_ntt_close(uint32_t* out, int nout, int m, const uint64_t* strip) {
  const int64_t inst = blockIdx.y;
  const int W = 4 * m / ntt::kStripLimbs;
  ntt::close_joined(out + inst * nout, nout, W, strip + inst * 2 * W,
                    __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + wave_id()));
}

// At most kQuarterChunk products at a time share the workspace.
constexpr int64_t kQuarterChunk = 256;

template <int Q>
static int launch_ntt_quarters(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb,
                               int64_t batch, int nout, void* ws, hipStream_t s) {
  typedef ntt::Size<256, Q, 16, 16> Z;
  BI_HIP(hipFuncSetAttribute((const void*)k_ntt_quarter<Z>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)Z::LDS_BYTES));
  for (int64_t first = 0; first < batch; first += kQuarterChunk) {
    const unsigned n = (unsigned)std::min(kQuarterChunk, batch - first);
    int32_t* y = reinterpret_cast<int32_t*>(ws);
    uint64_t* strip = reinterpret_cast<uint64_t*>(y + (int64_t)n * 12 * Z::M);
    uint32_t* o = out + first * nout;
    hipLaunchKernelGGL(k_ntt_quarter<Z>, dim3(12, n), dim3(Z::T), Z::LDS_BYTES, s, y, a + first * na, (int)na,
                       b + first * nb, (int)nb);
    BI_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_ntt_join, dim3(Q, n), dim3(128), 0, s, o, nout, y, Z::M, strip);
    BI_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_ntt_close, dim3(2 * Q, n), dim3(256), 0, s, o, nout, Z::M, strip);
    BI_LAUNCH_CHECK();
  }
  return BIGINT_OK;
}

static int quarter_q(int64_t need) { return (int)std::max<int64_t>(3, cdiv(need, 4096)); }

int ntt_quarters_points(int64_t na, int64_t nb) { return 4096 * quarter_q(na + nb); }

size_t ntt_quarters_ws(int64_t na, int64_t nb, int64_t batch) {
  return (size_t)std::min(batch, kQuarterChunk) * quarter_q(na + nb) * (12 * 1024 * 4 + 8 * 16);
}

// Estimated time (us) with the quarters apart: 15 us for one product's three
// launches, then what a product takes of a CU, and 8 us for every further
// chunk.  Against one work-group per product (us, one / quarters): 16384 limbs
// batch 3 106 / 23, 64 113 / 48, 256 135 / 134, 300 230 / 153, 512 241 / 252;
// 8192 limbs 58 / 18, 60 / 29, 72 / 68, 106 / 78, 114 / 120; 5120 limbs
// 43 / 18, 44 / 29, 49 / 58.  The gain is the chip filled by few products
// and the last round of work-groups filled; the price is the trip of the 12
// transforms through memory.
double ntt_quarters_us(int64_t na, int64_t nb, int64_t batch) {
  static const double load[9] = {0, 0, 0, 43, 54, 72, 83, 112, 118};
  if (na + nb <= 8192 || na + nb > 32768) return 1e30;
  return 15.0 + load[quarter_q(na + nb)] * (double)batch / num_cus() + 8.0 * (double)((batch - 1) / kQuarterChunk);
}

int launch_mul_ntt_quarters(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb,
                            int64_t batch, int nout, void* ws, hipStream_t s) {
  switch (quarter_q(na + nb)) {
    case 3: return launch_ntt_quarters<3>(out, a, na, b, nb, batch, nout, ws, s);
    case 4: return launch_ntt_quarters<4>(out, a, na, b, nb, batch, nout, ws, s);
    case 5: return launch_ntt_quarters<5>(out, a, na, b, nb, batch, nout, ws, s);
    case 6: return launch_ntt_quarters<6>(out, a, na, b, nb, batch, nout, ws, s);
    case 7: return launch_ntt_quarters<7>(out, a, na, b, nb, batch, nout, ws, s);
    case 8: return launch_ntt_quarters<8>(out, a, na, b, nb, batch, nout, ws, s);
    default: return BIGINT_EUNSUPPORTED;
  }
}

// ---- which kernel ------------------------------------------------------------------
// The sizes built: serial (one prime after another) and the three primes side
// by side, with what one product takes alone on an idle CU and what it takes
// of a CU in a large batch (us, measured on batches of 1 to 8192).  In
// between, work-groups that fill a CU by themselves go in whole rounds, and of
// the small ones several overlap (1536 limbs side by side: 256 14 us, 512 23,
// 1024 40), though a CU with one more than the others sets the end (1024 limbs
// side by side: 256 12 us, 257 18, 512 18).  Side by side wins wherever waves are idle, and above 3072 points
// also in large batches except at 5120 and 6144 points, whose serial kernels
// fit four work-groups a CU against one (2560-limb products, batch 1024: 73
// against 88 us; batch 256: 35 against 25 us).  Serial kernels below 3072
// points (2048: 5.8 us of a CU) are not built: where a batch would fill them,
// the MFMA multiply is faster (1024 limbs 5.2).  7168 points side by side
// take what 8192 do, and are built for ragged plans only.
struct NttKernel {
  int M;
  bool side;     // three primes side by side
  float lat, load;
};
constexpr NttKernel kNtt[] = {
    {2048, true, 11.5f, 8.2f},   {3072, false, 28.f, 8.9f},   {3072, true, 13.f, 9.5f},
    {4096, true, 15.f, 10.4f},   {5120, false, 31.f, 18.f},   {5120, true, 22.f, 22.f},
    {6144, false, 33.f, 20.f},   {6144, true, 23.f, 23.f},    {8192, true, 25.f, 26.f},
    {10240, false, 45.f, 36.f},  {12288, false, 48.f, 41.f},  {14336, false, 57.f, 53.f},
    {16384, false, 60.f, 53.f},  {20480, false, 80.f, 79.f},  {24576, false, 84.f, 86.f},
    {28672, false, 107.f, 123.f}, {32768, false, 108.f, 122.f}};
constexpr NttKernel kRaggedSide7 = {7168, true, 26.f, 27.f};

int ntt_pick(int64_t na, int64_t nb, int64_t batch, double* us) {
  int best = -1;
  *us = 0.0;
  for (int i = 0; i < (int)(sizeof(kNtt) / sizeof(kNtt[0])); ++i) {
    if (kNtt[i].M < na + nb) continue;
    if (best >= 0 && kNtt[i].M > 2 * kNtt[best].M) break;
    const NttKernel& k = kNtt[i];
    const double x = (double)batch / num_cus();
    const double t = k.M > (k.side ? 4096 : 8192) ? 1.1 * k.lat + k.load * std::max(0.0, std::ceil(x) - 1.0)
                     : k.side ? std::max<double>(k.lat, 0.4 * k.lat + k.load * (0.6 * x + 0.4 * std::ceil(x)))
                                                  : std::max(k.load * x, k.lat + 0.7 * k.load * x);
    if (best < 0 || t < *us) {
      best = i;
      *us = t;
    }
  }
  return best;
}

int ntt_points(int pick, bool* side) {
  *side = kNtt[pick].side;
  return kNtt[pick].M;
}

double ntt_alone_us(int pick) { return kNtt[pick].lat; }

int launch_mul_ntt(uint32_t* out, const uint32_t* a, int64_t na, const uint32_t* b, int64_t nb, int64_t batch,
                   int nout, int pick, hipStream_t s) {
#define NTT(T, Q, R1, R2) return launch_ntt_size<T, Q, R1, R2>(out, a, na, b, nb, batch, nout, s)
#define NTT3(Q) return launch_ntt3_size<256, Q, 16, 16>(out, a, na, b, nb, batch, nout, s)
  if (pick < 0 || pick >= (int)(sizeof(kNtt) / sizeof(kNtt[0])) || na + nb > kNtt[pick].M) return BIGINT_EINVAL;
  if (kNtt[pick].side) {
    switch (kNtt[pick].M) {
      case 2048: NTT3(2);
      case 3072: NTT3(3);
      case 4096: NTT3(4);
      case 5120: NTT3(5);
      case 6144: NTT3(6);
      case 8192: NTT3(8);
    }
  } else {
    switch (kNtt[pick].M) {
      case 3072: NTT(128, 6, 8, 16);
      case 5120: NTT(256, 5, 16, 16);
      case 6144: NTT(256, 6, 16, 16);
      case 10240: NTT(512, 5, 32, 16);
      case 12288: NTT(512, 6, 32, 16);
      case 14336: NTT(512, 7, 32, 16);
      case 16384: NTT(512, 8, 32, 16);
      case 20480: NTT(1024, 5, 32, 32);
      case 24576: NTT(1024, 6, 32, 32);
      case 28672: NTT(1024, 7, 32, 32);
      case 32768: NTT(1024, 8, 32, 32);
    }
  }
#undef NTT
#undef NTT3
  return BIGINT_EUNSUPPORTED;
}

// ============================================================================
// ragged batches: one launch per kernel family, its instances in queue order
// (largest first), one work-group each; the leaf size comes with the queue
// entry.  The families follow what fits a CU: T = 1024 (one work-group), T =
// 512 (two), the side-by-side kernels of 5120 to 8192 points (one) and of up
// to 4096 points (two).
// ============================================================================
enum { kRagged1024 = 1, kRagged512, kRaggedSide, kRaggedSideSmall };

template <int KIND>
struct RaggedFamily;
template <>
struct RaggedFamily<kRagged1024> {
  static constexpr int T = 1024, THREADS = 1024, Q0 = 5, Q1 = 8, R1 = 32, R2 = 32;
  static constexpr bool SIDE = false;
};
template <>
struct RaggedFamily<kRagged512> {
  static constexpr int T = 512, THREADS = 512, Q0 = 5, Q1 = 8, R1 = 32, R2 = 16;
  static constexpr bool SIDE = false;
};
template <>
struct RaggedFamily<kRaggedSide> {
  static constexpr int T = 256, THREADS = 768, Q0 = 5, Q1 = 8, R1 = 16, R2 = 16;
  static constexpr bool SIDE = true;
};
template <>
struct RaggedFamily<kRaggedSideSmall> {
  static constexpr int T = 256, THREADS = 768, Q0 = 2, Q1 = 4, R1 = 16, R2 = 16;
  static constexpr bool SIDE = true;
};

template <class F, int Q>
__device__ __forceinline__ void ragged_one(int q, uint32_t* po, const uint32_t* pa, int na, const uint32_t* pb,
                                           int nb, int32_t* lds) {
  if constexpr (Q <= F::Q1) {
    if (q != Q) {
      ragged_one<F, Q + 1>(q, po, pa, na, pb, nb, lds);
    } else {
      typedef ntt::Size<F::T, Q, F::R1, F::R2> Z;
      if constexpr (F::SIDE) ntt::wg_mul_ntt3<Z>(po, pa, na, pb, nb, na + nb, lds);
      else ntt::wg_mul_ntt<Z>(po, pa, na, pb, nb, na + nb, lds);
    }
  }
}

template <int KIND>
__global__ __launch_bounds__(RaggedFamily<KIND>::THREADS, RaggedFamily<KIND>::SIDE ? 1 : 4) void k_mul_ntt_ragged(
    uint32_t* out, const int64_t* out_off, const uint32_t* a, const int64_t* a_off, const uint32_t* b,
    const int64_t* b_off, const QueueItem* queue) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int64_t i = __builtin_amdgcn_readfirstlane(queue[blockIdx.x].inst);
  const int q = __builtin_amdgcn_readfirstlane(queue[blockIdx.x].cfg);
  ragged_one<RaggedFamily<KIND>, RaggedFamily<KIND>::Q0>(
      q, out + out_off[i], a + a_off[i], (int)(a_off[i + 1] - a_off[i]), b + b_off[i],
      (int)(b_off[i + 1] - b_off[i]), reinterpret_cast<int32_t*>(smem));
}

template <class F, int Q>
static size_t family_lds(int q) {
  if constexpr (Q > F::Q1) return 0;
  else if (q != Q) return family_lds<F, Q + 1>(q);
  else {
    typedef ntt::Size<F::T, Q, F::R1, F::R2> Z;
    return F::SIDE ? ntt::ntt3_lds_bytes<Z>() : Z::LDS_BYTES;
  }
}

static size_t ragged_lds(int kind, int q) {
  switch (kind) {
    case kRagged1024: return family_lds<RaggedFamily<kRagged1024>, 5>(q);
    case kRagged512: return family_lds<RaggedFamily<kRagged512>, 5>(q);
    case kRaggedSide: return family_lds<RaggedFamily<kRaggedSide>, 5>(q);
    default: return family_lds<RaggedFamily<kRaggedSideSmall>, 2>(q);
  }
}

static const void* ragged_kernel_ntt(int kind) {
  switch (kind) {
    case kRagged1024: return (const void*)k_mul_ntt_ragged<kRagged1024>;
    case kRagged512: return (const void*)k_mul_ntt_ragged<kRagged512>;
    case kRaggedSide: return (const void*)k_mul_ntt_ragged<kRaggedSide>;
    default: return (const void*)k_mul_ntt_ragged<kRaggedSideSmall>;
  }
}

static int ragged_threads(int kind) { return kind == kRagged1024 ? 1024 : (kind == kRagged512 ? 512 : 768); }

NttRagged ntt_ragged(int64_t na, int64_t nb) {
  NttRagged r;
  const int64_t need = na + nb;
  if (need > 32768) return r;
  if (need > 16384) r.kind = kRagged1024, r.q = (int)cdiv(need, 4096);
  else if (need > 8192) r.kind = kRagged512, r.q = (int)cdiv(need, 2048);
  else if (need > 4096) r.kind = kRaggedSide, r.q = (int)cdiv(need, 1024);
  else r.kind = kRaggedSideSmall, r.q = std::max(2, (int)cdiv(need, 1024));
  r.lds = ragged_lds(r.kind, r.q);
  const int M = r.q * (r.kind == kRagged1024 ? 4096 : (r.kind == kRagged512 ? 2048 : 1024));
  const NttKernel* k = M == kRaggedSide7.M ? &kRaggedSide7 : kNtt;
  while (k->M != M || k->side != (r.kind >= kRaggedSide)) ++k;   // (every ragged size is in the table)
  r.load = k->load;
  r.lat = k->lat;
  return r;
}

int ntt_ragged_slots(int kind, size_t lds) {
  int per_cu = 1;
  const void* k = ragged_kernel_ntt(kind);
  if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, ragged_threads(kind), lds) != hipSuccess || per_cu < 1)
    per_cu = 1;
  return num_cus() * per_cu;
}

int ntt_ragged_waves(int kind) { return ragged_threads(kind) / 64; }

int launch_mul_ntt_ragged(uint32_t* out, const int64_t* out_off, const uint32_t* a, const int64_t* a_off,
                          const uint32_t* b, const int64_t* b_off, const QueueItem* queue, const RaggedClass& c,
                          hipStream_t s) {
  if (c.count < 1) return BIGINT_OK;
  const int threads = ragged_threads(c.ntt);
  BI_HIP(hipFuncSetAttribute(ragged_kernel_ntt(c.ntt), hipFuncAttributeMaxDynamicSharedMemorySize, (int)c.lds));
  queue += c.first;
  for (int64_t first = 0, step = max_groups(threads); first < c.count; first += step, queue += step) {
    const dim3 gd((unsigned)std::min<int64_t>(step, c.count - first)), bd(threads);
    switch (c.ntt) {
      case kRagged1024:
        hipLaunchKernelGGL(k_mul_ntt_ragged<kRagged1024>, gd, bd, c.lds, s, out, out_off, a, a_off, b, b_off, queue);
        break;
      case kRagged512:
        hipLaunchKernelGGL(k_mul_ntt_ragged<kRagged512>, gd, bd, c.lds, s, out, out_off, a, a_off, b, b_off, queue);
        break;
      case kRaggedSide:
        hipLaunchKernelGGL(k_mul_ntt_ragged<kRaggedSide>, gd, bd, c.lds, s, out, out_off, a, a_off, b, b_off, queue);
        break;
      default:
        hipLaunchKernelGGL(k_mul_ntt_ragged<kRaggedSideSmall>, gd, bd, c.lds, s, out, out_off, a, a_off, b, b_off,
                           queue);
    }
    BI_LAUNCH_CHECK();
  }
  return BIGINT_OK;
}

}  // namespace bi
