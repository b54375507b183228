// kernels_div.hip -- division kernels: one work-group per division, the
// divisions taken in queue order (largest first).
#include <algorithm>
#include <cmath>
#include <mutex>

#include "internal.hpp"
#include "dev_divmod.hpp"

namespace bi {

// Threads of a division work-group: at most kDivThreads (the register budget
// is that of 4 waves per SIMD).
constexpr int kDivThreads = 512;

int64_t div_product_limbs(int64_t nu, int64_t nv) { return div::product_limbs(nu, nv); }

// Uniform batches pass null offsets and the limb counts nu / nv; ragged
// batches pass prefix offsets.  queue == nullptr means instance t is item t.
// Work-group g of a launch takes item first + g and workspace slot g.  Work-
// groups are dispatched in index order, so the items run as a list schedule
// in queue order.  (A persistent loop pulling items with an atomic was
// measured 11% slower on 512 ragged divisions: the loop made the compiler
// keep loop-invariant values live across the whole division.)
// INV is the shifted-inverse diagnostic: q[i] = floor(B^h_inv / v).
// adjust (nullable): 4 int64 per instance, the division's counters (Newton
// steps, fix-up unit steps, quotient corrections, MFMA multiply-accumulates).
template <bool INV>
__global__ __launch_bounds__(kDivThreads, 4) void k_divmod(uint32_t* q, const int64_t* q_off, uint32_t* r,
                                                const int64_t* r_off, int32_t* status,
                                                const uint32_t* u, const int64_t* u_off, int nu,
                                                const uint32_t* v, const int64_t* v_off, int nv,
                                                const int32_t* queue, int64_t first, int64_t nitems,
                                                uint32_t* ws, int cap_u, int cap_v, int prod, int h_inv,
                                                int64_t* adjust) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ div::Shared sh;
  const int64_t t = first + blockIdx.x;
  if (t >= nitems) return;
  uint32_t* myws = ws + (size_t)blockIdx.x * div::div_ws_limbs(cap_u, cap_v);
  const div::Bufs bf = div::carve_bufs(myws, cap_u, cap_v);
  const int64_t i = queue ? (int64_t)__builtin_amdgcn_readfirstlane(queue[t]) : t;
  int64_t uo, vo, qo, ro;
  int lu, lv, lq, lr;
  if (u_off) {
    uo = u_off[i]; lu = (int)(u_off[i + 1] - uo);
    vo = v_off[i]; lv = (int)(v_off[i + 1] - vo);
    qo = q_off[i]; lq = (int)(q_off[i + 1] - qo);
    ro = r_off ? r_off[i] : 0; lr = r_off ? (int)(r_off[i + 1] - ro) : 0;
  } else {
    lu = nu; lv = nv;
    uo = i * (int64_t)nu; vo = i * (int64_t)nv;
    lq = INV ? h_inv + 1 : nu; qo = i * (int64_t)lq;
    lr = nv; ro = i * (int64_t)nv;
  }
  int64_t cnt[4] = {0, 0, 0, 0};
  const int st = div::wg_divmod<INV>(q + qo, lq, r ? r + ro : nullptr, lr, u ? u + uo : nullptr, lu, v + vo, lv,
                                     bf, &sh, smem, h_inv, prod, cnt);
  if (threadIdx.x == 0) {
    if (status) status[i] = st;
    if (adjust) {
#pragma unroll
      for (int j = 0; j < 4; ++j) adjust[4 * i + j] = cnt[j];
    }
  }
}

size_t div_ws_bytes(int cap_u, int cap_v, int slots) {
  return (size_t)slots * div::div_ws_limbs(cap_u, cap_v) * 4;
}

static size_t div_lds_bytes(const DivCfg& c) {
  // (at least what the small-operand product and the one-wave steps need)
  return std::max<size_t>(mfma::lds_bytes_sum(c.prod, c.threads / 64, div::kP),
                          std::max(div::kSmallMulLds, div::kEarlyLds));
}

// Dividend limbs of the division by half as many limbs that does as much work.
double div_size(int64_t work) { return std::sqrt((double)work / 1.5); }

// A division is mostly a chain of short passes that wait on memory and on one
// another, and more of them on a CU hardly slow one another down (2048 / 1024
// limbs, 64 threads: one 182 us, 16 per CU 360).  So the work-group is the
// largest useful one that still lets the whole batch run at once (2048 / 1024
// limbs, us with 64 / 128 / 256 / 512 threads: batch 1 182 / 142 / 127 / 130,
// 1024 217 / 185 / 195 / 334, 4096 360 / 470 / 708 / 1247), and where none
// does, the one that finishes the most of them: half the threads take
// 1 + 0.16 log2(size / 8 threads) of the time, and are worth it only if the
// LDS lets that many more in (8192 / 4096 limbs, batch 2048: 4 per CU with 256
// threads 1090 us, 6 with 128 1346; 8192 / 6144, batch 1500: 4 with 256 713, 5
// with 64 1565; 16384 / 8192, batch 700: 2 with 512 1224, 3 with 128 2491).
// Up to some 4096 limbs, where caches hold their data, running all at once is
// worth it too (4096 / 2048, batch 2500: 8 with 128 627, 11 with 64 552).
// size: the largest division's (div_size).  count: the divisions that can be
// under way together, those of a ragged batch each by its time against the
// largest's, near twice the root of their sizes' ratio up to one (two in a row
// must fit beside the largest): what is done beside the largest needs no place
// of its own (600 of 64..16384 limbs by half as many: 512 threads, 2 per CU,
// 499 us; 128 threads, 3 per CU, 1094).
DivCfg div_cfg(int cap_u, int cap_v, int64_t prod, double size, double count) {
  DivCfg best{cap_u, cap_v, (int)prod, 0, 0};
  double slower = 1.0;   // than with best.threads
  for (int t = cap_u <= 724 ? 128 : (cap_u <= 2896 ? 256 : kDivThreads); t >= 64; t /= 2) {
    DivCfg c{cap_u, cap_v, (int)prod, t, 0};
    // work-groups that fit one CU: the kernel is built for 4 waves per SIMD (16
    // per CU), so that many waves (over the work-group's) and then the LDS decide
    const size_t per = div_lds_bytes(c) + sizeof(div::Shared) + 64;
    c.per_cu = std::min<int>(16 / (t / 64), (int)(163840 / per));
    if (best.per_cu > 0) slower *= 1.0 + 0.16 * std::max(0.0, std::log2(size / (8 * t)));
    const bool all = size < 4500 && num_cus() * c.per_cu >= count;
    if (c.per_cu > best.per_cu * (all ? 1.0 : slower)) {
      best = c;
      slower = 1.0;
    }
    if (num_cus() * best.per_cu >= count) break;
  }
  return best;
}

// divisions per launch, a workspace slot each: 8 rounds of those resident, or
// what 640 MiB hold, but at least two rounds
int div_chunk(const DivCfg& c, int64_t batch) {
  const int64_t resident = (int64_t)num_cus() * c.per_cu;
  const int64_t fit = ((int64_t)640 << 20) / (int64_t)div_ws_bytes(c.cap_u, c.cap_v, 1);
  return (int)std::max<int64_t>(1, std::min(batch, std::min(8 * resident, std::max(2 * resident, fit))));
}

// ---- workspace of the allocation-free division (bigint_divmod_noalloc) ----------
// A file-scope device array, one copy per GPU, held until the process ends.
// Every call on a GPU shares that GPU's copy (calls that overlap on one GPU
// race); the division needs none of it cleared.  In host code the array's
// name is only a stand-in: its device address comes from
// hipGetSymbolAddress, looked up once per device and kept.
constexpr size_t kDivScratchBytes = (size_t)128 << 20;
__device__ __align__(256) uint8_t scratch[kDivScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

int div_scratch(void** ptr, size_t* bytes) {
  int dev = 0;
  BI_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return BIGINT_EUNSUPPORTED;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    BI_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return BIGINT_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  *bytes = kDivScratchBytes;
  return BIGINT_OK;
}

int launch_divmod(uint32_t* q, const int64_t* q_off, uint32_t* r, const int64_t* r_off,
                  int32_t* status, const uint32_t* u, const int64_t* u_off, int nu,
                  const uint32_t* v, const int64_t* v_off, int nv, const int32_t* queue,
                  int64_t nitems, void* ws, const DivCfg& cfg, int chunk, int h_inv,
                  int64_t* adjust, hipStream_t s) {
  const size_t lds = div_lds_bytes(cfg);
  if (cfg.per_cu < 1) return BIGINT_EUNSUPPORTED;
  if (chunk < 1) return BIGINT_EINVAL;
  const auto kernel = h_inv >= 0 ? k_divmod<true> : k_divmod<false>;
  BI_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lds));
  // chunks run one after another on the stream, so a workspace slot is never
  // held by two live work-groups
  for (int64_t first = 0; first < nitems; first += chunk) {
    const int64_t g = std::min<int64_t>(chunk, nitems - first);
    hipLaunchKernelGGL(kernel, dim3((unsigned)g), dim3((unsigned)cfg.threads), lds, s, q, q_off, r, r_off,
                       status, u, u_off, nu, v, v_off, nv, queue, first, nitems,
                       reinterpret_cast<uint32_t*>(ws), cfg.cap_u, cfg.cap_v, cfg.prod, h_inv, adjust);
    BI_LAUNCH_CHECK();
  }
  return BIGINT_OK;
}

}  // namespace bi
