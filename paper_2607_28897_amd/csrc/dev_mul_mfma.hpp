// dev_mul_mfma.hpp -- the MFMA-split multiply: 7-bit (or signed 8-bit)
// digits, int8 MFMA Toeplitz tiles, int32 accumulation, 64-bit recombination
// and a carry scan.
//
// What is computed is the quadratic formula of Section 5.2,
// c_k = sum_{i+j=k} alpha_i beta_j, over the 7-bit digits alpha, beta of the
// operands (digit k = bits [7k, 7k+7)), followed by a * b = sum_k c_k 2^(7k).
// Every c_k is at most min(Na, Nb) * 127^2, below 2^31 for up to 133,144
// digits, so int32 accumulation is exact with no floating point anywhere.
//
// Tiling (v_mfma_i32_16x16x64_i8, D[16x16] += A[16x64] B[64x16]):
//   A_Z[r][s] = alpha[Z + 16r - s]   (a Toeplitz slice of alpha)
//   B_Y[s][p] = beta [Y + s + p]     (overlapping windows of beta)
//   (A_Z B_Y)[r][p] = sum_{s<64} alpha[Z+16r-s] beta[Y+p+s]
// is the part of c[Z+Y+16r+p] whose beta index lies in [Y+p, Y+p+64).  With
// Z + Y = 256w fixed the 16x16 outputs are the "strip" c[256w .. 256w+256),
// and summing over all Y = 64 * integer covers every beta index once.
//   Write Y = 256y + 64rho (phase rho in 0..3) and Z = 256x - 64rho; then
// strip w = x + y.  A wave owns P consecutive strips w0..w0+P-1 (one int32
// accumulator tile each) and, per phase, walks y: strip w0+i needs A tile
// x = w0+i-y, so one step needs one new A tile and one B tile for P MFMAs;
// the other P-1 A tiles are still in registers from the previous steps (a
// ring of P tiles).  Loads per MFMA: 2/P tiles.
//
// Register layout (lane l, idx = l & 15, grp = l >> 4; operand byte t):
//   A lane holds alpha[Z + 16 idx - 16 grp - t]: 16 contiguous bytes of the
//     reversed digit array, one aligned ds_read_b128.
//   B lane holds beta[Y + idx + 16 grp + t]: 16 bytes at an offset of idx
//     bytes, assembled from 5 aligned dwords with v_alignbyte.
// Both operands use the same (grp, t) <-> contraction index map, so the
// MFMA's own K ordering inside a lane does not matter.  The result tile
// holds column p = l & 15, rows 4 (l >> 4) + v in register v.
//
// Recombination: c_k sits at bit 7k.  A strip of 256 coefficients covers
// exactly 56 limbs (7*256 = 56*32), so strips are limb-aligned.  Per strip a
// wave forms the 57 column sums X_j (lo 32 bits of every c_k 2^(7k - 32j)
// whose low bit falls in limb j, plus the high parts from limb j-1; each
// X_j < 2^35), splits X_j = L_j + 2^32 H_j, adds L + (H shifted up one
// limb) with a one-bit ballot carry scan, writes the 56 limbs and keeps the
// 57th column (with its carry) as the strip's carry word C_w.  A final
// work-group carry scan adds every C_w at limb 56(w+1).
//
// Signed 8-bit digits (DW = 8).  The digits are the bytes of a + C less 128
// each, C = sum_i 128 256^i, in [-128, 127], and the carry out of that sum
// as one more digit: their sum is a (|alpha beta| <= 2^14, so int32 is exact
// up to 131,071 digits).  A strip's 256 coefficients are 64 limbs; limb j
// takes X_j = sum_t c_{4j+t} 2^(8t), |X_j| < 2^55, and the spill of limb 63
// is the strip's carry word.
#pragma once

#include "common.hpp"
#include "dev_addsub.hpp"

namespace bi {
namespace mfma {

constexpr int kPadA = 320;  // zero bytes on both sides of reversed alpha (>= 303)
constexpr int kPadA32 = 1040;  // the same for 32x32 tiles (an A tile spans 1023 digits)
constexpr int kPadB = 64;   // zero bytes before beta (a tile reads from Y >= -64)
constexpr int kPadBt = 96;  // zero bytes after beta (reads reach Y + 80)
constexpr int kStrip = 256; // coefficients per strip

// limbs per strip of 256 coefficients: 7 * 256 / 32 and 8 * 256 / 32
template <int DW>
__host__ __device__ constexpr int strip_limbs() { return 8 * DW; }

// 7-bit digits of an n-limb integer
__host__ __device__ inline int ndigits(int n) { return (32 * n + 6) / 7; }

template <int DW>
__host__ __device__ inline int ndigits_w(int n) { return DW == 8 ? 4 * n : ndigits(n); }

struct Geo {
  int na, nb, Na, Nb;
  int QA;   // Abuf[q] = alpha[QA - q]
  int SA;   // bytes of Abuf
  int SB;   // bytes of Bbuf; Bbuf[kPadB + j] = beta[j]
  int W;    // strips
  int nout; // na + nb
};

// nout < na + nb asks for the product mod B^nout only: the strips past limb
// nout are not computed (carries only move up, so the low limbs are exact).
// TS: the MFMA tile (16: 16x16x64, 32: 32x32x32), which sets the padding.
template <int DW, int TS = 16>
__host__ __device__ inline Geo make_geo(int na, int nb, int nout = -1) {
  constexpr int kPA = TS == 32 ? kPadA32 : kPadA;
  Geo g;
  g.na = na; g.nb = nb;
  g.Na = ndigits_w<DW>(na); g.Nb = ndigits_w<DW>(nb);
  g.QA = ((g.Na - 1 + kPA) + 15) & ~15;
  g.SA = ((g.QA + kPA + 1) + 15) & ~15;
  g.SB = ((kPadB + g.Nb + kPadBt) + 15) & ~15;
  const int K = g.Na + g.Nb - 1;
  g.W = (K + kStrip - 1) / kStrip;
  g.nout = (nout < 0 || nout > na + nb) ? na + nb : nout;
  g.W = min(g.W, (g.nout + strip_limbs<DW>() - 1) / strip_limbs<DW>());
  return g;
}

// LDS layout: [Abuf SA][Bbuf SB][per-wave scratch 1 KiB each][strip carries
// 8W][with lead (8-bit digits): every strip's limbs 0-1, 8W][band order
// 2*NB][misc 128]
template <int DW, int TS = 16>
__host__ __device__ inline size_t lds_bytes(int na, int nb, int nwaves, int P, bool lead = false) {
  const Geo g = make_geo<DW, TS>(na, nb);
  const int NB = (g.W + P - 1) / P;
  return (size_t)g.SA + g.SB + (size_t)nwaves * 1024 + (size_t)((DW == 8 && lead) ? 16 : 8) * g.W +
         (size_t)((2 * NB + 15) & ~15) + 128;
}

// enough for any product of operands of na + nb = n limbs in all (signed digits)
__host__ __device__ inline size_t lds_bytes_sum(int n, int nwaves, int P) {
  const int W = n / strip_limbs<8>() + 1, NB = (W + P - 1) / P;
  return (size_t)4 * n + 2 * kPadA + kPadB + kPadBt + 64 + (size_t)nwaves * 1024 + (size_t)8 * W +
         (size_t)((2 * NB + 15) & ~15) + 128;
}

struct Lds {
  uint8_t* A;
  uint8_t* B;
  int32_t* wscr;     // this wave's 256 ints
  int32_t* scr;      // all waves' scratch (256 ints per wave)
  uint64_t* carry;   // W words
  uint64_t* lead = nullptr;  // nullable, W words: limbs 0-1 of every strip as its output wrote
                             // them, so the closing scan need not read them back from out
  uint16_t* order;   // NB entries
  uint32_t* misc;    // [0] band counter, [1..16] scan scratch (32 words)
};

// lead: carve the strips' limbs 0-1 area (8-bit digits; the LDS must have
// been sized by lds_bytes with lead)
template <int DW>
__device__ __forceinline__ Lds carve(char* smem, const Geo& g, int P, bool lead) {
  Lds s;
  const int NB = (g.W + P - 1) / P;
  char* p = smem;
  s.A = reinterpret_cast<uint8_t*>(p); p += g.SA;
  s.B = reinterpret_cast<uint8_t*>(p); p += g.SB;
  s.scr = reinterpret_cast<int32_t*>(p);
  s.wscr = s.scr + wave_id() * 256; p += num_waves() * 1024;
  s.carry = reinterpret_cast<uint64_t*>(p); p += 8 * g.W;
  if (DW == 8 && lead) {
    s.lead = reinterpret_cast<uint64_t*>(p);
    p += 8 * g.W;
  }
  s.order = reinterpret_cast<uint16_t*>(p); p += (2 * NB + 15) & ~15;
  s.misc = reinterpret_cast<uint32_t*>(p);
  return s;
}

// Four consecutive 7-bit digits k0..k0+3 of the n-limb integer a (0 outside
// [0, 32n) bits), packed low digit first: a 28-bit window of at most two
// adjacent limbs.
__device__ __forceinline__ uint32_t digits4(const uint32_t* __restrict__ a, int n, int k0) {
  // branch-free so that the loads of consecutive calls can be batched: the
  // limb indices are clamped and the values masked instead
  const int kc = max(k0, 0);
  const int bit = 7 * kc;
  const int l = bit >> 5, sft = bit & 31;
  const uint32_t lo = a[min(l, n - 1)] & (l < n ? 0xffffffffu : 0u);
  const uint32_t hi = a[min(l + 1, n - 1)] & (l + 1 < n ? 0xffffffffu : 0u);
  const uint32_t v = (uint32_t)((((uint64_t)hi << 32) | lo) >> sft);
  const uint32_t w =
      (v & 0x7fu) | ((v << 1) & 0x7f00u) | ((v << 2) & 0x7f0000u) | ((v << 3) & 0x7f000000u);
  // k0 < 0: digits k0..-1 are padding zeros, the window at 0 moves up
  return k0 >= 0 ? w : (k0 <= -4 ? 0u : w << (8 * -k0));
}

// Stage the reversed 7-bit digits of a and the digits of b into LDS (zero
// padded).  Abuf[q] = alpha[QA - q]: dword d holds digits QA-4d-3 .. QA-4d,
// byte-reversed.
__device__ __forceinline__ void stage7(const Lds& s, const Geo& g, const uint32_t* __restrict__ a,
                                       const uint32_t* __restrict__ b) {
  uint32_t* A32 = reinterpret_cast<uint32_t*>(s.A);
  uint32_t* B32 = reinterpret_cast<uint32_t*>(s.B);
  const int nA = g.SA / 4, nB = g.SB / 4;
#pragma unroll 8
  for (int d = threadIdx.x; d < nA; d += blockDim.x) {
    const int k0 = g.QA - 4 * d - 3;
    // digits at index >= Na come out 0 because the bits past the top limb are 0
    A32[d] = __builtin_bswap32(digits4(a, g.na, k0));
  }
#pragma unroll 8
  for (int d = threadIdx.x; d < nB; d += blockDim.x) B32[d] = digits4(b, g.nb, 4 * d - kPadB);
}

// y range of phase rho for the band starting at strip w0 (P strips).
struct Range { int lo, hi, xlo, xhi; };

__device__ __forceinline__ Range band_range(const Geo& g, int w0, int P, int rho) {
  Range r;
  // B tile covers beta[Y .. Y+78]; it is nonzero iff that meets [0, Nb)
  // (arithmetic shifts: floors; x + 255 for the ceilings)
  const int yb_lo = (177 - 64 * rho) >> 8;
  const int yb_hi = (g.Nb - 1 - 64 * rho) >> 8;
  // A tile covers alpha[Z-63 .. Z+240]; nonzero iff that meets [0, Na)
  r.xlo = (64 * rho + 15) >> 8;
  r.xhi = (g.Na + 62 + 64 * rho) >> 8;
  r.lo = max(yb_lo, w0 - r.xhi);
  r.hi = min(yb_hi, w0 + P - 1 - r.xlo);
  return r;
}

__device__ __forceinline__ int band_cost(const Geo& g, int band, int P) {
  int c = 0;
  for (int rho = 0; rho < 4; ++rho) {
    const Range r = band_range(g, band * P, P, rho);
    c += max(0, r.hi - r.lo + 1);
  }
  return c;
}

// A tile x of phase rho.  Tiles entirely outside alpha read the zero padding
// at the start of Abuf, so no branch is needed.
__device__ __forceinline__ v4i load_A(const uint8_t* Abuf, const Geo& g, int x, int rho,
                                      const Range& r) {
  const int lane = lane_id();
  // the scalar part of the address (240: every lane inside the low padding)
  const int at = (unsigned)(x - r.xlo) <= (unsigned)(r.xhi - r.xlo) ? g.QA + 64 * rho - 256 * x : 240;
  const int addr = at + 16 * ((lane >> 4) - (lane & 15));
  return *reinterpret_cast<const v4i*>(Abuf + addr);
}

// B tile y of phase rho in two halves: the five aligned dwords a lane needs
// (issued early) and their byte alignment into the operand (done late).
struct BRaw {
  uint32_t d[5];
};

__device__ __forceinline__ BRaw load_B_raw(const uint8_t* Bbuf, int y, int rho) {
  const int lane = lane_id();
  const int p = lane & 15;
  const int Y = 256 * y + 64 * rho;
  const uint32_t* src =
      reinterpret_cast<const uint32_t*>(Bbuf + kPadB + Y + 16 * (lane >> 4) + 4 * (p >> 2));
  BRaw b;
#pragma unroll
  for (int i = 0; i < 5; ++i) b.d[i] = src[i];
  return b;
}

__device__ __forceinline__ v4i align_B(const BRaw& b) {
  const uint32_t sh = lane_id() & 3;
  v4i v;
  v.x = (int)__builtin_amdgcn_alignbyte(b.d[1], b.d[0], sh);
  v.y = (int)__builtin_amdgcn_alignbyte(b.d[2], b.d[1], sh);
  v.z = (int)__builtin_amdgcn_alignbyte(b.d[3], b.d[2], sh);
  v.w = (int)__builtin_amdgcn_alignbyte(b.d[4], b.d[3], sh);
  return v;
}

// One phase of one band: acc[i] += sum over the y range of A(w0+i-y) B(y).
// Software pipeline per step: the step's P MFMAs run on the B tile aligned at
// the end of the previous step; the raw dwords of the next B tile were loaded
// one step earlier, and the one new A tile goes into the ring slot that the
// first MFMA of the step has just read.
//
// Band edges: where the low end of the band's y range is set by the A
// operand (the upper half of the product), strip i's first useful step is i,
// so the first P-1 steps hold a staircase of MFMAs on all-zero A tiles.
// There the first P steps run as a "ramp" block that leaves those MFMAs out
// at compile time.  (The mirror staircase at the high end of the range, in
// the lower half of the product, is kept: walking those ranges downwards
// with reversed accumulators measured slower, its extra registers costing
// more than the MFMAs it saves.)
template <int P>
__device__ __forceinline__ void band_phase(v4i (&acc)[P], const Lds& s, const Geo& g, int w0,
                                           int rho) {
  const Range r = band_range(g, w0, P, rho);
  const int L = r.hi - r.lo + 1;
  if (L <= 0) return;
  const int xb = w0 - r.lo;  // strip i at step u uses x = xb + i - u
  // the low end of the range is set by the A operand: strip i starts at step i
  const bool ramp = L >= 2 * P && r.lo == w0 - r.xhi;
  v4i ring[P];
#pragma unroll
  for (int i = 0; i < P; ++i) ring[i] = load_A(s.A, g, xb + i, rho, r);
  v4i Bc = align_B(load_B_raw(s.B, r.lo, rho));
  BRaw raw = load_B_raw(s.B, min(r.lo + 1, r.hi), rho);

  // one step (st = step mod P and the ramp flag known at compile time).  The
  // next B tile is aligned into a second register set half-way through the
  // step, so the step boundary carries no VALU -> MFMA dependency.
  auto step_fn = [&](const int step, const int st, const bool rmp) __attribute__((always_inline)) {
    auto mma = [&](int i) __attribute__((always_inline)) {
      if (!rmp || i <= st)
        acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ring[(P + i - st) % P], Bc, acc[i], 0, 0, 0);
    };
    // strip P-1 first: its slot is the one the next step's new tile takes
    mma(P - 1);
    ring[(2 * P - 1 - st) % P] = load_A(s.A, g, xb - step - 1, rho, r);
#pragma unroll
    for (int i = P - 2; i >= P / 2; --i) mma(i);
    __builtin_amdgcn_sched_barrier(0);
    const v4i Bn = align_B(raw);
    raw = load_B_raw(s.B, min(r.lo + step + 2, r.hi), rho);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = P / 2 - 1; i >= 0; --i) mma(i);
    __builtin_amdgcn_sched_barrier(0);
    Bc = Bn;
  };
  // full blocks of P steps: no exit inside, the ring returns to its layout
  const int nfull = L / P;
  int blk0 = 0;
  if (ramp) {
#pragma unroll
    for (int st = 0; st < P; ++st) step_fn(st, st, true);
    blk0 = 1;
  }
#pragma unroll 1
  for (int blk = blk0; blk < nfull; ++blk) {
#pragma unroll
    for (int st = 0; st < P; ++st) step_fn(blk * P + st, st, false);
  }
  // the remaining L mod P steps
  const int rem = L - nfull * P;
  if (rem > 0) {
    // a guarded, fully unrolled block keeps every ring index a constant
#pragma unroll
    for (int st = 0; st < P - 1; ++st)
      if (st < rem) step_fn(nfull * P + st, st, false);
  }
}

// Per strip: turn the 256 coefficients of acc (strip w) into 56 limbs of out
// and the strip carry word; or, for the diagnostic path, store them raw.
__device__ __forceinline__ void strip_out7(v4i acc, int w, const Lds& s, const Geo& g,
                                           uint32_t* out, int32_t* coef) {
  constexpr int kStripLimbs = strip_limbs<7>();
  const int lane = lane_id();
  int32_t* sc = s.wscr;
  // lane l holds column p = l & 15, rows 4(l>>4)+v: coefficient 16 row + p
#pragma unroll
  for (int v = 0; v < 4; ++v) sc[16 * (4 * (lane >> 4) + v) + (lane & 15)] = acc[v];
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  if (coef) {
    const int K = g.Na + g.Nb - 1;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int kk = 64 * v + lane;
      const int k = kStrip * w + kk;
      if (k < K) coef[k] = sc[kk];
    }
    __builtin_amdgcn_wave_barrier();
    return;
  }
  // column sums: lane j in [0, 57) gathers the coefficients of limb j (at
  // most 5 whose low bits start in limb j, at most 5 spilling from limb j-1);
  // fixed trip counts with masks keep the LDS reads unconditional
  uint64_t X = 0;
  {
    const int j = min(lane, kStripLimbs);
    const int klo = (32 * j + 6) / 7;          // first kappa with floor(7 kappa/32) == j
    const int khi = (32 * (j + 1) + 6) / 7;    // one past the last
    const int plo = (32 * (j - 1) + 6) / 7;    // first kappa of limb j-1 (j > 0)
#pragma unroll
    for (int e = 0; e < 5; ++e) {
      const int kk = klo + e;
      const uint64_t v = (uint64_t)(uint32_t)sc[min(kk, kStrip - 1)] << ((7 * kk - 32 * j) & 63);
      X += (kk < khi && kk < kStrip) ? (v & 0xffffffffull) : 0ull;
      const int pk = plo + e;
      const uint64_t u = (uint64_t)(uint32_t)sc[max(min(pk, kStrip - 1), 0)]
                         << ((7 * pk - 32 * (j - 1)) & 63);
      X += (j > 0 && pk < klo) ? (u >> 32) : 0ull;
    }
    if (lane > kStripLimbs) X = 0;
  }
  __builtin_amdgcn_wave_barrier();
  const uint32_t L = (uint32_t)X;
  const uint32_t H = (uint32_t)(X >> 32);
  // H of the lane below, 0 into lane 0 (DPP wave_shr:1)
  const uint32_t Hprev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)H, 0x138, 0xf, 0xf, false);
  const uint64_t sum = (uint64_t)L + Hprev;
  const uint32_t res = (uint32_t)sum;
  const bool gb = (sum >> 32) != 0;
  const bool pb = (lane <= kStripLimbs) && res == 0xffffffffu;
  const WaveCarry wc = wave_carry_masks(gb, pb);
  const uint32_t cin = wave_carry_in(wc, 0);
  const uint32_t limb = res + cin;
  const int jg = kStripLimbs * w + lane;
  // limbs 2..55 all ones (limbs past the product count as ones): a carry
  // entering limb 2 then runs through the whole strip
  const uint64_t tail = ((1ull << kStripLimbs) - 1) & ~3ull;
  const uint64_t ones = __ballot(jg >= g.nout || limb == 0xffffffffu);
  if (lane < kStripLimbs) {
    if (jg < g.nout) out[jg] = limb;
  } else if (lane == kStripLimbs) {
    const uint32_t cout = (uint32_t)gb | ((uint32_t)pb & cin);
    s.carry[w] = (uint64_t)limb | ((uint64_t)(H + cout) << 32) |
                 ((uint64_t)((ones & tail) == tail) << 63);
  }
}

// ---- signed digits ----------------------------------------------------------------
// The matrix instructions take signed bytes.  Bytes less 128 would do, but bring
// a sum of digits into every coefficient, half of the vector instructions of
// a short product.  Recoding the operand instead brings none: with C = sum_i 128 256^i, the bytes of a + C less 128 each are signed
// digits whose sum is a itself (the carry out of the top limb is one more
// digit, 0 or 1).  The addition's carries are ballots of the waves that stage
// the operand; a wave finds the carry into its part by looking at the limbs
// below, of which nearly always the first decides.  The coefficients are then
// signed, and so are the carries between limbs and strips.  (Carry words kept
// positive by a bias that the next strip takes off again made strips of zero
// limbs borrow and carry through all their limbs: 43 divisions of all-ones
// operands took 340 us, of random ones 222.)

constexpr int kEqual = 32, kGreater = 34, kLess = 36;   // predicates of the unsigned comparison builtin

// limb l of a + C less C digit by digit, for l = 64 r + lane (l >= n: the
// last carry at l = n, then 0); c: the carry into the round, updated
__device__ __forceinline__ uint32_t signed_digits(uint32_t x, uint32_t& c) {
  const uint32_t t = x + 0x80808080u;
  const uint64_t g = __builtin_amdgcn_uicmp(x, 0x7f7f7f7fu, kGreater), p = __builtin_amdgcn_uicmp(x, 0x7f7f7f7fu, kEqual);
  const uint64_t in = carry_bits(g, p, c);
  return (t + (__builtin_amdgcn_inverse_ballot_w64(in) ? 1u : 0u)) ^ 0x80808080u;
}

// the carry into limb 64 r of a + C
__device__ __forceinline__ uint32_t signed_carry_into(const Limbs& a, int r) {
  while (r > 0) {
    const uint32_t x = a(64 * --r + lane_id()), t = x + 0x80808080u;
    const uint64_t g = __ballot(t < x), p = __ballot(t == ~0u);
    if (p != ~0ull) return (uint32_t)(g >> (63 - __clzll(~p))) & 1u;
  }
  return 0u;
}

// Stage the signed digits of both operands (layout as stage7) on waves
// wv = 0 .. nw - 1; with one wave the operands' last carries are returned.
struct LastDigits { int a, b; };
__device__ __forceinline__ LastDigits stage_signed(const Lds& s, const Geo& g, const uint32_t* a, const uint32_t* b,
                                                   int wv, int nw) {
  constexpr int U = 4;
  const int lane = lane_id();
  LastDigits last{0, 0};
  uint32_t* A32 = reinterpret_cast<uint32_t*>(s.A);
  uint32_t* B32 = reinterpret_cast<uint32_t*>(s.B);
  const Limbs a_(a, g.na), b_(b, g.nb);
  {
    // dword QA/4 - 1 - l holds digits 4 l + 4 .. 4 l + 1; limb l - 1 is written
    // with limb l at hand, so limb 0's low digit goes with "limb -1"
    const int top = g.QA / 4, rounds = g.na / 64 + 1;   // (the round of limb na included)
    const int tid = 64 * wv + lane, T = 64 * nw;
    for (int d = tid; d < top - g.na; d += T) A32[d] = 0u;   // (digits 4 na + 1 and up)
    for (int d = top + 1 + tid; d < g.SA / 4; d += T) A32[d] = 0u;
    const int per = (rounds + nw - 1) / nw, first = per * wv, end = min(rounds, first + per);
    uint32_t c = 0u, below = 0u;   // below: limb 64 r - 1
    if (first > 0 && first < end) {
      c = signed_carry_into(a_, first - 1);
      below = (uint32_t)__builtin_amdgcn_readlane((int)signed_digits(a_(64 * (first - 1) + lane), c), 63);
    }
    for (int r0 = first; r0 < end; r0 += U) {
      uint32_t x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = a_(64 * (r0 + u) + lane);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r0 + u < end) {
          const int l = 64 * (r0 + u) + lane;
          const uint32_t v = signed_digits(x[u], c);
          // limb l - 1: the lane below (DPP wave_shr:1), below into lane 0
          const uint32_t w = (uint32_t)__builtin_amdgcn_update_dpp((int)below, (int)v, 0x138, 0xf, 0xf, false);
          below = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
          if (l <= g.na) A32[top - l] = __builtin_bswap32(__builtin_amdgcn_alignbyte(v, w, 1));
          if (nw == 1 && r0 + u == rounds - 1) last.a = __builtin_amdgcn_readlane((int)v, g.na & 63);
        }
    }
  }
  {
    const int base = kPadB / 4, n = g.SB / 4 - base, rounds = (n + 63) / 64;
    if (wv == 0 && lane < base) B32[lane] = 0u;
    const int per = (rounds + nw - 1) / nw, first = per * wv, end = min(rounds, first + per);
    uint32_t c = first < end ? signed_carry_into(b_, first) : 0u;
    for (int r0 = first; r0 < end; r0 += U) {
      uint32_t x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = b_(64 * (r0 + u) + lane);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r0 + u < end) {
          const int l = 64 * (r0 + u) + lane;
          const uint32_t v = signed_digits(x[u], c);
          if (l < n) B32[base + l] = v;
          if (nw == 1 && r0 + u == g.nb / 64) last.b = __builtin_amdgcn_readlane((int)v, g.nb & 63);
        }
    }
  }
  return last;
}

// the largest |X_j|: four coefficients of at most kMaxDigits products each
constexpr int64_t kMaxDigits = 4 * BIGINT_MFMA_MAX_LIMBS + 1;
static_assert(kMaxDigits << 14 < (int64_t)1 << 31, "int32 coefficients");
static_assert((kMaxDigits << 14) * 0x01010101 < (int64_t)1 << 55, "X_j, and with it signed 32-bit carry words");

// Strip w from signed digits: its 64 limbs and signed carry word (32 bits, and
// the tail flag in bit 63).  With X_j the sum of limb j's four
// coefficients (|X_j| < 2^55), limb j takes L_j + H_(j-1) - 1 + B, whose carry
// is 0, 1 or 2; after that carry has moved up, what is left is a sum of
// 32-bit words with carries 0 or 1.  One unit is added
// at limb bump.
// TS = 32: acc is a quarter of a 32x32 result tile (registers 4q..4q+3:
// column lane & 31, rows 4 (lane >> 5) + v of the quarter's eight).
template <int TS = 16>
__device__ __forceinline__ void strip_out_signed(v4i acc, int w, const Lds& s, const Geo& g, uint32_t* out,
                                                 int bump) {
  const int lane = lane_id();
  int32_t* sc = s.wscr;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if constexpr (TS == 32) sc[32 * (4 * (lane >> 5) + v) + (lane & 31)] = acc[v];
    else sc[16 * (4 * (lane >> 4) + v) + (lane & 15)] = acc[v];
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const v4i cp = *reinterpret_cast<const v4i*>(sc + 4 * lane);
  __builtin_amdgcn_wave_barrier();
  int k8 = 1 << 8, k16 = 1 << 16, k24 = 1 << 24;   // (opaque: multiply-adds, not 64-bit shifts)
  asm("" : "+s"(k8), "+s"(k16), "+s"(k24));
  int64_t X = cp[0];
  X += (int64_t)cp[1] * k8;
  X += (int64_t)cp[2] * k16;
  X += (int64_t)cp[3] * k24;
  if (64 * w + lane == bump) X += 1;
  const uint32_t L = (uint32_t)X;
  const int H = (int)(X >> 32);
  const int h = __builtin_amdgcn_update_dpp(1, H, 0x138, 0xf, 0xf, false) - 1;
  const uint32_t t = L + (uint32_t)h;
  const int up = (t < L ? 1 : 0) + (h >> 31) + 1;
  const uint32_t from = (uint32_t)__builtin_amdgcn_update_dpp(0, up, 0x138, 0xf, 0xf, false);
  const uint32_t y = t + from;
  const uint64_t gm = __builtin_amdgcn_uicmp(y, t, kLess), pm = __builtin_amdgcn_uicmp(y, ~0u, kEqual);
  uint32_t cout = 0u;
  const uint64_t in = carry_bits(gm, pm, cout);
  const uint32_t limb = y + (__builtin_amdgcn_inverse_ballot_w64(in) ? 1u : 0u);
  const int jg = 64 * w + lane;
  const uint64_t tail = ~3ull;   // limbs 2..63
  const uint64_t ones = __builtin_amdgcn_uicmp(limb, ~0u, kEqual) |
                        ~__builtin_amdgcn_uicmp((uint32_t)jg, (uint32_t)g.nout, kLess);
  Limbs(out, g.nout).put(jg, limb);
  if (s.lead && lane < 2) reinterpret_cast<uint32_t*>(s.lead)[2 * w + lane] = jg < g.nout ? limb : 0u;
  if (lane == 63)
    s.carry[w] = (uint64_t)(uint32_t)(H - 1 + up + (int)cout) |
                 ((uint64_t)((ones & tail) == tail) << 63);
}

// ---- 32x32x32 tiles (v_mfma_i32_32x32x32_i8) ----------------------------------------
// D[32x32] += A[32x32] B[32x32] with A_Z[r][s] = alpha[Z + 32r - s] and
// B_Y[s][p] = beta[Y + s + p]: the 1024 outputs are c[Z+Y .. Z+Y+1024),
// tile T = four consecutive strips.  With Y = 1024y + 32rho (32 phases) and
// Z = 1024x - 32rho the tile is T = x + y, and a band of P/4 tiles walks y
// with a ring of A tiles exactly as the 16x16 bands do.  Each instruction
// does twice the 16x16x64 tile's multiply-accumulates for the same operand
// bytes per lane.  Register layout (lane l, row r = l & 31, k-group
// g = l >> 5, byte t: contraction index 16g + t): A lane holds
// alpha[Z + 32r - 16g - t], one aligned ds_read_b128 of the reversed
// digits; B lane holds beta[Y + p + 16g + t] with p = l & 31, five dwords
// aligned with v_alignbyte.  Result register v holds column l & 31, row
// (v & 3) + 8 (v >> 2) + 4 (l >> 5): registers 4q..4q+3 are strip 4T + q.
typedef int v16i __attribute__((ext_vector_type(16)));

__device__ __forceinline__ Range band_range32(const Geo& g, int T0, int P32, int rho) {
  Range r;
  // B tile covers beta[Y .. Y+62]; A tile covers alpha[Z-31 .. Z+992]
  const int yb_lo = (961 - 32 * rho) >> 10;
  const int yb_hi = (g.Nb - 1 - 32 * rho) >> 10;
  r.xlo = (32 * rho + 31) >> 10;
  r.xhi = (g.Na + 30 + 32 * rho) >> 10;
  r.lo = max(yb_lo, T0 - r.xhi);
  r.hi = min(yb_hi, T0 + P32 - 1 - r.xlo);
  return r;
}

__device__ __forceinline__ int band_cost32(const Geo& g, int band, int P) {
  int c = 0;
  for (int rho = 0; rho < 32; ++rho) {
    const Range r = band_range32(g, band * (P / 4), P / 4, rho);
    c += max(0, r.hi - r.lo + 1);
  }
  return c;
}

__device__ __forceinline__ v4i load_A32(const uint8_t* Abuf, const Geo& g, int x, int rho,
                                        const Range& r) {
  const int lane = lane_id();
  const int Z = 1024 * x - 32 * rho;
  const bool ok = x >= r.xlo && x <= r.xhi;  // wave-uniform
  const int addr = ok ? g.QA - Z - 32 * (lane & 31) + 16 * (lane >> 5) : 0;
  return *reinterpret_cast<const v4i*>(Abuf + addr);
}

__device__ __forceinline__ BRaw load_B_raw32(const uint8_t* Bbuf, int y, int rho) {
  const int lane = lane_id();
  const int p = lane & 31;
  const int Y = 1024 * y + 32 * rho;
  const uint32_t* src =
      reinterpret_cast<const uint32_t*>(Bbuf + kPadB + Y + 16 * (lane >> 5) + 4 * (p >> 2));
  BRaw b;
#pragma unroll
  for (int i = 0; i < 5; ++i) b.d[i] = src[i];
  return b;
}

// One phase of one band of P32 tiles: acc[i] += sum over the y range of
// A(T0+i-y) B(y); the software pipeline and the ramp block of band_phase.
template <int P32>
__device__ __forceinline__ void band_phase32(v16i (&acc)[P32], const Lds& s, const Geo& g, int T0,
                                             int rho) {
  const Range r = band_range32(g, T0, P32, rho);
  const int L = r.hi - r.lo + 1;
  if (L <= 0) return;
  const int xb = T0 - r.lo;
  const bool ramp = L >= 2 * P32 && r.lo == T0 - r.xhi;
  v4i ring[P32];
#pragma unroll
  for (int i = 0; i < P32; ++i) ring[i] = load_A32(s.A, g, xb + i, rho, r);
  v4i Bc = align_B(load_B_raw32(s.B, r.lo, rho));
  BRaw raw = load_B_raw32(s.B, min(r.lo + 1, r.hi), rho);
  auto step_fn = [&](const int step, const int st, const bool rmp) __attribute__((always_inline)) {
    auto mma = [&](int i) __attribute__((always_inline)) {
      if (!rmp || i <= st)
        acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ring[(P32 + i - st) % P32], Bc, acc[i], 0, 0, 0);
    };
    mma(P32 - 1);
    ring[(2 * P32 - 1 - st) % P32] = load_A32(s.A, g, xb - step - 1, rho, r);
#pragma unroll
    for (int i = P32 - 2; i >= P32 / 2; --i) mma(i);
    __builtin_amdgcn_sched_barrier(0);
    const v4i Bn = align_B(raw);
    raw = load_B_raw32(s.B, min(r.lo + step + 2, r.hi), rho);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = P32 / 2 - 1; i >= 0; --i) mma(i);
    __builtin_amdgcn_sched_barrier(0);
    Bc = Bn;
  };
  const int nfull = L / P32;
  int blk0 = 0;
  if (ramp) {
#pragma unroll
    for (int st = 0; st < P32; ++st) step_fn(st, st, true);
    blk0 = 1;
  }
#pragma unroll 1
  for (int blk = blk0; blk < nfull; ++blk) {
#pragma unroll
    for (int st = 0; st < P32; ++st) step_fn(blk * P32 + st, st, false);
  }
  const int rem = L - nfull * P32;
  if (rem > 0) {
#pragma unroll
    for (int st = 0; st < P32 - 1; ++st)
      if (st < rem) step_fn(nfull * P32 + st, st, false);
  }
}

// A band of P strips (P / 4 tiles of 32x32) with signed 8-bit digits.
template <int P>
__device__ __forceinline__ void run_band32(int band, const Lds& s, const Geo& g, uint32_t* out) {
  constexpr int P32 = P / 4;
  const int T0 = band * P32;
  v16i acc[P32];
#pragma unroll
  for (int i = 0; i < P32; ++i) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0;
  }
#pragma unroll 1
  for (int rho = 0; rho < 32; ++rho) band_phase32<P32>(acc, s, g, T0, rho);
#pragma unroll
  for (int i = 0; i < P32; ++i) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int w = 4 * (T0 + i) + q;
      if (w < g.W) {
        const v4i part = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
        strip_out_signed<32>(part, w, s, g, out, -1);
      }
    }
  }
}

template <int DW, int P>
__device__ __forceinline__ void run_band(int band, const Lds& s, const Geo& g, uint32_t* out, int32_t* coef,
                                         int bump = -1) {
  const int w0 = band * P;
  v4i acc[P];
#pragma unroll
  for (int i = 0; i < P; ++i) acc[i] = v4i{0, 0, 0, 0};
#pragma unroll 1
  for (int rho = 0; rho < 4; ++rho) band_phase<P>(acc, s, g, w0, rho);
#pragma unroll
  for (int i = 0; i < P; ++i)
    if (w0 + i < g.W) {
      if constexpr (DW == 8) {
        strip_out_signed(acc[i], w0 + i, s, g, out, bump);
      } else {
        strip_out7(acc[i], w0 + i, s, g, out, coef);
      }
    }
}

// One unit off out at limb j, by one wave (modulo B^nout): the borrow runs up
// through zero limbs, 64 a step.
__device__ __forceinline__ void wave_borrow(uint32_t* out, int j, int nout) {
  for (; j < nout; j += 64) {
    const int k = j + lane_id();
    const uint32_t v = k < nout ? out[k] : 1u;
    const uint64_t stop = __ballot(v != 0u);
    const int last = stop ? __ffsll((long long)stop) - 1 : 63;
    if (lane_id() <= last && k < nout) out[k] = v - 1u;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    if (stop) break;
  }
}

// The signed carry word of a strip (8-bit digits) onto limbs 0-1 of the next:
// whether they overflow, or go below zero (x is then modulo 2^64, and the
// borrow is taken from the limbs above once all strips are closed)
struct StripSum { uint64_t x; bool over, under; };
__device__ __forceinline__ StripSum strip_sum(uint64_t x0, int32_t d) {
  const uint64_t x = x0 + (uint64_t)(int64_t)d;
  return {x, d >= 0 && x < x0, d < 0 && x > x0};
}

// The closing strip carry scan of an instance (whole work-group): carry[w]
// holds strip w's carry word (bits 0-62; with 8-bit digits signed, bits 0-31)
// and tail flag (bit 63), out its limbs, strips from w_first up; scratch: >= 16 words of LDS.  lead
// (nullable, LDS): lead[w] = strip w's limbs 0-1 as written to out, read
// there instead of from out.
template <int DW>
__device__ __forceinline__ void close_strips(uint32_t* out, const Geo& g, uint64_t* carry, int w_first,
                                             uint32_t* scratch, const uint64_t* lead = nullptr) {
  constexpr int kStripLimbs = strip_limbs<DW>();
  // out += sum_w C_w B^(L(w+1)), L limbs per strip.  Strip w' receives C_{w'-1} (< 2^35) on its
  // limbs 0 and 1; a carry out of limb 1 runs on only through a tail of
  // all-ones limbs.  So an exclusive carry scan over strips, one strip per
  // thread, resolves everything: strip w' generates when limbs 0..1 plus
  // C_{w'-1} overflow and its tail is all ones, and propagates when limbs
  // 0..1 plus C_{w'-1} are all ones and so is its tail.
  const uint64_t kC = (1ull << 63) - 1;
  uint32_t cy = 0u;
  int under = 0;
  for (int base = w_first; base < g.W; base += blockDim.x) {
    const int w = base + threadIdx.x;
    const bool valid = w < g.W;
    const int j0 = kStripLimbs * (valid ? w : 0);
    uint64_t x0;
    if (lead) {
      x0 = valid ? lead[w] : 0ull;
    } else {
      const uint32_t l0 = (valid && j0 < g.nout) ? out[j0] : 0u;
      const uint32_t l1 = (valid && j0 + 1 < g.nout) ? out[j0 + 1] : 0u;
      x0 = ((uint64_t)l1 << 32) | l0;
    }
    const uint64_t d = (valid && w > w_first) ? (carry[w - 1] & kC) : 0ull;
    const bool ones = valid && (carry[w] >> 63);
    uint64_t x = x0 + d;
    bool xh = x < x0;  // carry out of limb 1
    if constexpr (DW == 8) {
      const StripSum sum = strip_sum(x0, (int32_t)(uint32_t)d);
      x = sum.x;
      xh = sum.over;
      if (sum.under) {   // (the strip above reads only the low half of this word)
        reinterpret_cast<uint32_t*>(carry + w)[1] |= 1u << 30;
        under = 1;
      }
    }
    const bool gen = valid && xh && ones;
    const bool prop = valid && !xh && x == ~0ull && ones;
    uint32_t cout;
    const uint32_t c = wg_carry_scan(gen, prop, cy, scratch, &cout);
    cy = cout;
    if (valid) {
      const uint64_t y = x + c;
      const bool yh = xh || (y < x);
      if (y != x0) {
        if (j0 < g.nout) out[j0] = (uint32_t)y;
        if (j0 + 1 < g.nout) out[j0 + 1] = (uint32_t)(y >> 32);
      }
      if (yh) {  // ripple into the tail (stops at its first limb that is not all ones)
        for (int j = j0 + 2; j < min(j0 + kStripLimbs, g.nout); ++j) {
          const uint32_t v = out[j];
          out[j] = v + 1u;
          if (v != 0xffffffffu) break;
        }
      }
    }
  }
  if constexpr (DW == 8) {
    if (__syncthreads_or(under) && wave_id() == 0)
      for (int base = w_first; base < g.W; base += 64) {
        const int w = base + lane_id();
        uint64_t mask = __ballot(w < g.W && ((carry[min(w, g.W - 1)] >> 62) & 1ull));
        for (; mask; mask &= mask - 1ull)
          wave_borrow(out, kStripLimbs * (base + __ffsll((long long)mask) - 1) + 2, g.nout);
      }
  }
}

// First band of a product whose limbs below nlo are not needed: the strips
// of the bands before it lie entirely below limb nlo - 2, and the part of the
// product that they hold is below 2^31 B^(the first strip's limb) < B^(nlo-1).
template <int DW>
__host__ __device__ inline int high_band(int nlo, int P) {
  return nlo > 2 ? ((nlo - 2) / strip_limbs<DW>()) / P : 0;
}

// out[0 .. nout) = a * b mod B^nout for one instance (whole work-group),
// digits of DW bits; nout < 0 means the whole na+nb limbs.  nlo > 0 asks
// only for the limbs from nlo up: the bands below high_band(nlo) are not
// computed, out[nlo ..) then holds floor(a b / B^nlo) mod B^(nout-nlo) or
// one more (the part left out can have either sign and is below B^(nlo-1),
// which is added), and the limbs below nlo are left as they were or wrong.  With
// coef != nullptr (7-bit digits only, whole product) the raw coefficients
// c_k (k < Na+Nb-1) are written instead.
// nparts > 1 (full products, coef == nullptr, nlo == 0): this work-group is
// part `part` of nparts sharing the instance.  The bands are cut into nparts
// contiguous runs of about equal cost (band t goes to the part its cost
// midpoint falls in); this part computes only its run, writes its strips'
// carry words to carry_ext[w] (global memory, one word per strip) instead of
// LDS and leaves the closing strip carry scan to close_strips once every
// part has finished (a later launch).
// lead (8-bit digits, whole instance; smem sized by lds_bytes with lead):
// every strip's limbs 0-1 are also kept in LDS, where the closing scan reads
// them instead of reading them back from out.
template <int DW, int P, int TS = 16>
__device__ __forceinline__ void wg_mul_mfma(uint32_t* out, int32_t* coef, const uint32_t* __restrict__ a, int na,
                            const uint32_t* __restrict__ b, int nb, char* smem, int nout = -1,
                            int nlo = 0, int part = 0, int nparts = 1, uint64_t* carry_ext = nullptr,
                            bool lead = false) {
  static_assert(DW == 7 || DW == 8, "digit width");
  static_assert(TS == 16 || (TS == 32 && DW == 8 && P % 4 == 0), "32x32 tiles: 8-bit digits, whole tiles per band");
  out = uniform_ptr(out);
  a = uniform_ptr(a);
  b = uniform_ptr(b);
  Geo g = make_geo<DW, TS>(na, nb, coef ? -1 : nout);
  Lds s = carve<DW>(smem, g, P, lead && coef == nullptr && nparts == 1);
  if (nparts > 1) s.carry = carry_ext;
  const int NBall = (g.W + P - 1) / P;
  // bands [band_lo, NBall) are computed; strips from w_first up
  const int band_lo = coef ? 0 : min(high_band<DW>(nlo, P), NBall);
  const int w_first = band_lo * P;
  const int NB = NBall - band_lo;

  if constexpr (DW == 8) {
    (void)stage_signed(s, g, a, b, __builtin_amdgcn_readfirstlane(wave_id()),
                       __builtin_amdgcn_readfirstlane(num_waves()));
    g.Na += 1;   // (the operands' last carries)
    g.Nb += 1;
  } else {
    stage7(s, g, a, b);
  }
  // band order: most expensive first (rank sort by cost; the costs sit in
  // the wave scratch area, which holds 256 ints per wave >= NB)
  for (int t = threadIdx.x; t < NB; t += blockDim.x)
    s.scr[t] = TS == 32 ? band_cost32(g, band_lo + t, P) : band_cost(g, band_lo + t, P);
  if (threadIdx.x == 0) s.misc[0] = 0;
  __syncthreads();
  // this part's bands [pb0, pb1) (all of them for a whole instance)
  int pb0 = 0, pb1 = NB;
  if (nparts > 1) {
    if (threadIdx.x == 0) {
      int64_t tot = 0;
      for (int t = 0; t < NB; ++t) tot += s.scr[t];
      int64_t acc = 0;
      int b0 = NB, b1 = NB;
      for (int t = 0; t < NB; ++t) {
        const int64_t c2 = 2 * acc + s.scr[t];   // twice the cost midpoint
        const int pt = tot > 0 ? (int)min<int64_t>(nparts - 1, c2 * nparts / (2 * tot)) : 0;
        if (pt >= part && b0 == NB) b0 = t;
        if (pt > part && b1 == NB) b1 = t;
        acc += s.scr[t];
      }
      s.misc[1] = (uint32_t)b0;
      s.misc[2] = (uint32_t)max(b0, b1);
    }
    __syncthreads();
    pb0 = (int)s.misc[1];
    pb1 = (int)s.misc[2];
  }
  const int PN = pb1 - pb0;
  for (int t = threadIdx.x; t < PN; t += blockDim.x) {
    const int c = s.scr[pb0 + t];
    int rank = 0;
    for (int u2 = 0; u2 < PN; ++u2) {
      const int cu = s.scr[pb0 + u2];
      rank += (cu > c) || (cu == c && u2 < t);
    }
    s.order[rank] = (uint16_t)(pb0 + t);
  }
  __syncthreads();

  for (;;) {
    uint32_t t = 0;
    if (lane_id() == 0) t = atomicAdd(&s.misc[0], 1u);
    t = __builtin_amdgcn_readfirstlane(t);
    if ((int)t >= PN) break;
    const int band = band_lo + __builtin_amdgcn_readfirstlane((int)s.order[t]);
    if constexpr (TS == 32) run_band32<P>(band, s, g, out);
    else run_band<DW, P>(band, s, g, out, coef, band_lo > 0 ? nlo - 1 : -1);
  }
  __syncthreads();
  if (coef == nullptr && nparts == 1) close_strips<DW>(out, g, s.carry, w_first, s.misc + 1, s.lead);
  __syncthreads();
}

// ---- one wave per instance (small operands) ----------------------------------------
// For operands of a few hundred limbs the work-group phases (staging, block
// sums, band scheduling, the strip carry scan) and their barriers cost more
// than the MFMA work, so several instances share a work-group, one wave each
// (the paper's ipb instances per block), and every phase runs inside the
// wave: the staging with its recoding to signed digits, the bands, and the
// strip carry scan on one lane per strip.  Needs W <= 64 strips (na + nb <=
// 4096 limbs).  The vector and the scalar ALU bound it (256 limbs, 16384
// products: with digits offset by 128 and their sums 2457 vector instructions
// a product, 85.7 us; with signed digits 1638 and as many scalar ones, of
// which a CU runs one a cycle, 64.9 us; with ranges by shifts, descriptors in
// scalar registers and multiply-adds for the columns 53.7 us.  128 limbs 43.4,
// 32.7 and 27.9 us; 512 limbs 172, 143 and 118.)

// LDS bytes of one wave's instance (8-bit digits): operands, the wave's
// scratch, strip carries
__host__ __device__ inline size_t wave_lds_bytes(int na, int nb) {
  const Geo g = make_geo<8>(na, nb);
  return (((size_t)g.SA + g.SB + 1024 + (size_t)8 * g.W) + 15) & ~(size_t)15;
}

__device__ __forceinline__ Lds carve_wave(char* smem, const Geo& g) {
  Lds s;
  char* p = smem;
  s.A = reinterpret_cast<uint8_t*>(p); p += g.SA;
  s.B = reinterpret_cast<uint8_t*>(p); p += g.SB;
  s.scr = s.wscr = reinterpret_cast<int32_t*>(p); p += 1024;
  s.carry = reinterpret_cast<uint64_t*>(p);
  s.order = nullptr;
  s.misc = nullptr;
  return s;
}

// LDS writes of this wave visible to its later LDS reads
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// out[0 .. nout) = a * b mod B^nout on the calling wave alone (signed 8-bit
// digits; nout < 0: the whole na+nb limbs); smem: wave_lds_bytes(na, nb)
// bytes of this wave's own LDS.
template <int P>
__device__ __forceinline__ void wave_mul_mfma(uint32_t* out, const uint32_t* __restrict__ a, int na,
                                              const uint32_t* __restrict__ b, int nb, char* smem,
                                              int nout = -1) {
  // (scalar registers: otherwise every access through a descriptor loops over its values)
  out = uniform_ptr(out);
  a = uniform_ptr(a);
  b = uniform_ptr(b);
  Geo g = make_geo<8>(na, nb, nout);
  const Lds s = carve_wave(smem, g);
  const int lane = lane_id();
  const LastDigits last = stage_signed(s, g, a, b, 0, 1);
  g.Na += last.a;
  g.Nb += last.b;
  wave_sync();
  const int NB = (g.W + P - 1) / P;
#pragma unroll 1
  for (int band = 0; band < NB; ++band) run_band<8, P>(band, s, g, out, nullptr);
  wave_sync();
  // strip carries (one lane per strip), as in wg_mul_mfma's closing scan
  constexpr int kStripLimbs = strip_limbs<8>();
  const int w = lane;
  const bool valid = w < g.W;
  const int j0 = kStripLimbs * (valid ? w : 0);
  const uint32_t l0 = (valid && j0 < g.nout) ? out[j0] : 0u;
  const uint32_t l1 = (valid && j0 + 1 < g.nout) ? out[j0 + 1] : 0u;
  const int32_t d = (valid && w > 0) ? (int32_t)(uint32_t)s.carry[w - 1] : 0;
  const bool ones = valid && (s.carry[w] >> 63);
  const uint64_t x0 = ((uint64_t)l1 << 32) | l0;
  const StripSum sum = strip_sum(x0, d);
  const uint64_t x = sum.x;
  const bool xh = sum.over;
  const bool gen = valid && xh && ones;
  const bool prop = valid && !xh && x == ~0ull && ones;
  const WaveCarry wc = wave_carry_masks(gen, prop);
  const uint32_t c = wave_carry_in(wc, 0u);
  if (valid) {
    const uint64_t y = x + c;
    const bool yh = xh || (y < x);
    if (y != x0) {
      if (j0 < g.nout) out[j0] = (uint32_t)y;
      if (j0 + 1 < g.nout) out[j0 + 1] = (uint32_t)(y >> 32);
    }
    if (yh) {
      for (int j = j0 + 2; j < min(j0 + kStripLimbs, g.nout); ++j) {
        const uint32_t v = out[j];
        out[j] = v + 1u;
        if (v != 0xffffffffu) break;
      }
    }
  }
  uint64_t mask = __ballot(valid && sum.under);
  if (mask) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  for (; mask; mask &= mask - 1ull)
    wave_borrow(out, kStripLimbs * (__ffsll((long long)mask) - 1) + 2, g.nout);
}

}  // namespace mfma
}  // namespace bi
