// dev_mul_ntt.hpp -- the transform multiply: the product as a convolution of
// the limbs themselves modulo three 27-bit primes (number-theoretic
// transforms, integers only), recombined by the Chinese remainder theorem and
// resolved by the same carry scan as the other multiplies.
//
// Section 5.2's C_k = sum_{i+j=k} A_i B_j over 32-bit limbs is at most
// min(na, nb) (2^32 - 1)^2 < 2^78 for operands whose smaller one has at most
// 16,384 limbs, and the three primes' product is 1.009 * 2^78: the residues
// of C_k determine it exactly.  No value is ever rounded.
//
// Transform.  With M >= na + nb points, the operands are polynomials modulo
// x^M - 1.  A node of the transform is x^m - r; its level splits it into
// x^(m/2) - s and x^(m/2) + s with s^2 = r: (u, v) -> (u + s v, u - s v) on
// coefficients m/2 apart.  s depends only on the node's index i in its level
// (the root whose exponent is the bit-reversed fraction of i), so one table
// of 2048 roots per prime serves every level of every size, and no twisting,
// reordering or scaling pass is needed.  The splitting stops at leaves
// x^Q - r of Q = 5..8 coefficients (2..4 in the smallest transforms), whose
// products are formed directly (64-bit multiply-adds): that costs less than
// three more levels in three transforms, and it makes M = Q 2^k available in
// steps of 14 to 25% (20 to 50% below 8192 points) without any radix-5 or
// radix-7 pass.
//
// Arithmetic.  Montgomery products of signed 32-bit words, R = 2^32:
// mont(b, wR) = b w mod p in (-3p/4, 3p/4) for any 32-bit b: one 32x32->64
// multiply-add, two 32-bit multiplies and a subtraction.  With p = 2^26 a
// 32-bit word holds 31.8 p, so sums and differences grow lazily: a whole
// forward transform (12 levels, each two adding at most 7p/4) takes no
// reduction.  Inverse sums double per level; which of them need a reduction
// is decided at compile time from their bounds (InvPlan).
//
// Work split.  One work-group per product: T threads, M = 4 Q T points.
// Three passes per transform, with the points in registers inside a pass and
// exchanged through LDS between passes:
//   pass 1  sets {s + S1 c, c < R1}: the first log2 R1 levels (uniform roots)
//   pass 2  sets {b S1 + j + 4Q c, c < R2}: the next log2 R2 (R1 R2 = T)
//   pass 3  thread t holds the 4Q points of block t: two levels, the leaves
// The inverse runs the passes backwards.  LDS holds one word per point, in
// blocks of 4Q words padded to 4Q + 4, which keeps pass 3's 16-byte accesses
// free of bank conflicts.
#pragma once

#include "common.hpp"

namespace bi {
namespace ntt {

// roots are read through the constant address space: uniform ones by scalar
// loads, and never as flat accesses
#ifdef __HIP_DEVICE_COMPILE__
#define BI_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
typedef const __attribute__((address_space(4))) int32_t* Tab;
#else
#define BI_SCHED_FENCE() (void)0
typedef const int32_t* Tab;
#endif

constexpr int kPrimes = 3;
constexpr int kTab = 2048;   // roots per prime and direction: node indices below 2048

// p = 1 mod 8192, just above 2^26 (the product exceeds 2^78)
constexpr int32_t kP[kPrimes] = {67239937, 67280897, 67411969};

constexpr uint64_t mulmod(uint64_t a, uint64_t b, uint64_t p) { return a * b % p; }
constexpr uint64_t powmod(uint64_t a, uint64_t e, uint64_t p) {
  uint64_t r = 1;
  for (; e; e >>= 1, a = mulmod(a, a, p))
    if (e & 1) r = mulmod(r, a, p);
  return r;
}
constexpr uint64_t invmod(uint64_t a, uint64_t p) { return powmod(a, p - 2, p); }
// a 2^32 mod p (Montgomery form), in [0, p)
constexpr int32_t to_mont(uint64_t a, uint64_t p) {
  return (int32_t)(mulmod(a % p, (1ull << 32) % p, p));
}
// the same, centred: |.| <= p / 2
constexpr int32_t to_mont_c(uint64_t a, uint64_t p) {
  const int32_t m = to_mont(a, p);
  return m > (int32_t)(p / 2) ? m - (int32_t)p : m;
}
// p^-1 mod 2^32
constexpr uint32_t inv32(uint32_t p) {
  uint32_t x = p;
  for (int i = 0; i < 5; ++i) x *= 2u - p * x;
  return x;
}
// an element of order 2 kTab
constexpr uint64_t root4096(uint64_t p) {
  for (uint64_t g = 2;; ++g) {
    const uint64_t w = powmod(g, (p - 1) / (2 * kTab), p);
    if (powmod(w, kTab, p) == p - 1) return w;
  }
}

struct alignas(64) Roots {
  int32_t f[kTab];    // s of node i (any level), Montgomery form, centred
  int32_t fv[kTab];   // s(i / 2) s(i), negated for odd i (see fwd_net)
  int32_t b[kTab];    // inverses of f and fv
  int32_t bv[kTab];
};

constexpr Roots make_roots(int pr) {
  Roots t{};
  uint64_t s[2][kTab] = {};
  const uint64_t p = (uint64_t)kP[pr], w = root4096(p), wi = invmod(w, p);
  uint64_t e = 1, d = 1;
  for (int k = 0; k < kTab; ++k) {
    int rev = 0;
    for (int j = 1, h = kTab / 2; h; j <<= 1, h >>= 1) rev |= (k & j) ? h : 0;
    s[0][rev] = e;
    s[1][rev] = d;
    e = mulmod(e, w, p);
    d = mulmod(d, wi, p);
  }
  for (int k = 0; k < kTab; ++k) {
    const uint64_t v = mulmod(s[0][k / 2], s[0][k], p), u = mulmod(s[1][k / 2], s[1][k], p);
    t.f[k] = to_mont_c(s[0][k], p);
    t.b[k] = to_mont_c(s[1][k], p);
    t.fv[k] = k & 1 ? -to_mont_c(v, p) : to_mont_c(v, p);
    t.bv[k] = k & 1 ? -to_mont_c(u, p) : to_mont_c(u, p);
  }
  return t;
}

// The leaf products come out of one Montgomery reduction (a factor 2^-32) and
// the inverse's levels leave a factor 2^k: operand A's reduction before the
// leaf products multiplies by 2^32 2^-k, so that the residues need no scaling.
constexpr int32_t leaf_scale(int pr, int k) {
  const uint64_t p = (uint64_t)kP[pr];
  return to_mont_c(mulmod((1ull << 32) % p, invmod(1ull << k, p), p), p);
}

// Per-prime constants and tables.  The kernels read them from memory: with
// the values visible, the compiler turns the signed high products by p into
// longer unsigned sequences.
constexpr int kMaxK = 12;
struct Field {
  int32_t p;
  uint32_t pinv;     // p^-1 mod 2^32
  int32_t one;       // mont(x, one) = x reduced
  uint32_t load;     // limb loads: mont_u(x, load) = x (Montgomery form, in [0, p))
  int32_t scale[kMaxK + 1];   // leaf_scale
  Roots roots;
};

constexpr Field make_field(int pr) {
  const uint64_t p = (uint64_t)kP[pr];
  Field f{};
  f.p = kP[pr];
  f.pinv = inv32((uint32_t)p);
  f.one = to_mont_c(1, p);
  f.load = (uint32_t)to_mont(1, p);
  for (int k = 0; k <= kMaxK; ++k) f.scale[k] = leaf_scale(pr, k);
  f.roots = make_roots(pr);
  return f;
}
constexpr Field kF0 = make_field(0), kF1 = make_field(1), kF2 = make_field(2);

struct Fields { Field f[kPrimes]; };
__device__ const Fields d_fields = {{kF0, kF1, kF2}};

// b w for a Montgomery-form w (|w| <= p): in (-3p/4, 3p/4) when |w| <= p / 2
__host__ __device__ __forceinline__ int32_t mulhi32(int32_t a, int32_t b) {
#ifdef __HIP_DEVICE_COMPILE__
  return __mulhi(a, b);
#else
  return (int32_t)(((int64_t)a * b) >> 32);
#endif
}
__host__ __device__ __forceinline__ int32_t redc(int64_t m, int32_t p, uint32_t pinv) {
  const int32_t q = (int32_t)((uint32_t)m * pinv);
  return (int32_t)(m >> 32) - mulhi32(q, p);
}
__host__ __device__ __forceinline__ int32_t mont(int32_t b, int32_t w, int32_t p, uint32_t pinv) {
  return redc((int64_t)b * w, p, pinv);
}
// x w for an unsigned limb x and w in [0, p): in (-p/2, 3p/2)
__host__ __device__ __forceinline__ int32_t mont_u(uint32_t x, uint32_t w, int32_t p, uint32_t pinv) {
  const uint64_t m = (uint64_t)x * w;
  const int32_t q = (int32_t)((uint32_t)m * pinv);
  return (int32_t)(m >> 32) - mulhi32(q, p);
}

// ---- compile-time bounds (units of p / 4) --------------------------------------------
constexpr int kLim = 127;      // 2^31 > 31.8 p for every prime
constexpr int kRed = 3;        // a Montgomery product of a 32-bit word: below 3p/4
constexpr int kRed2 = 4;       // a reduced sum of two: (31.8 p^2) / 2^32 + p / 2 < p
constexpr int kLoad = 6;       // a loaded limb: 3p/2
constexpr int kPassEnd = 6;    // bound of every point between inverse passes

constexpr int log2i(int x) { return x <= 1 ? 0 : 1 + log2i(x / 2); }

// A network of R points runs its levels in pairs (radix 4) from level 0, an
// odd last one alone.  FREE (even): levels below it run their first node,
// whose root is 1, without its products; its outputs' bounds add up instead.
constexpr int kFwdFree = 4;
constexpr int kInvFree = 2;

// largest bound after a forward network of R points that start at `start`
constexpr int fwd_bound(int R, int start, int free_levels) {
  int node0 = start, rest = start;   // points of node 0, of the other nodes
  const int L = log2i(R);
  for (int l = 0; l + 1 < L; l += 2) {
    const int r = (rest > node0 ? rest : node0) + kRed + kRed2;   // a + P + Q
    if (l < free_levels) {
      const int n = 4 * node0;                                    // a + b + c + d
      rest = r > 2 * node0 + kRed ? r : 2 * node0 + kRed;         // a - c + i (b - d)
      node0 = n;
    } else {
      node0 = rest = r;
    }
  }
  const int top = node0 > rest ? node0 : rest;
  return L & 1 ? top + kRed : top;
}

// Which points of an R-point inverse network are reduced, and where: before
// the step at level l (red[l][pos]) when one of its sums could leave 32
// bits, and at the end (end[pos]) when the point leaves above kPassEnd.
template <int R>
struct InvPlan {
  bool red[6][R];
  bool end[R];
  int top;       // largest bound at the end (before the end reductions)
};

template <int R>
constexpr InvPlan<R> inv_plan(int start, int free_levels) {
  InvPlan<R> q{};
  int b[R] = {};
  for (int i = 0; i < R; ++i) b[i] = start;
  int l = log2i(R);
  if (l & 1) {   // the single last level
    l -= 1;
    for (int u = 0; u < R; u += 2) {
      while (b[u] + b[u + 1] > kLim) {
        const int w = b[u] >= b[u + 1] ? u : u + 1;
        q.red[l][w] = true;
        b[w] = kRed;
      }
      b[u] += b[u + 1];
      b[u + 1] = kRed;
    }
  }
  while (l > 0) {
    l -= 2;
    const int h = R >> (l + 2);
    for (int i = 0; i < (1 << l); ++i)
      for (int j = 0; j < h; ++j) {
        const int x = i * 4 * h + j;
        for (;;) {
          int sum = 0, w = x;
          for (int k = 0; k < 4; ++k) {
            sum += b[x + k * h];
            if (b[x + k * h] > b[w]) w = x + k * h;
          }
          if (sum <= kLim) break;
          q.red[l][w] = true;
          b[w] = kRed;
        }
        const int d0 = b[x] + b[x + h], all = d0 + b[x + 2 * h] + b[x + 3 * h];
        const bool fr = l < free_levels && i == 0;
        b[x] = all;
        b[x + 2 * h] = fr ? all : kRed;
        b[x + h] = b[x + 3 * h] = fr ? d0 + kRed : kRed2;
      }
  }
  for (int i = 0; i < R; ++i) {
    q.end[i] = b[i] > kPassEnd;
    if (b[i] > q.top) q.top = b[i];
  }
  return q;
}

// ---- butterfly networks on registers ----------------------------------------------
// Two levels at once on (a, b, c, d), h points apart, of node i with root s1
// and its children's roots s2 and s3 = i s2 (i^2 = -1):
//   X0, X1 = (a + s1 c) +- (s2 b + s1 s2 d)
//   X2, X3 = (a - s1 c) +- (s3 b - s1 s3 d)
// Each bracket of two products takes one reduction: 5 multiply-adds and
// three reductions, 20 instructions for four points where two separate
// levels take 24.  s(l, i) and v(l, i): the root of node i of level l, and
// that root times its parent's (negated for odd i).
// HALF: the points of the upper half are 0 on entry.
template <int R, int FREE, bool HALF = false, class S, class V>
__host__ __device__ __forceinline__ void fwd_net(int32_t (&x)[R], S s, V v, int32_t p, uint32_t pinv) {
  constexpr int L = log2i(R);
#pragma unroll
  for (int l = 0; l + 1 < L; l += 2) {
    const int h = R >> (l + 2);
#pragma unroll
    for (int i = 0; i < (1 << l); ++i) {
#pragma unroll
      for (int j = 0; j < h; ++j) {
        const int k = i * 4 * h + j;
        const int32_t a = x[k], b = x[k + h], c = x[k + 2 * h], d = x[k + 3 * h];
        int32_t t, q0, q1;
        if (HALF && l == 0) {
          t = 0;
          q0 = b;
          q1 = mont(b, s(1, 1), p, pinv);
        } else if (l < FREE && i == 0) {
          t = c;
          q0 = b + d;
          q1 = mont(b - d, s(l + 1, 1), p, pinv);
        } else {
          t = mont(c, s(l, i), p, pinv);
          q0 = redc((int64_t)b * s(l + 1, 2 * i) + (int64_t)d * v(l + 1, 2 * i), p, pinv);
          q1 = redc((int64_t)b * s(l + 1, 2 * i + 1) + (int64_t)d * v(l + 1, 2 * i + 1), p, pinv);
        }
        const int32_t e = a + t, f = a - t;
        x[k] = e + q0;
        x[k + h] = e - q0;
        x[k + 2 * h] = f + q1;
        x[k + 3 * h] = f - q1;
      }
    }
  }
  if (L & 1) {
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      const int32_t t = mont(x[2 * i + 1], s(L - 1, i), p, pinv), a = x[2 * i];
      x[2 * i] = a + t;
      x[2 * i + 1] = a - t;
    }
  }
}

// The inverse (each level times 2): with E0 = X0 + X1, E1 = X2 + X3,
// D0 = X0 - X1, D1 = X2 - X3 and the inverse roots,
//   a = E0 + E1, c = s1 (E0 - E1), b = s2 D0 + s3 D1, d = s1 s2 D0 - s1 s3 D1.
template <int R, int START, int FREE, bool LAST, class S, class V>
__host__ __device__ __forceinline__ void inv_net(int32_t (&x)[R], S s, V v, int32_t p, uint32_t pinv,
                                                 int32_t one) {
  constexpr int L = log2i(R);
  constexpr InvPlan<R> plan = inv_plan<R>(START, FREE);
  if (L & 1) {
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      if (plan.red[L - 1][2 * i]) x[2 * i] = mont(x[2 * i], one, p, pinv);
      if (plan.red[L - 1][2 * i + 1]) x[2 * i + 1] = mont(x[2 * i + 1], one, p, pinv);
      const int32_t a = x[2 * i], b = x[2 * i + 1];
      x[2 * i] = a + b;
      x[2 * i + 1] = mont(a - b, s(L - 1, i), p, pinv);
    }
  }
#pragma unroll
  for (int l = (L & ~1) - 2; l >= 0; l -= 2) {
    const int h = R >> (l + 2);
#pragma unroll
    for (int i = 0; i < (1 << l); ++i) {
#pragma unroll
      for (int j = 0; j < h; ++j) {
        const int k = i * 4 * h + j;
#pragma unroll
        for (int m = 0; m < 4; ++m)
          if (plan.red[l][k + m * h]) x[k + m * h] = mont(x[k + m * h], one, p, pinv);
        const int32_t e0 = x[k] + x[k + h], d0 = x[k] - x[k + h];
        const int32_t e1 = x[k + 2 * h] + x[k + 3 * h], d1 = x[k + 2 * h] - x[k + 3 * h];
        x[k] = e0 + e1;
        if (l < FREE && i == 0) {
          const int32_t q = mont(d1, s(l + 1, 1), p, pinv);
          x[k + 2 * h] = e0 - e1;
          x[k + h] = d0 + q;
          x[k + 3 * h] = d0 - q;
        } else {
          x[k + 2 * h] = mont(e0 - e1, s(l, i), p, pinv);
          x[k + h] = redc((int64_t)d0 * s(l + 1, 2 * i) + (int64_t)d1 * s(l + 1, 2 * i + 1), p, pinv);
          x[k + 3 * h] = redc((int64_t)d0 * v(l + 1, 2 * i) + (int64_t)d1 * v(l + 1, 2 * i + 1), p, pinv);
        }
      }
    }
  }
  if (!LAST) {
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (plan.end[i]) x[i] = mont(x[i], one, p, pinv);
  }
}

// ---- geometry of one size ------------------------------------------------------------
template <int T_, int Q_, int R1_, int R2_>
struct Size {
  static constexpr int T = T_, Q = Q_, R1 = R1_, R2 = R2_;
  static constexpr int S2 = 4 * Q;        // points per thread block
  static constexpr int PS2 = S2 + 4;      // padded
  static constexpr int S1 = R2 * S2;      // pass-1 stride
  static constexpr int M = T * S2;
  static constexpr int L1 = log2i(R1), L2 = log2i(R2), K = L1 + L2 + 2;
  static constexpr int NW = T / 64;
  static constexpr int NC1 = S1 / 64;     // 64-set chunks of pass 1
  static constexpr int G1 = (NC1 + NW - 1) / NW;
  static constexpr int N2 = M / R2;       // sets of pass 2
  static constexpr int G2 = (N2 + T - 1) / T;
  static constexpr int LDS_WORDS = T * PS2;
  static constexpr size_t LDS_BYTES = (size_t)LDS_WORDS * 4 + 256;
  static_assert(R1 * R2 == T && S1 % 64 == 0, "sizes");
  static_assert(2 * T <= kTab, "root table");
  static constexpr int FWD = fwd_bound(4, fwd_bound(R2, fwd_bound(R1, kLoad, kFwdFree), 0), 0);
  static_assert(FWD <= kLim, "forward bound");

  // LDS word of pass-1 point c of set s, and of pass-2 point c of set (b, j)
  __host__ __device__ static __forceinline__ int pos1(int s, int c) { return (c * R2 + s / S2) * PS2 + s % S2; }
  __host__ __device__ static __forceinline__ int pos2(int s, int c) { return ((s / S2) * R2 + c) * PS2 + s % S2; }
};

// ---- passes ---------------------------------------------------------------------------
// Each takes the thread's place in the pass explicitly, so that the same code
// runs on the host for one thread after another.

// root first + i, addressed by a 32-bit offset from the table's uniform base
__host__ __device__ __forceinline__ int32_t at(Tab f, int first, int i) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef const __attribute__((address_space(4))) char* Bytes;
  return *(Tab)((Bytes)f + (uint32_t)(4 * first) + 4 * i);
#else
  return f[first + i];
#endif
}

struct Prime {
  int32_t p;
  uint32_t pinv;
  int32_t one;
  uint32_t load;
  Tab f, fv;   // forward roots
  Tab b, bv;   // inverse roots
};

// P re-read where it is used: the products by p and by roots are 32 x 32-bit
// only while their sign extensions sit in the same basic block, so none may
// be hoisted out of the loops over sets and primes.
__host__ __device__ __forceinline__ Prime local(const Prime& P) {
  Prime L = P;
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(L.p), "+s"(L.pinv), "+s"(L.one), "+s"(L.load), "+s"(L.f), "+s"(L.fv),
               "+s"(L.b), "+s"(L.bv));
#endif
  return L;
}

// pass 1 of set s: limbs src(s + S1 c) (0 past the operand's end) to LDS
// HALF: the operand has at most M / 2 limbs, so the upper half of every set
// is zero: no loads, no reductions and no sums with it.
template <class Z, bool HALF, class Src>
__host__ __device__ __forceinline__ void fwd1(const Src& src, int s, int32_t* lds, const Prime& P_) {
  const Prime P = local(P_);
  constexpr int N = HALF ? Z::R1 / 2 : Z::R1;
  int32_t x[Z::R1];
  uint32_t raw[N];
#pragma unroll
  for (int c = 0; c < N; ++c) raw[c] = src(s + Z::S1 * c);
#pragma unroll
  for (int c = 0; c < Z::R1; ++c) x[c] = c < N ? mont_u(raw[c], P.load, P.p, P.pinv) : 0;
  fwd_net<Z::R1, kFwdFree, HALF>(x, [&](int, int i) { return P.f[i]; }, [&](int, int i) { return P.fv[i]; }, P.p, P.pinv);
#pragma unroll
  for (int c = 0; c < Z::R1; ++c) lds[Z::pos1(s, c)] = x[c];
}

// pass 2 of set s, in place; node: the transform's root is node `node` of its
// level in a larger one (a factor of it), else 0
template <class Z>
__host__ __device__ __forceinline__ void fwd2(int s, int32_t* lds, const Prime& P_, int node = 0) {
  const Prime P = local(P_);
  int32_t x[Z::R2];
  const int b = node * Z::R1 + s / Z::S2;
#pragma unroll
  for (int c = 0; c < Z::R2; ++c) x[c] = lds[Z::pos2(s, c)];
  fwd_net<Z::R2, 0>(
      x, [&](int l, int i) { return at(P.f, b << l, i); }, [&](int l, int i) { return at(P.fv, b << l, i); }, P.p,
      P.pinv);
#pragma unroll
  for (int c = 0; c < Z::R2; ++c) lds[Z::pos2(s, c)] = x[c];
}

// the 4Q points of block t
template <class Z>
__host__ __device__ __forceinline__ void block_get(int t, const int32_t* lds, int32_t (&x)[Z::S2]) {
  const v4i* src = reinterpret_cast<const v4i*>(lds + t * Z::PS2);
#pragma unroll
  for (int e = 0; e < Z::Q; ++e) {
    const v4i v = src[e];
    x[4 * e] = v.x; x[4 * e + 1] = v.y; x[4 * e + 2] = v.z; x[4 * e + 3] = v.w;
  }
}
template <class Z>
__host__ __device__ __forceinline__ void block_put(int t, int32_t* lds, const int32_t (&x)[Z::S2]) {
  v4i* dst = reinterpret_cast<v4i*>(lds + t * Z::PS2);
#pragma unroll
  for (int e = 0; e < Z::Q; ++e) dst[e] = v4i{x[4 * e], x[4 * e + 1], x[4 * e + 2], x[4 * e + 3]};
}

// pass 3 of thread t: the last two levels, leaf k in x[k]
// the roots of thread t's two levels
struct Roots3 {
  int32_t s0, s1, s2, v1, v2;
};
__host__ __device__ __forceinline__ Roots3 load3(int t, Tab f, Tab fv) {
  return Roots3{at(f, t, 0), at(f, 2 * t, 0), at(f, 2 * t, 1), at(fv, 2 * t, 0), at(fv, 2 * t, 1)};
}

template <class Z>
__host__ __device__ __forceinline__ void fwd3(int t, const int32_t* lds, int32_t (&x)[4][Z::Q], const Roots3& w,
                                              const Prime& P_) {
  const Prime P = local(P_);
  int32_t raw[Z::S2];
  block_get<Z>(t, lds, raw);
#pragma unroll
  for (int j = 0; j < Z::Q; ++j) {
    int32_t y[4] = {raw[j], raw[Z::Q + j], raw[2 * Z::Q + j], raw[3 * Z::Q + j]};
    fwd_net<4, 0>(
        y, [&](int l, int i) { return l == 0 ? w.s0 : (i == 0 ? w.s1 : w.s2); },
        [&](int, int i) { return i == 0 ? w.v1 : w.v2; },
        P.p, P.pinv);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k][j] = y[k];
  }
}

// the leaf products of thread t: b[k] = a[k] b[k] mod x^Q - r_k (a reduced)
template <class Z>
__host__ __device__ __forceinline__ void leaves(const int32_t (&a)[4][Z::Q], int32_t (&b)[4][Z::Q], const Roots3& w,
                                                const Prime& P_) {
  const Prime P = local(P_);
  constexpr int Q = Z::Q;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int32_t r = k == 0 ? w.s1 : (k == 1 ? -w.s1 : (k == 2 ? w.s2 : -w.s2));
    int32_t c[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      int64_t lo = 0;
      if (j < Q - 1) {
        int64_t hi = 0;
#pragma unroll
        for (int i = j + 1; i < Q; ++i) hi += (int64_t)a[k][i] * b[k][Q + j - i];
        lo = (int64_t)redc(hi, P.p, P.pinv) * r;
      }
#pragma unroll
      for (int i = 0; i <= j; ++i) lo += (int64_t)a[k][i] * b[k][j - i];
      c[j] = redc(lo, P.p, P.pinv);
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) b[k][j] = c[j];
    BI_SCHED_FENCE();
  }
}

// bound of a leaf product's coefficient (units of p/4): redc of a sum of at
// most Q products 3p/4 * B p/4 and h r with |h| < 2^28, |r| <= p/2
constexpr int leaf_bound(int q, int bound) {
  // |lo| / 2^32 + p / 2 with p < 1.005 * 2^26: (q 3 bound / 16 p^2 + 2^28 p / 2) / 2^32
  //   = p ((3 q bound / 16) p / 2^32 + 1/32) ; p / 2^32 < 1/63
  return 4 * ((3 * q * bound / 16 + 1) / 63 + 1) + 3;
}

// inverse pass 3 of thread t: two levels, points to LDS
template <class Z>
__host__ __device__ __forceinline__ void inv3(int t, const int32_t (&x)[4][Z::Q], int32_t* lds, const Roots3& w,
                                              const Prime& P_) {
  const Prime P = local(P_);
  int32_t raw[Z::S2];
  constexpr int start = leaf_bound(Z::Q, Z::FWD);
#pragma unroll
  for (int j = 0; j < Z::Q; ++j) {
    int32_t y[4] = {x[0][j], x[1][j], x[2][j], x[3][j]};
    inv_net<4, start, 0, false>(
        y, [&](int l, int i) { return l == 0 ? w.s0 : (i == 0 ? w.s1 : w.s2); },
        [&](int, int i) { return i == 0 ? w.v1 : w.v2; },
        P.p, P.pinv, P.one);
#pragma unroll
    for (int k = 0; k < 4; ++k) raw[k * Z::Q + j] = y[k];
  }
  block_put<Z>(t, lds, raw);
}

template <class Z>
__host__ __device__ __forceinline__ void inv2(int s, int32_t* lds, const Prime& P_, int node = 0) {
  const Prime P = local(P_);
  int32_t x[Z::R2];
  const int b = node * Z::R1 + s / Z::S2;
#pragma unroll
  for (int c = 0; c < Z::R2; ++c) x[c] = lds[Z::pos2(s, c)];
  inv_net<Z::R2, kPassEnd, 0, false>(
      x, [&](int l, int i) { return at(P.b, b << l, i); }, [&](int l, int i) { return at(P.bv, b << l, i); }, P.p,
      P.pinv, P.one);
#pragma unroll
  for (int c = 0; c < Z::R2; ++c) lds[Z::pos2(s, c)] = x[c];
}

// inverse pass 1 of set s: x[c] = the residue of coefficient s + S1 c, |x| < 32p
template <class Z>
__host__ __device__ __forceinline__ void inv1(int s, const int32_t* lds, int32_t (&x)[Z::R1], const Prime& P_) {
  const Prime P = local(P_);
  static_assert(inv_plan<Z::R1>(kPassEnd, kInvFree).top <= kLim - 4, "garner subtracts a residue");
#pragma unroll
  for (int c = 0; c < Z::R1; ++c) x[c] = lds[Z::pos1(s, c)];
  inv_net<Z::R1, kPassEnd, kInvFree, true>(
      x, [&](int, int i) { return P.b[i]; }, [&](int, int i) { return P.bv[i]; }, P.p, P.pinv, P.one);
}

// ---- a factor of a larger transform ---------------------------------------------------
// A product of 4 M points splits by its first two levels into the factors
// x^M - r with r = 1, -1, i, -i (nodes 0..3 of level 2).  Operand x is
// x_0 + x_1 r + x_2 r^2 + x_3 r^3 there, x_k its k-th run of M limbs.

// c[node][k] = r^k, Montgomery form in [0, p)
struct Quarters { uint32_t c[kPrimes][4][4]; };
constexpr Quarters make_quarters() {
  Quarters q{};
  for (int pr = 0; pr < kPrimes; ++pr) {
    const uint64_t p = (uint64_t)kP[pr], w = root4096(p), i = powmod(w, kTab / 2, p);
    const uint64_t r[4] = {1, p - 1, i, p - i};
    for (int f = 0; f < 4; ++f)
      for (int k = 0; k < 4; ++k) q.c[pr][f][k] = (uint32_t)to_mont(powmod(r[f], (uint64_t)k, p), p);
  }
  return q;
}
constexpr Quarters kQuarters = make_quarters();
__device__ const Quarters d_quarters = kQuarters;
constexpr int kLoad4 = 18;   // a loaded point: a sum of four limbs times roots, redc in (-p/2, 9p/2)

// pass 1 of set s of factor `node`: runs > 2: all four runs of the operand
// (else its first two; the others are 0)
template <class Z, bool HALF, class Src>
__host__ __device__ __forceinline__ void fwd1_quarter(const Src& src, int s, int node, const uint32_t (&c)[4],
                                                      int32_t* lds, const Prime& P_) {
  const Prime P = local(P_);
  constexpr int N = HALF ? 2 : 4;
  static_assert(fwd_bound(4, fwd_bound(Z::R2, fwd_bound(Z::R1, kLoad4, 0), 0), 0) <= Z::FWD, "leaf bound");
  int32_t x[Z::R1];
#pragma unroll
  for (int e = 0; e < Z::R1; ++e) {
    uint64_t m = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) m += (uint64_t)src(s + Z::S1 * e + Z::M * k) * c[k];
    x[e] = redc((int64_t)m, P.p, P.pinv);
  }
  fwd_net<Z::R1, 0>(
      x, [&](int l, int i) { return P.f[(node << l) + i]; }, [&](int l, int i) { return P.fv[(node << l) + i]; }, P.p,
      P.pinv);
#pragma unroll
  for (int e = 0; e < Z::R1; ++e) lds[Z::pos1(s, e)] = x[e];
}

// inverse pass 1 of set s of factor `node`: x[c] reduced, |x| < p
template <class Z>
__host__ __device__ __forceinline__ void inv1_quarter(int s, int node, const int32_t* lds, int32_t (&x)[Z::R1],
                                                      const Prime& P_) {
  const Prime P = local(P_);
#pragma unroll
  for (int c = 0; c < Z::R1; ++c) x[c] = lds[Z::pos1(s, c)];
  inv_net<Z::R1, kPassEnd, 0, false>(
      x, [&](int l, int i) { return P.b[(node << l) + i]; }, [&](int l, int i) { return P.bv[(node << l) + i]; }, P.p,
      P.pinv, P.one);
}

// the last two inverse levels: y[f] = a point of factor f (bound kPassEnd);
// y[k] = the residue of the coefficient of run k, bound 4 kPassEnd
__host__ __device__ __forceinline__ void join_quarters(int32_t (&y)[4], int32_t i_inv, const Prime& P) {
  const int32_t e0 = y[0] + y[1], d0 = y[0] - y[1], e1 = y[2] + y[3];
  const int32_t q = mont(y[2] - y[3], i_inv, P.p, P.pinv);
  y[0] = e0 + e1;
  y[2] = e0 - e1;
  y[1] = d0 + q;
  y[3] = d0 - q;
}

// ---- Chinese remainders ------------------------------------------------------------
__host__ __device__ __forceinline__ uint32_t canon(int32_t x, int32_t p) {   // (-p, p) -> [0, p)
  const uint32_t a = (uint32_t)x, b = (uint32_t)(x + p);
  return a < b ? a : b;
}

struct Crt {
  int32_t p1, p2;
  uint32_t i1, i2;           // p1^-1, p2^-1 mod 2^32
  int32_t c01, c02, c12;     // p0^-1 mod p1, p0^-1 mod p2, p1^-1 mod p2 (Montgomery form)
  uint32_t p0, p01l, p01h;   // p0, p0 p1
};
constexpr Crt make_crt() {
  const uint64_t p0 = kP[0], p1 = kP[1], p2 = kP[2];
  return Crt{kP[1], kP[2], inv32((uint32_t)p1), inv32((uint32_t)p2), to_mont_c(invmod(p0, p1), p1),
             to_mont_c(invmod(p0, p2), p2), to_mont_c(invmod(p1, p2), p2), (uint32_t)p0, (uint32_t)(p0 * p1),
             (uint32_t)((p0 * p1) >> 32)};
}
constexpr Crt kCrt = make_crt();
__device__ const Crt d_crt = kCrt;

// The next limb of a product: C = r0 + p0 k1 + p0 p1 k2 from r0 in [0, p0) and
// any representatives r1, r2 (|.| < 2^31 - p); returns the low limb of
// C + *acc and leaves the rest (< 2^50) in *acc.
__host__ __device__ __forceinline__ uint32_t crt_limb(uint32_t r0, int32_t r1, int32_t r2, uint64_t* acc,
                                                      const Crt& K) {
  const uint32_t k1 = canon(mont(r1 - (int32_t)r0, K.c01, K.p1, K.i1), K.p1);
  const int32_t u = mont(r2 - (int32_t)r0, K.c02, K.p2, K.i2) - (int32_t)k1;   // |u| < 2p
  const uint32_t k2 = canon(mont(u, K.c12, K.p2, K.i2), K.p2);
  const uint64_t low = (uint64_t)K.p0 * k1 + *acc + r0;   // < 2^54
  const uint64_t l = (uint64_t)K.p01l * k2 + low;         // < 2^60
  *acc = (uint64_t)K.p01h * k2 + (l >> 32);
  return (uint32_t)l;
}

// ---- the whole product on one work-group -------------------------------------------
#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)

// The cyclic convolution of a and b modulo the prime of P on the T threads
// t = 0 .. T - 1 (waves wv = 0 .. NW - 1 of a work-group whose other waves do
// the same for other primes); the residues of the coefficients stay in lds,
// in natural order, complete after the closing barrier.
template <class Z>
__device__ __forceinline__ void conv_prime(const Limbs& a, const Limbs& b, int t, int wv, int32_t* lds,
                                           const Prime& P, int32_t scale) {
  const int lane = t & 63;
  int32_t xa[4][Z::Q], xb[4][Z::Q];
  // (loops, also where they run once: unrolled or with their loads moved
  // ahead of the barriers, the kernel spills a hundred registers)
  auto fwd12 = [&](const Limbs& src) __attribute__((always_inline)) {
    if (src.n <= Z::M / 2) {
#pragma unroll 1
      for (int ch = wv; ch < Z::NC1; ch += Z::NW) fwd1<Z, true>(src, 64 * ch + lane, lds, P);
    } else {
#pragma unroll 1
      for (int ch = wv; ch < Z::NC1; ch += Z::NW) fwd1<Z, false>(src, 64 * ch + lane, lds, P);
    }
    __syncthreads();
#pragma unroll 1
    for (int s = t; s < Z::N2; s += Z::T) fwd2<Z>(s, lds, P);
    __syncthreads();
  };
  fwd12(a);
  fwd3<Z>(t, lds, xa, load3(t, P.f, P.fv), P);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int j = 0; j < Z::Q; ++j) xa[k][j] = mont(xa[k][j], scale, P.p, P.pinv);
  }
  __syncthreads();
  fwd12(b);
  const Roots3 w = load3(t, P.f, P.fv);
  fwd3<Z>(t, lds, xb, w, P);
  leaves<Z>(xa, xb, w, P);
  inv3<Z>(t, xb, lds, load3(t, P.b, P.bv), P);
  __syncthreads();
#pragma unroll 1
  for (int s = t; s < Z::N2; s += Z::T) inv2<Z>(s, lds, P);
  __syncthreads();
#pragma unroll 1
  for (int ch = wv; ch < Z::NC1; ch += Z::NW) {
    int32_t r[Z::R1];
    inv1<Z>(64 * ch + lane, lds, r, P);
#pragma unroll
    for (int c = 0; c < Z::R1; ++c) lds[Z::pos1(64 * ch + lane, c)] = r[c];
  }
  __syncthreads();
}

__device__ __forceinline__ Prime prime_of(int pr) {
  const Field& F = d_fields.f[pr];
  return Prime{F.p, F.pinv, F.one, F.load, (Tab)F.roots.f, (Tab)F.roots.fv, (Tab)F.roots.b, (Tab)F.roots.bv};
}

// Carries between the threads' runs of E limbs (thread order = limb order):
// the word above a run goes to limbs 0-1 of the next one, a carry out of
// limb 1 runs on through runs of all ones, one work-group scan.  over: one
// word of LDS per wave; scratch: 16 words.
template <int E>
__device__ __forceinline__ void close_runs(uint32_t (&x)[E], uint64_t acc, bool live, uint64_t* over,
                                           uint32_t* scratch) {
  const int lane = lane_id(), wv = wave_id();
  uint64_t d = ((uint64_t)(uint32_t)__builtin_amdgcn_update_dpp(0, (int)(acc >> 32), 0x138, 0xf, 0xf, false) << 32) |
               (uint32_t)__builtin_amdgcn_update_dpp(0, (int)acc, 0x138, 0xf, 0xf, false);
  if (num_waves() > 1) {
    if (lane == 63) over[wv] = acc;
    __syncthreads();
    if (lane == 0 && wv > 0) d = over[wv - 1];
  }
  uint32_t ones = 0xffffffffu;
#pragma unroll
  for (int e = 2; e < E; ++e) ones &= x[e];
  const uint64_t x0 = ((uint64_t)x[1] << 32) | x[0], y0 = x0 + d;
  const bool h = y0 < x0, full = live && ones == 0xffffffffu;
  const uint32_t c = wg_carry_scan(h && full, !h && full && y0 == ~0ull, 0u, scratch, nullptr);
  const uint64_t y = y0 + c;
  x[0] = (uint32_t)y;
  x[1] = (uint32_t)(y >> 32);
  if (h || y < y0) {
    bool on = true;
#pragma unroll
    for (int e = 2; e < E; ++e) {
      x[e] += on ? 1u : 0u;
      on = on && x[e] == 0u;
    }
  }
}

// out[0 .. nout) = a * b mod B^nout (nout <= na + nb <= M, the smaller operand
// at most 16,384 limbs) on T threads, one prime after another; lds:
// Z::LDS_BYTES.
template <class Z>
__device__ __forceinline__ void wg_mul_ntt(uint32_t* __restrict__ out, const uint32_t* __restrict__ a, int na,
                                           const uint32_t* __restrict__ b, int nb, int nout, int32_t* lds) {
  uint64_t* over = reinterpret_cast<uint64_t*>(lds + Z::LDS_WORDS);
  uint32_t* scratch = reinterpret_cast<uint32_t*>(over + Z::NW);
  const Limbs la(a, na), lb(b, nb), lo(out, nout);
  // residues of the first two primes: kept in private memory (the opaque
  // index keeps them there), the registers are needed for the next prime
  int32_t keep[2 * Z::S2];
  int zero = 0;
  asm volatile("" : "+v"(zero));
#pragma unroll 1
  for (int pr = 0; pr < kPrimes; ++pr) {
    // the thread's place, opaque per prime: nothing derived from it is held
    // in registers from one prime to the next
    int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(wave_id());
    asm volatile("" : "+v"(t));
    asm volatile("" : "+s"(wv));
    const Prime P = prime_of(pr);
    conv_prime<Z>(la, lb, t, wv, lds, P, d_fields.f[pr].scale[Z::K]);
    int32_t r[Z::S2];
    block_get<Z>(t, lds, r);
    __syncthreads();
    if (pr == 0) {
#pragma unroll
      for (int e = 0; e < Z::S2; ++e) keep[e + zero] = (int32_t)canon(mont(r[e], P.one, P.p, P.pinv), P.p);
    } else if (pr == 1) {
#pragma unroll
      for (int e = 0; e < Z::S2; ++e) keep[Z::S2 + e + zero] = r[e];
    } else {
      uint64_t acc = 0;
      uint32_t x[Z::S2];
#pragma unroll
      for (int e = 0; e < Z::S2; ++e)
        x[e] = crt_limb((uint32_t)keep[e + zero], keep[Z::S2 + e + zero], r[e], &acc, d_crt);
      close_runs<Z::S2>(x, acc, true, over, scratch);
      block_put<Z>(t, lds, reinterpret_cast<int32_t(&)[Z::S2]>(x));
      __syncthreads();
#pragma unroll 1
      for (int ch = wv; ch < Z::NC1; ch += Z::NW) {
        const int s = 64 * ch + (t & 63);
#pragma unroll
        for (int c2 = 0; c2 < Z::R1; ++c2) lo.put(s + Z::S1 * c2, (uint32_t)lds[Z::pos1(s, c2)]);
      }
    }
  }
}

// One prime and one factor of a product of 4 Z::M points, on T threads: the
// residues of the factor's points (bound kPassEnd) to y[0 .. Z::M).
template <class Z>
__device__ __forceinline__ void wg_ntt_quarter(int32_t* __restrict__ y, const uint32_t* __restrict__ a, int na,
                                               const uint32_t* __restrict__ b, int nb, int pr, int node,
                                               int32_t* lds) {
  const Limbs la(a, na), lb(b, nb);
  const Prime P = prime_of(pr);
  const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(wave_id());
  int32_t xa[4][Z::Q], xb[4][Z::Q];
  auto fwd12 = [&](const Limbs& src) __attribute__((always_inline)) {
    if (src.n <= 2 * Z::M) {
#pragma unroll 1
      for (int ch = wv; ch < Z::NC1; ch += Z::NW)
        fwd1_quarter<Z, true>(src, 64 * ch + lane, node, d_quarters.c[pr][node], lds, P);
    } else {
#pragma unroll 1
      for (int ch = wv; ch < Z::NC1; ch += Z::NW)
        fwd1_quarter<Z, false>(src, 64 * ch + lane, node, d_quarters.c[pr][node], lds, P);
    }
    __syncthreads();
#pragma unroll 1
    for (int s = t; s < Z::N2; s += Z::T) fwd2<Z>(s, lds, P, node);
    __syncthreads();
  };
  const Roots3 w = load3(node * Z::T + t, P.f, P.fv);
  const int32_t scale = d_fields.f[pr].scale[Z::K + 2];
  fwd12(la);
  fwd3<Z>(t, lds, xa, w, P);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int j = 0; j < Z::Q; ++j) xa[k][j] = mont(xa[k][j], scale, P.p, P.pinv);
  }
  __syncthreads();
  fwd12(lb);
  fwd3<Z>(t, lds, xb, w, P);
  leaves<Z>(xa, xb, w, P);
  inv3<Z>(t, xb, lds, load3(node * Z::T + t, P.b, P.bv), P);
  __syncthreads();
#pragma unroll 1
  for (int s = t; s < Z::N2; s += Z::T) inv2<Z>(s, lds, P, node);
  __syncthreads();
#pragma unroll 1
  for (int ch = wv; ch < Z::NC1; ch += Z::NW) {
    int32_t r[Z::R1];
    inv1_quarter<Z>(64 * ch + lane, node, lds, r, P);
#pragma unroll
    for (int c = 0; c < Z::R1; ++c) y[64 * ch + lane + Z::S1 * c] = r[c];
  }
}

// Joins the factors of a product (y[prime][node][m]) into limbs.  Thread j
// takes points 8 j .. 8 j + 7 of every factor, that is 8 limbs in each of the
// product's four runs of m limbs; a wave's 512 limbs in each run form a strip,
// resolved here but for what enters it from below: strip[2 w] = its carry word
// with "limbs 2..511 all ones" in bit 63, strip[2 w + 1] = its limbs 0-1.
constexpr int kRun = 8, kStripLimbs = 64 * kRun;
__device__ __forceinline__ void join_strip(uint32_t* __restrict__ out, int nout, const int32_t* __restrict__ y,
                                           int m, int j, uint64_t* strip) {
  const int lane = lane_id();
  int32_t r[kPrimes][4][kRun];
#pragma unroll
  for (int pr = 0; pr < kPrimes; ++pr) {
    const Prime P = prime_of(pr);
    const int32_t i_inv = P.b[1];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const v4i* src = reinterpret_cast<const v4i*>(y + ((int64_t)(pr * 4 + f) * m + kRun * j));
#pragma unroll
      for (int e = 0; e < kRun; e += 4) {
        const v4i v = src[e / 4];
        r[pr][f][e] = v.x; r[pr][f][e + 1] = v.y; r[pr][f][e + 2] = v.z; r[pr][f][e + 3] = v.w;
      }
    }
#pragma unroll
    for (int e = 0; e < kRun; ++e) {
      int32_t v[4] = {r[pr][0][e], r[pr][1][e], r[pr][2][e], r[pr][3][e]};
      join_quarters(v, i_inv, P);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        r[pr][k][e] = pr == 0 ? (int32_t)canon(mont(v[k], P.one, P.p, P.pinv), P.p) : v[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int base = k * m + kRun * j;   // this run's first limb
    uint64_t acc = 0;
    uint32_t x[kRun];
#pragma unroll
    for (int e = 0; e < kRun; ++e) x[e] = crt_limb((uint32_t)r[0][k][e], r[1][k][e], r[2][k][e], &acc, d_crt);
    const uint64_t d = ((uint64_t)(uint32_t)__builtin_amdgcn_update_dpp(0, (int)(acc >> 32), 0x138, 0xf, 0xf, false) << 32) |
                       (uint32_t)__builtin_amdgcn_update_dpp(0, (int)acc, 0x138, 0xf, 0xf, false);
    uint32_t ones = 0xffffffffu;
#pragma unroll
    for (int e = 2; e < kRun; ++e) ones &= x[e];
    const uint64_t x0 = ((uint64_t)x[1] << 32) | x[0], y0 = x0 + d;
    const bool h = y0 < x0, full = ones == 0xffffffffu;
    const bool g = h && full, pp = !h && full && y0 == ~0ull;
    const WaveCarry wc = wave_carry_masks(g, pp);
    const uint32_t c = wave_carry_in(wc, 0u);
    const uint64_t yy = y0 + c;
    x[0] = (uint32_t)yy;
    x[1] = (uint32_t)(yy >> 32);
    if (h || yy < y0) {
      bool on = true;
#pragma unroll
      for (int e = 2; e < kRun; ++e) {
        x[e] += on ? 1u : 0u;
        on = on && x[e] == 0u;
      }
    }
    if (base + kRun <= nout) {
      store4(out + base, x[0], x[1], x[2], x[3]);
      store4(out + base + 4, x[4], x[5], x[6], x[7]);
    } else {
#pragma unroll
      for (int e = 0; e < kRun; ++e)
        if (base + e < nout) out[base + e] = x[e];
    }
    // limbs of the strip from limb 2 up (limbs past the product count as ones)
    bool all = true;
#pragma unroll
    for (int e = 0; e < kRun; ++e) all = all && (x[e] == 0xffffffffu || base + e >= nout || (lane == 0 && e < 2));
    const bool tail = __ballot(all) == ~0ull;
    uint64_t* st = strip + 2 * (base / kStripLimbs);
    if (lane == 63) st[0] = (acc + wave_carry_out(wc, 0u)) | ((uint64_t)tail << 63);
    if (lane == 0) st[1] = yy;
  }
}

// The closing scan over the W <= 64 strips of a product, on one wave for its
// strip `mine` (every wave repeats the scan): strip w takes carry word w - 1
// at its limbs 0-1, one-bit carries run on through strips of all ones; a
// carry into strip `mine`'s tail runs up to its first limb not all ones.
__device__ __forceinline__ void close_joined(uint32_t* out, int nout, int W, const uint64_t* strip, int mine) {
  const int w = lane_id();
  const bool valid = w < W;
  const uint64_t kC = (1ull << 63) - 1;
  const uint64_t x0 = valid ? strip[2 * w + 1] : 0ull;
  const uint64_t x = x0 + ((valid && w > 0) ? (strip[2 * (w - 1)] & kC) : 0ull);
  const bool ones = valid && (strip[2 * w] >> 63), h = x < x0;
  const WaveCarry wc = wave_carry_masks(valid && h && ones, valid && !h && x == ~0ull && ones);
  const uint64_t y = x + wave_carry_in(wc, 0u);
  const int j0 = kStripLimbs * mine;
  if (w == mine && y != x0) {
    if (j0 < nout) out[j0] = (uint32_t)y;
    if (j0 + 1 < nout) out[j0 + 1] = (uint32_t)(y >> 32);
  }
  if (!(__ballot(h || y < x) >> mine & 1)) return;
  uint32_t v[kRun];
#pragma unroll
  for (int c = 0; c < kRun; ++c) {
    const int j = j0 + 64 * c + w;
    v[c] = j < nout ? out[j] : 0u;
  }
  bool on = true;
#pragma unroll
  for (int c = 0; c < kRun; ++c) {
    const int j = j0 + 64 * c + w;
    uint64_t stop = __ballot(v[c] != 0xffffffffu);
    if (c == 0) stop &= ~3ull;
    const int at = stop ? __ffsll((long long)stop) - 1 : 64;
    if (on && j < nout && w <= at && j >= j0 + 2) out[j] = v[c] + 1u;
    on = on && !stop;
  }
}

// LDS of wg_mul_ntt3
template <class Z>
constexpr size_t ntt3_lds_bytes() { return (size_t)3 * Z::LDS_WORDS * 4 + 3 * Z::NW * 8 + 128; }

// The same on 3T threads, the three primes side by side: a third of the
// latency, for batches that leave waves of the chip idle.  2T threads then
// recombine 2Q coefficients each.
template <class Z>
__device__ __forceinline__ void wg_mul_ntt3(uint32_t* __restrict__ out, const uint32_t* __restrict__ a, int na,
                                            const uint32_t* __restrict__ b, int nb, int nout, int32_t* lds) {
  constexpr int E = 2 * Z::Q;
  uint64_t* over = reinterpret_cast<uint64_t*>(lds + 3 * Z::LDS_WORDS);
  uint32_t* scratch = reinterpret_cast<uint32_t*>(over + 3 * Z::NW);
  const Limbs la(a, na), lb(b, nb), lo(out, nout);
  const int wv = __builtin_amdgcn_readfirstlane(wave_id()), pr = wv / Z::NW;
  const Prime P = prime_of(pr);
  conv_prime<Z>(la, lb, threadIdx.x - pr * Z::T, wv - pr * Z::NW, lds + pr * Z::LDS_WORDS, P,
                d_fields.f[pr].scale[Z::K]);
  const int t = threadIdx.x, at = (t >> 1) * Z::PS2 + (t & 1) * E;   // this thread's run of E points
  uint32_t x[E];
  uint64_t acc = 0;
  const bool live = t < 2 * Z::T;
  if (live) {
    const Field& F = d_fields.f[0];
    int32_t r[3][E];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int2* src = reinterpret_cast<const int2*>(lds + q * Z::LDS_WORDS + at);
#pragma unroll
      for (int e = 0; e < E / 2; ++e) {
        const int2 v = src[e];
        r[q][2 * e] = v.x;
        r[q][2 * e + 1] = v.y;
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
      x[e] = crt_limb(canon(mont(r[0][e], F.one, F.p, F.pinv), F.p), r[1][e], r[2][e], &acc, d_crt);
  }
  close_runs<E>(x, acc, live, over, scratch);
  if (live) {
    int2* dst = reinterpret_cast<int2*>(lds + at);
#pragma unroll
    for (int e = 0; e < E / 2; ++e) dst[e] = int2{(int)x[2 * e], (int)x[2 * e + 1]};
  }
  __syncthreads();
#pragma unroll 4
  for (int i = t; i < nout; i += 3 * Z::T) out[i] = (uint32_t)lds[(i / Z::S2) * Z::PS2 + i % Z::S2];
}

#endif

}  // namespace ntt
}  // namespace bi
