// The passes of the transform multiply on the host, thread after thread: every
// size that is built, whole and as a quarter of four times the points, against
// schoolbook products.  Signed overflow traps (the bounds of the lazily reduced
// sums are worst cases that the headers assert at compile time; these operands
// stay far below them), and the sets of each pass must cover the same LDS
// words, each once.
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "../paper_2607_28897_amd/csrc/dev_mul_ntt.hpp"

using namespace bi::ntt;
typedef std::vector<uint32_t> Vec;
static const Field* kField[3] = {&kF0, &kF1, &kF2};

static Vec school(const Vec& a, const Vec& b) {
  Vec r(a.size() + b.size(), 0);
  for (size_t i = 0; i < a.size(); ++i) {
    uint64_t c = 0;
    for (size_t j = 0; j < b.size(); ++j) {
      const uint64_t t = (uint64_t)a[i] * b[j] + r[i + j] + c;
      r[i + j] = (uint32_t)t;
      c = t >> 32;
    }
    r[i + b.size()] = (uint32_t)c;
  }
  return r;
}

struct Src {
  const Vec& v;
  uint32_t operator()(int i) const { return i < (int)v.size() ? v[i] : 0u; }
};

static bool fail(const char* what) {
  printf("%s\n", what);
  return false;
}

// res[0 .. Z::M): the residues of the convolution of a and b, of the whole
// product (node 0) or of factor `node` of a product of four times the points
template <class Z, bool QUARTER>
static bool conv(const Vec& a, const Vec& b, int pr, int node, int32_t* res) {
  const Field& F = *kField[pr];
  const Prime P{F.p, F.pinv, F.one, F.load, F.roots.f, F.roots.fv, F.roots.b, F.roots.bv};
  const int t0 = node * Z::T;
  const int32_t scale = leaf_scale(pr, Z::K + (QUARTER ? 2 : 0));
  std::vector<int32_t> words(Z::LDS_WORDS + 4);
  int32_t* lds = (int32_t*)(((uintptr_t)words.data() + 15) & ~(uintptr_t)15);
  std::vector<int32_t> keep((size_t)Z::T * Z::S2);
  for (int op = 0; op < 2; ++op) {
    const Vec& v = op ? b : a;
    const Src src{v};
    std::vector<char> hit(Z::LDS_WORDS, 0), hit2(Z::LDS_WORDS, 0);
    for (int s = 0; s < Z::S1; ++s) {
      if constexpr (!QUARTER) {
        if ((int)v.size() <= Z::M / 2) fwd1<Z, true>(src, s, lds, P);
        else fwd1<Z, false>(src, s, lds, P);
      } else {
        if ((int)v.size() <= 2 * Z::M) fwd1_quarter<Z, true>(src, s, node, kQuarters.c[pr][node], lds, P);
        else fwd1_quarter<Z, false>(src, s, node, kQuarters.c[pr][node], lds, P);
      }
      for (int c = 0; c < Z::R1; ++c) {
        const int q = Z::pos1(s, c);
        if (q < 0 || q >= Z::LDS_WORDS || hit[q]) return fail("pass 1: position");
        hit[q] = 1;
      }
    }
    for (int s = 0; s < Z::N2; ++s) {
      for (int c = 0; c < Z::R2; ++c) {
        const int q = Z::pos2(s, c);
        if (q < 0 || q >= Z::LDS_WORDS || hit2[q]) return fail("pass 2: position");
        hit2[q] = 1;
      }
      fwd2<Z>(s, lds, P, node);
    }
    if (hit != hit2) return fail("passes 1 and 2 cover different words");
    if (op == 0) {
      for (int t = 0; t < Z::T; ++t) {
        int32_t x[4][Z::Q];
        fwd3<Z>(t, lds, x, load3(t0 + t, P.f, P.fv), P);
        for (int k = 0; k < 4; ++k)
          for (int j = 0; j < Z::Q; ++j) keep[t * Z::S2 + k * Z::Q + j] = mont(x[k][j], scale, P.p, P.pinv);
      }
    }
  }
  for (int t = 0; t < Z::T; ++t) {
    int32_t x[4][Z::Q], y[4][Z::Q];
    const Roots3 w = load3(t0 + t, P.f, P.fv);
    memcpy(x, &keep[(size_t)t * Z::S2], sizeof x);
    fwd3<Z>(t, lds, y, w, P);
    leaves<Z>(x, y, w, P);
    inv3<Z>(t, y, lds, load3(t0 + t, P.b, P.bv), P);
  }
  for (int s = 0; s < Z::N2; ++s) inv2<Z>(s, lds, P, node);
  for (int s = 0; s < Z::S1; ++s) {
    int32_t x[Z::R1];
    if constexpr (!QUARTER) inv1<Z>(s, lds, x, P);
    else inv1_quarter<Z>(s, node, lds, x, P);
    for (int c = 0; c < Z::R1; ++c) res[s + Z::S1 * c] = x[c];
  }
  return true;
}

template <class Z, bool QUARTER>
static bool product(int na, int nb, bool ones, unsigned seed) {
  std::mt19937 g(seed);
  Vec a(na), b(nb);
  for (auto& x : a) x = ones ? 0xffffffffu : g();
  for (auto& x : b) x = ones ? 0xffffffffu : g();
  const int M = QUARTER ? 4 * Z::M : Z::M;
  std::vector<int32_t> res[3];
  for (int pr = 0; pr < 3; ++pr) {
    res[pr].resize(M);
    if constexpr (!QUARTER) {
      if (!conv<Z, false>(a, b, pr, 0, res[pr].data())) return false;
    } else {
      const Field& F = *kField[pr];
      const Prime P{F.p, F.pinv, F.one, F.load, F.roots.f, F.roots.fv, F.roots.b, F.roots.bv};
      for (int f = 0; f < 4; ++f)
        if (!conv<Z, true>(a, b, pr, f, res[pr].data() + f * Z::M)) return false;
      for (int m = 0; m < Z::M; ++m) {
        int32_t y[4];
        for (int f = 0; f < 4; ++f) y[f] = res[pr][f * Z::M + m];
        join_quarters(y, P.b[1], P);
        for (int f = 0; f < 4; ++f) res[pr][f * Z::M + m] = y[f];
      }
    }
  }
  const Vec want = school(a, b);
  uint64_t acc = 0;
  for (int k = 0; k < M; ++k) {
    const Field& F = *kField[0];
    const uint32_t r0 = canon(mont(res[0][k], F.one, F.p, F.pinv), F.p);
    const uint32_t limb = crt_limb(r0, res[1][k], res[2][k], &acc, kCrt);
    if (acc >> 50) return fail("carry word");
    if (limb != (k < na + nb ? want[k] : 0u)) return fail("limb");
  }
  return true;
}

static int failures = 0, checked = 0;

template <int T, int Q, int R1, int R2, bool QUARTER = false>
static void size() {
  typedef Size<T, Q, R1, R2> Z;
  const int M = QUARTER ? 4 * Z::M : Z::M;
  const int shapes[3][2] = {{M / 2, M - M / 2}, {M - 3, 3}, {7, M / 3}};
  for (const auto& s : shapes)
    for (int ones = 0; ones < 2; ++ones) {
      ++checked;
      if (!product<Z, QUARTER>(s[0], s[1], ones, 5u + M)) {
        printf("  %d points, %d x %d limbs%s\n", M, s[0], s[1], ones ? ", all ones" : "");
        ++failures;
      }
    }
}

int main() {
  size<256, 2, 16, 16>();
  size<128, 6, 8, 16>();
  size<256, 3, 16, 16>();
  size<256, 4, 16, 16>();
  size<256, 5, 16, 16>();
  size<256, 6, 16, 16>();
  size<256, 7, 16, 16>();
  size<256, 8, 16, 16>();
  size<512, 5, 32, 16>();
  size<512, 6, 32, 16>();
  size<512, 7, 32, 16>();
  size<512, 8, 32, 16>();
  size<1024, 5, 32, 32>();
  size<1024, 6, 32, 32>();
  size<1024, 7, 32, 32>();
  size<1024, 8, 32, 32>();
  size<256, 3, 16, 16, true>();
  size<256, 5, 16, 16, true>();
  size<256, 8, 16, 16, true>();
  printf("%d products, %d wrong\n", checked, failures);
  return failures != 0;
}
