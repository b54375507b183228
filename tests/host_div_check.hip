// The extent of every buffer and product of a division in pieces, over edge
// and random sizes: the steps of wg_divmod and shifted_inverse with lengths in
// place of numbers, on the sizes that the kernels themselves compute.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../paper_2607_28897_amd/csrc/dev_divmod.hpp"

using namespace bi::div;

static long checked = 0;
#define NEED(c)                                                                                              \
  do {                                                                                                       \
    if (!(c)) {                                                                                              \
      printf("%s: %d / %d limbs (%d / %d used), capacities %d / %d, products %d\n", #c, nu, nv, h, k1, capu, \
             capv, prod);                                                                                    \
      exit(1);                                                                                               \
    }                                                                                                        \
  } while (0)

// dividend and divisor of nu and nv limbs, h and k1 of them used, in a batch
// with slots for capu and capv limbs and LDS for products of prod limbs
static void check(int nu, int nv, int k1, int h, int capu, int capv, int prod) {
  if (k1 < 2 || h < k1) return;   // (other paths, without products)
  ++checked;
  static uint32_t base[1];
  const Bufs bf = carve_bufs(base, capu, capv);
  NEED((size_t)(bf.T - base) + bf.ct == div_ws_limbs(capu, capv));
  NEED(bf.U2 - bf.W == bf.cw && bf.E - bf.U2 == bf.cw && bf.T - bf.E == bf.ce);
  const size_t lds[4] = {bi::mfma::lds_bytes_sum(prod, 1, kP), bi::mfma::lds_bytes_sum(prod, 2, kP),
                         bi::mfma::lds_bytes_sum(prod, 4, kP), bi::mfma::lds_bytes_sum(prod, 8, kP)};
  // a product of a and b limbs to out limbs of room
  auto product = [&](int a, int b, int room) {
    NEED(a >= 1 && b >= 1 && a + b <= room);
    if (a <= kSmallMul && b <= kSmallMul) return;
    NEED(a + b <= prod);
    for (int i = 0; i < 4; ++i) NEED(bi::mfma::lds_bytes<kDW>(a, b, 1 << i, kP) <= lds[i]);
  };
  // a product of which only `out` limbs are wanted, to `room`
  auto low = [&](int a, int b, int out, int room) {
    NEED(out <= room);
    product(a, b, a + b);
  };
  const int s = piece_limbs(h - k1, k1, prod);
  const int pieces = s > 0 ? (h - k1 + s - 1) / s : 1, h2 = k1 + s;
  NEED(pieces >= 1 && s >= 0 && (pieces - 1) * s <= h - k1);
  int lw_end = 0;
  for (int extra = 0; extra < 2; ++extra) {   // w at its usual and its largest length
    int cur = k1 + 2;
    if (cur > h2) cur = h2;
    int lw = cur - k1 + 1 + extra;
    if (lw > 4) lw = 4;
    while (cur < h2) {
      const int m = std::min(h2 - cur, cur - k1 - 1);
      NEED(m >= 1);
      const int t = std::min(k1, cur + m - k1 + 1 + kGuard), c = cur - (k1 - t), le = t + 2;
      low(t, lw, le, bf.ce);
      const int sd = std::max(0, std::min(le - 1, c - m - 1 - lw));
      NEED(c - m - sd >= 0);
      product(lw, le - sd, bf.ct);
      NEED(lw + m + 1 <= bf.cw);
      cur += m;
      lw = cur - k1 + 1 + extra;
    }
    lw_end = lw;
    const int lr = k1 + 2;
    for (int p = pieces - 1; p >= 0; --p) {
      const int hd = p == pieces - 1 ? h - p * s : k1 + s;
      NEED(hd >= 1 && hd <= h2);
      const int su = std::max(0, h2 - 1 - lw), nd = hd - su;
      product(nd, lw, pieces == 1 ? bf.ct : 2 * s + 8);   // (buf1 lies behind)
      int lq = nd + lw - (h2 - su);
      NEED(lq >= 1 && (h2 - su) + lq <= nd + lw);
      if (p < pieces - 1) lq = std::min(lq, s + 1);
      low(lq, k1, lr, bf.ce);
      const int off = p > 0 ? s : 0;
      NEED(off + lr <= bf.cw);                              // buf0
      if (pieces > 1) NEED(2 * s + 8 + off + lr <= bf.ct);  // buf1
      NEED(p == 0 || p * s - s >= 0);
      NEED(p * s < std::max(h, 1));
    }
  }
  (void)lw_end;
}

static void uniform(int nu, int nv, int k1, int h) {
  if (k1 > nv || h > nu) return;
  check(nu, nv, k1, h, nu, nv, (int)product_limbs(nu, nv));
}

int main() {
  std::mt19937 g(1);
  auto pick = [&](int lo, int hi) { return lo + (int)(g() % (unsigned)(hi - lo + 1)); };
  const int more[] = {299, 300, 301, 302, 303, 310, 600, 601, 602, 650, 1000};
  for (int i = 2; i < 60 + 11; ++i) {
    const int nu = i < 60 ? i : more[i - 60];
    for (int j = 2; j < 40 + 7; ++j) {
      const int edge[] = {nu - 301, nu - 300, nu - 299, nu / 2, nu - 1, nu, nu + 5};
      const int nv = j < 40 ? j : edge[j - 40];
      if (nv < 2) continue;
      for (int k1 : {2, 3, 4, 5, nv / 2, nv - 1, nv})
        for (int h : {k1, k1 + 1, k1 + 2, k1 + 3, nu / 2, nu - 1, nu}) uniform(nu, nv, k1, h);
    }
  }
  for (int i = 0; i < 300000; ++i) {
    int nu = (int)(2 * std::pow(8192.0, (g() >> 8) / 16777216.0));
    nu = std::max(2, std::min(16384, nu));
    const int nv = pick(2, std::min(16384, nu + 20));
    const int r = pick(0, 2), k1 = r == 0 ? nv : (r == 1 ? 2 : pick(2, nv));
    if (k1 > nu) continue;
    const int h = pick(0, 1) ? nu : pick(k1, nu);
    uniform(nu, nv, k1, h);
    // in a ragged batch with larger dividends, divisors and products
    const int capu = std::min(16384, nu + pick(0, 3000)), capv = std::min(16384, nv + pick(0, 300));
    check(nu, nv, k1, h, capu, capv,
          (int)std::max(product_limbs(nu, nv), product_limbs(capu, pick(1, capv))));
  }
  printf("%ld divisions\n", checked);
  return checked < 500000;
}
