// Workspace layouts of Stage 3's factor calls, in doubles from the (256-byte
// aligned) workspace's start. Host arithmetic only.
#pragma once

#include <stdint.h>

namespace lx {

// Partial products: at most kDgParts doubles. (The rotation log of k_jacobi
// takes the same buffer: 40 sweeps of 127 steps of 64 rotations at most.)
constexpr int64_t kDgParts = 384 * 64 * 64;

struct Stage3Ws {
  int64_t R;     // rows x cols: the residual
  int64_t Xp;    // weighted fit: np x cols
  int64_t P;     // weighted fit: cols x l
  int64_t Y;     // rows x l
  int64_t Z;     // cols x l (weighted fit: np x l)
  int64_t T;     // l x cols: Y^T R
  int64_t Wt;    // weighted fit: l x np
  int64_t G, U, Ve;  // lp x lp each
  int64_t lam, sig;  // lp each
  int64_t Ad;    // rows x l
  int64_t part;  // kDgParts, on a 16-byte boundary: the log is read and written as pairs
  int64_t total;
};

// np < 0: the plain fit. total counts four lp x lp blocks, of which three are
// in use: the fourth's at least 4 doubles hold the padding before part.
inline Stage3Ws stage3_ws(int64_t rows, int64_t cols, int64_t np, int64_t l) {
  const int64_t lp = l + (l & 1);
  const bool weighted = np >= 0;
  Stage3Ws w{};
  int64_t at = 0;
  auto take = [&](int64_t n) {
    const int64_t a = at;
    at += n;
    return a;
  };
  w.R = take(rows * cols);
  w.Xp = take(weighted ? np * cols : 0);
  w.P = take(weighted ? cols * l : 0);
  w.Y = take(rows * l);
  w.Z = take((weighted ? np : cols) * l);
  w.T = take(l * cols);
  w.Wt = take(weighted ? l * np : 0);
  w.G = take(lp * lp);
  w.U = take(lp * lp);
  w.Ve = take(lp * lp);
  w.lam = take(lp);
  w.sig = take(lp);
  w.Ad = take(rows * l);
  w.total = at + lp * lp + kDgParts;
  w.part = (at + 1) / 2 * 2;
  return w;
}

}  // namespace lx
