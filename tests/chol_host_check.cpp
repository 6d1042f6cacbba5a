// Host driver for the steps of the blocked Cholesky factor (chol_steps.hpp):
// one thread a lane, barriers that count every thread, and lane exchanges
// between threads.  A schedule hook delays some threads after a barrier or an
// exchange, as a wavefront or lane may run late on the device.
//
//   diag N BAD LATE   factor of an N x N block whose column BAD breaks down (-1:
//                     none); wave LATE runs late after every barrier (-1: none).
//                     Prints the result of every wave, or "hang" when a barrier
//                     waits for a wave that has left.
//   tri RB CJ LATE    substitution of 16 right hand sides, RB unknowns, conjugated
//                     triangle for CJ = 1; lane LATE of every quad runs late after
//                     every exchange (-1: none).  Prints the largest deviation.
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#define __device__
struct cplx {
  double x, y;
};
static inline cplx cmk(double r, double i) { return cplx{r, i}; }
static inline cplx cscale(cplx a, double s) { return cplx{a.x * s, a.y * s}; }
using std::fma;
using std::sqrt;
constexpr int CHOL_NB = 64;

struct Hang {};
class Barrier {
 public:
  explicit Barrier(int n = 4) : n_(n) {}
  void wait() {
    std::unique_lock<std::mutex> lk(m_);
    const long gen = gen_;
    if (++in_ == n_) {
      in_ = 0;
      ++gen_;
      cv_.notify_all();
      return;
    }
    if (!cv_.wait_for(lk, std::chrono::seconds(20), [&] { return gen_ != gen; })) throw Hang{};
  }

 private:
  std::mutex m_;
  std::condition_variable cv_;
  int n_, in_ = 0;
  long gen_ = 0;
};

struct Dim {
  unsigned x;
};
static thread_local Dim threadIdx;
static Barrier* g_block;                       // 256 threads
static Barrier* g_wave[4];                     // 64 threads each
static double g_lane[256];
static Barrier g_quad[64];                     // 4 lanes each
static int g_quad_v[256];
static int g_late = -1, g_late_lane = -1;
static void nap() { std::this_thread::sleep_for(std::chrono::milliseconds(4)); }

static void __syncthreads() {
  g_block->wait();
  if ((int)(threadIdx.x >> 6) == g_late) nap();
}
static double __shfl(double v, int src) {
  const int w = threadIdx.x >> 6;
  g_lane[threadIdx.x] = v;
  g_wave[w]->wait();
  const double r = g_lane[w * 64 + src];
  g_wave[w]->wait();
  return r;
}
// a quad's lanes all take the value of lane ctrl & 3
static int __builtin_amdgcn_update_dpp(int, int v, int ctrl, int, int, bool) {
  const int t = threadIdx.x;
  g_quad_v[t] = v;
  g_quad[t >> 2].wait();
  const int r = g_quad_v[(t & ~3) + (ctrl & 3)];
  g_quad[t >> 2].wait();
  if ((t & 3) == g_late_lane) std::this_thread::sleep_for(std::chrono::microseconds(200));
  return r;
}
static void wave_sync() { g_wave[threadIdx.x >> 6]->wait(); }

#include "chol_steps.hpp"

// Hermitian positive definite n x n matrix, or with column `bad` a copy of
// column 0 (bad > 0) or a zero column (bad = 0): breakdown there
static std::vector<cplx> matrix(int n, int bad) {
  std::mt19937 gen(7);
  std::normal_distribution<double> g;
  std::vector<cplx> r((size_t)n * n), a((size_t)n * n);
  for (auto& v : r) v = cmk(g(gen), g(gen));
  if (bad >= 0)
    for (int k = 0; k < n; ++k) r[(size_t)bad * n + k] = bad > 0 ? r[k] : cmk(0.0, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      cplx s = cmk(0.0, 0.0);
      for (int k = 0; k < n; ++k) {
        const cplx x = r[(size_t)i * n + k], y = r[(size_t)j * n + k];
        s.x += x.x * y.x + x.y * y.y;
        s.y += x.y * y.x - x.x * y.y;
      }
      a[(size_t)i * n + j] = s;
    }
  return a;
}

static int run_diag(int n, int bad, int late) {
  const std::vector<cplx> a = matrix(n, bad);
  double dmax = 0.0;
  for (int i = 0; i < n; ++i) dmax = std::fmax(dmax, a[(size_t)i * n + i].x);
  std::vector<cplx> l((size_t)n * n);
  static cplx col[2][CHOL_NB];
  static int s_bad[2];
  Barrier block(256), w0(64), w1(64), w2(64), w3(64);
  g_block = &block;
  Barrier* ws[4] = {&w0, &w1, &w2, &w3};
  memcpy(g_wave, ws, sizeof(ws));
  g_late = late;
  bool hang = false, ok[256];
  std::vector<std::thread> th;
  for (int t = 0; t < 256; ++t)
    th.emplace_back([&, t] {
      threadIdx.x = t;
      const int lane = t & 63, w = t >> 6;
      cplx d[16];
      for (int e = 0; e < 16; ++e) {
        const int c = 4 * e + w;
        d[e] = lane < n && c <= lane ? a[(size_t)lane * n + c] : cmk(0.0, 0.0);
      }
      try {
        block.wait();
        ok[t] = diag_steps<0>(d, col, s_bad, 1e-13 * dmax, n, lane, w);
      } catch (const Hang&) {
        hang = true;
        return;
      }
      if (ok[t])
        for (int e = 0; e < 16; ++e)
          if (lane < n && 4 * e + w <= lane) l[(size_t)lane * n + 4 * e + w] = d[e];
    });
  for (auto& t : th) t.join();
  if (hang) {
    printf("hang\n");
    return 0;
  }
  for (int t = 0; t < 256; ++t)
    if (ok[t] != ok[0]) {
      printf("divided\n");
      return 0;
    }
  if (!ok[0]) {
    printf("breakdown\n");
    return 0;
  }
  double err = 0.0;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j <= i; ++j) {
      cplx s = cmk(0.0, 0.0);
      for (int k = 0; k <= j; ++k) {
        const cplx x = l[(size_t)i * n + k], y = l[(size_t)j * n + k];
        s.x += x.x * y.x + x.y * y.y;
        s.y += x.y * y.x - x.x * y.y;
      }
      err = std::fmax(err, std::hypot(s.x - a[(size_t)i * n + j].x, s.y - a[(size_t)i * n + j].y) / dmax);
    }
  printf("factor %.3e\n", err);
  return 0;
}

template <bool CJ>
static int run_tri(int rb, int late) {
  static Tri64 t;
  std::mt19937 gen(11);
  std::normal_distribution<double> g;
  for (int c = 0; c < CHOL_NB; ++c) {
    for (int d = 0; d < CHOL_NB; ++d) t.T[d][c] = d < c ? cmk(0.1 * g(gen), 0.1 * g(gen)) : cmk(d == c, 0.0);
    const double diag = 1.0 + 0.5 * (c % 3);
    t.T[c][c] = cmk(diag, 0.0);
    t.rinv[c] = 1.0 / diag;
    for (int r = 0; r < 64; ++r) t.X[r][c] = cmk(g(gen), g(gen));
  }
  const Tri64 in = t;
  Barrier w0(64);
  g_wave[0] = &w0;
  g_late_lane = late;
  std::vector<std::thread> th;
  for (int i = 0; i < 64; ++i)
    th.emplace_back([&, i] {
      threadIdx.x = i;
      tri_solve64<CJ>(t, rb);
    });
  for (auto& x : th) x.join();
  double err = 0.0;
  for (int r = 0; r < 16; ++r) {
    cplx x[CHOL_NB];
    for (int c = 0; c < rb; ++c) {
      cplx s = in.X[r][c];
      for (int d = 0; d < c; ++d) {
        const cplx l = cmk(in.T[d][c].x, CJ ? -in.T[d][c].y : in.T[d][c].y);
        s.x -= l.x * x[d].x - l.y * x[d].y;
        s.y -= l.x * x[d].y + l.y * x[d].x;
      }
      x[c] = cscale(s, in.rinv[c]);
      err = std::fmax(err, std::hypot(x[c].x - t.X[r][c].x, x[c].y - t.X[r][c].y) / (1.0 + std::hypot(x[c].x, x[c].y)));
    }
  }
  printf("%.3e\n", err);
  return 0;
}

int main(int argc, char** argv) {
  if (argc == 5 && !strcmp(argv[1], "diag")) return run_diag(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
  if (argc == 5 && !strcmp(argv[1], "tri"))
    return atoi(argv[3]) ? run_tri<true>(atoi(argv[2]), atoi(argv[4])) : run_tri<false>(atoi(argv[2]), atoi(argv[4]));
  return 2;
}
