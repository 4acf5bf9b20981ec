// Linear regression through its normal equations (gfx950).
//
// With a squared loss the inner gradient of batch b is (2/N) (G_b theta - c_b),
// G_b = X_b^T X_b and c_b = X_b^T y_b, and its Hessian-vector product is
// (2/N) G_b v (Section 2.2).  Neither G_b nor c_b depends on theta, so all of
// them are formed at once over the whole chip (linreg_gram_kernel); what is left
// of the sweep is one d x d matrix-vector product per phase, in one workgroup
// (linreg_sweep_kernel).  Walking the batches themselves, 2 T + 1 of them, one
// compute unit receives about 20 bytes a cycle: 130 features, 1000 rows, T = 3
// took 620 us that way, 24 us this way.
//
// G, c and the whole sweep are float64.  Near a fit, or with features far from
// zero mean, G theta - c cancels: from float32 matrices d eta lay up to six times as
// far from the exact one as from float32 residuals (200 features, 50 rows, T = 2,
// mean 3, at the fit: 7.1e-4 against 1.1e-4; now 5e-8).  The products of float32
// values are exact in float64, so the sums are what rounds, at 1e-16.
#include <algorithm>

#include "kernels.h"

namespace mfmg {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int GR_THREADS = 1024;
constexpr int GR_WAVES = GR_THREADS / 64;

struct GramArgs {
  const float* xs[LINREG_MAXT + 1];   // the T training batches, then the validation batch
  const float* ys[LINREG_MAXT + 1];
  int T, rows, vrows, d;
  int nr, ldg;                    // rows (d + 1 in whole tiles) and row pitch of G
  int rps, rounds;                // of the sweep: rows a step; rounds of R steps a phase
  double* G;                      // [T + 1][nr][ldg], zero past row d
  const float* theta0;
  const float* eta;
  double* gsave;                  // [T][d] inner gradients
  float* d_eta;
  float* val_loss;
};

// [X | y]^T [X | y] of every batch: one workgroup per 16 x 16 output tile on or
// above the diagonal, whose 16 waves take every 16th group of four rows; the
// v_mfma_f64_16x16x4_f64 operands are read straight from the rows (lane: column
// lane % 16 of row lane / 16, 64-byte runs), so no LDS staging is needed.  Small
// tiles, because the batches are few: 130 features and T = 3 give 180 workgroups
// (60 with 32 x 32 tiles, and four times the matrix work in each).  The waves' sums
// are added in wave order.
__global__ void __launch_bounds__(GR_THREADS) linreg_gram_kernel(GramArgs a) {
  __shared__ double part[GR_WAVES][16 * 17];
  const int b = blockIdx.y;
  const int nt = a.nr / 16;
  int p = blockIdx.x, ti = 0;
  while (p >= nt - ti) {
    p -= nt - ti;
    ++ti;
  }
  const int tj = ti + p;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float* X = a.xs[b];
  const float* y = a.ys[b];
  const int rows = b < a.T ? a.rows : a.vrows;
  // two columns per lane: one of the tile's rows, one of its columns
  const float* base[2];
  unsigned stride[2];
  bool in[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c = (q == 0 ? ti : tj) * 16 + (lane & 15);
    base[q] = c < a.d ? X + c : y;
    stride[q] = c < a.d ? a.d : 1;
    in[q] = c <= a.d;
  }
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  constexpr int UN = 8;   // steps whose loads are in flight together
  const int steps = (rows + 4 * GR_WAVES - 1) / (4 * GR_WAVES);
  for (int s0 = 0; s0 < steps; s0 += UN) {
    float v[UN][2];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int r = (s0 + u) * 4 * GR_WAVES + 4 * w + (lane >> 4);
#pragma unroll
      for (int q = 0; q < 2; ++q) v[u][q] = base[q][(unsigned)min(r, rows - 1) * stride[q]];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (s0 + u >= steps) break;
      const int r = (s0 + u) * 4 * GR_WAVES + 4 * w + (lane >> 4);
#pragma unroll
      for (int q = 0; q < 2; ++q) v[u][q] = in[q] && r < rows ? v[u][q] : 0.0f;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[u][0], (double)v[u][1], acc, 0, 0, 0);
    }
  }
  // lane and element r of the result: row 4 r + lane / 16, column lane % 16
#pragma unroll
  for (int r = 0; r < 4; ++r) part[w][(4 * r + (lane >> 4)) * 17 + (lane & 15)] = acc[r];
  __syncthreads();
  if (tid >= 256) return;
  double* G = a.G + (long)b * a.nr * a.ldg;
  const int r = tid >> 4, c = tid & 15;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < GR_WAVES; ++k) s += part[k][r * 17 + c];
  const int gr = ti * 16 + r, gc = tj * 16 + c;
  if (gc < a.ldg) G[(long)gr * a.ldg + gc] = s;
  if (ti != tj && gr < a.ldg) G[(long)gc * a.ldg + gr] = s;   // the mirrored tile
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ double quad_sum(double v) {   // over the four lanes of a quad
  v += dpp_f64<0xB1>(v);
  v += dpp_f64<0x4E>(v);
  return v;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The sweep: T inner steps, the seed at theta_T, T reverse steps, in one workgroup of
// NT threads.  The rows 0 .. d - 1 of G, each ldg / 2 pieces of 16 bytes, are read as
// one run of pieces, rps whole rows a step (NT pieces but for a last part of a row): a
// compute unit's loads bound the sweep (64 bytes a cycle), so none may be spent on
// lanes past a row's end (a power of two of lanes per row, half of them past the end
// at 130 features, took 3.1 us a phase there, this 1.8).  A thread keeps R pieces
// in flight: a piece is replaced by the one R steps on, of the next phase's matrix at
// the end.  The column sums go over a thread's steps, then over the rps rows of a step
// through LDS (four lanes per column), in a fixed order.
// The validation loss is theta^T (G theta - 2 c) + y^T y of its batch: what cancels there
// is 1e-16 of |y|^2, less than the square of a float32 residual's rounding.
constexpr int GR_RPS = 32;      // most rows a step
constexpr int GR_XROWS = 512;   // rows of all steps, at most

template <int NT, int R>
__global__ void __launch_bounds__(NT) linreg_sweep_kernel(GramArgs a) {
  __shared__ double x[GR_XROWS];           // the vector of this phase, zero past d
  __shared__ __attribute__((aligned(16))) double part[2 * NT];   // [rps][ldg]
  __shared__ double red[NT / 64];
  const int tid = threadIdx.x;
  const int d = a.d, T = a.T, ldg = a.ldg, cp = ldg >> 1;
  const int rps = a.rps, span = rps * cp, rounds = a.rounds;
  const int row0 = min(tid / cp, rps - 1);
  const int last = a.nr * cp - 1;
  double2 g[R];
  // piece of step k0 + k; past G's rows its last one (x is zero there)
  const int own_piece = min(tid, span - 1);
  auto load = [&](int b, int k0, int k) {
    const double2* G = reinterpret_cast<const double2*>(a.G) + (long)b * (last + 1);
    g[k] = G[(unsigned)min((k0 + k) * span + own_piece, last)];
  };
  // thread 4 j + q works on column j
  const int q = tid & 3, j = min(tid >> 2, d - 1);
  const bool own = (tid >> 2) < d && q == 0;
#pragma unroll
  for (int k = 0; k < R; ++k) load(0, 0, k);
  auto rhs = [&](int b) { return a.G[((long)b * a.nr + d) * ldg + j]; };   // c_b
  double c = rhs(0), th = a.theta0[j], tb = 0.0, eb = 0.0;
  const float eta = a.eta[j];
  for (int i = tid; i < GR_XROWS; i += NT) x[i] = 0.0;
  __syncthreads();
  const double lam = expf(eta);
  if (own) x[j] = th;
  __syncthreads();
  const double inv = 2.0 / a.rows, invv = 2.0 / a.vrows;
  // Phases 0 .. 2 T: the training batches, the validation batch, the training batches
  // in reverse.
#pragma unroll 1
  for (int p = 0; p <= 2 * T; ++p) {
    const int b = p <= T ? p : 2 * T - p;
    const int nb = p < T ? p + 1 : max(2 * T - p - 1, 0);   // the next phase's
    double gr = 0.0;
    if (p > T && own) gr = a.gsave[(long)b * d + j];   // by the lane that saved it
    double2 s = make_double2(0.0, 0.0);
#pragma unroll 1
    for (int n = 0; n < rounds; ++n) {
      const bool more = n + 1 < rounds;
      const int bn = more ? b : nb, kn = more ? (n + 1) * R : 0;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const double xk = x[(n * R + k) * rps + row0];
        s.x = fma(g[k].x, xk, s.x);
        s.y = fma(g[k].y, xk, s.y);
        load(bn, kn, k);
      }
    }
    if (tid < span) *reinterpret_cast<double2*>(&part[2 * tid]) = s;
    __syncthreads();
    double u = 0.0;   // column j of G_b x
#pragma unroll
    for (int k = 0; k < GR_RPS / 4; ++k) {
      if (4 * k >= rps) break;
      const double t = part[min(4 * k + q, rps - 1) * ldg + j];
      u += 4 * k + q < rps ? t : 0.0;
    }
    u = quad_sum(u);
    // x is rewritten now that every wave has passed the barrier after its last read
    // of it; part, once every wave has passed the one below
    if (p < T) {
      gr = inv * (u - c);
      c = rhs(p + 1);
      th -= lam * gr;
      if (own) {
        x[j] = th;
        a.gsave[(long)p * d + j] = gr;
      }
    } else {
      if (p == T) {
        if (a.val_loss) {
          const double v = wave_sum_f64(own ? th * (u - 2.0 * c) : 0.0);
          if ((tid & 63) == 0) red[tid >> 6] = v;
        }
        tb = invv * (u - c);   // the seed, dV/dtheta_T
      } else {
        eb = fma(-lam * gr, tb, eb);
        tb += inv * u;
      }
      if (own) x[j] = -lam * tb;
    }
    __syncthreads();
  }
  if (own) a.d_eta[j] = (float)eb;
  if (a.val_loss && tid == 0) {
    double v = a.G[((long)T * a.nr + d) * ldg + d];   // y^T y
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) v += red[k];
    *a.val_loss = (float)((v < 0.0 ? 0.0 : v) / a.vrows);
  }
}

// R: the steps of a phase, or a half or third .. of them where these are more than 13
// (4 registers each).
template <int NT, int R = 1>
hipError_t launch_sweep(const GramArgs& a, int r, hipStream_t s) {
  if constexpr (R <= 13) {
    if (r > R) return launch_sweep<NT, R + 1>(a, r, s);
    hipLaunchKernelGGL((linreg_sweep_kernel<NT, R>), dim3(1), dim3(NT), 0, s, a);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

inline long rup2(long n) { return (n + 1) / 2 * 2; }
inline int gram_rows(int d) { return (d + 1 + 15) / 16 * 16; }

}  // namespace

// G, then the inner gradients.
long linreg_gram_scratch_floats(int T, int d) {
  return 2 * ((T + 1) * (long)gram_rows(d) * rup2(d + 1) + (long)T * d);
}

hipError_t linreg_gram_meta_grad(const float* theta0, const float* eta, const float* const* xs,
                                 const float* const* ys, int T, int rows, int d, const float* vx,
                                 const float* vy, int vrows, float* d_eta, float* val_loss,
                                 float* scratch, hipStream_t s) {
  if (!linreg_fits(T, rows, vrows, d)) return hipErrorInvalidValue;
  GramArgs a = {};
  for (int t = 0; t < T; ++t) {
    a.xs[t] = xs[t];
    a.ys[t] = ys[t];
  }
  a.xs[T] = vx;
  a.ys[T] = vy;
  a.T = T; a.rows = rows; a.vrows = vrows; a.d = d;
  a.nr = gram_rows(d);
  a.ldg = (int)rup2(d + 1);
  a.G = reinterpret_cast<double*>(scratch);
  a.gsave = a.G + (long)(T + 1) * a.nr * a.ldg;
  a.theta0 = theta0; a.eta = eta; a.d_eta = d_eta; a.val_loss = val_loss;
  const int nt = a.nr / 16;
  hipLaunchKernelGGL(linreg_gram_kernel, dim3(nt * (nt + 1) / 2, T + 1), dim3(GR_THREADS), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int threads = d <= 32 ? 128 : d <= 64 ? 512 : 1024;   // at least four per column
  a.rps = std::min(threads / (a.ldg / 2), GR_RPS);
  const int steps = (d + a.rps - 1) / a.rps;
  a.rounds = (steps + 12) / 13;
  const int r = (steps + a.rounds - 1) / a.rounds;
  if (r * a.rounds * a.rps > GR_XROWS) return hipErrorInvalidValue;
  return threads == 128   ? launch_sweep<128>(a, r, s)
         : threads == 512 ? launch_sweep<512>(a, r, s)
                          : launch_sweep<1024>(a, r, s);
}

}  // namespace mfmg
