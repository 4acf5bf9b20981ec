// Linear regression through its normal equations (gfx950).
//
// With a squared loss the inner gradient of batch b is (2/N) (G_b theta - c_b),
// G_b = X_b^T X_b and c_b = X_b^T y_b, and its Hessian-vector product is
// (2/N) G_b v (Section 2.2).  Neither G_b nor c_b depends on theta, so all of
// them are formed at once over the whole chip (linreg_gram_kernel); what is left
// of the sweep is one d x d matrix-vector product per phase, in one workgroup
// (linreg_sweep_kernel).  Walking the batches themselves, 2 T + 1 of them, one
// compute unit receives about 20 bytes a cycle: 130 features, 1000 rows, T = 3
// took 620 us that way.  The validation loss is formed from its residuals (as a
// quadratic form it would cancel near a fit).
#include <algorithm>

#include "kernels.h"

namespace mfmg {

namespace {

constexpr int GR_MAXD = 256;
constexpr int GR_MAXR = 1024;
constexpr int GR_MAXT = 64;
constexpr int GR_THREADS = 1024;
constexpr int GR_WAVES = GR_THREADS / 64;
constexpr int GR_SAVE = 8192;         // floats of inner gradients kept in LDS (T d)

struct GramArgs {
  const float* xs[GR_MAXT + 1];   // the T training batches, then the validation batch
  const float* ys[GR_MAXT + 1];
  int T, rows, vrows, d;
  int n, nr, ldg;                 // n = d + 1 columns [X | y]; rows (zero past n) and row
                                  // pitch of G
  float* G;                       // [T + 1][nr][ldg]
  const float* theta0;
  const float* eta;
  float* gsave;                   // [T][d] inner gradients, when they do not fit LDS
  float* thetaT;                  // [d], for linreg_val_kernel
  float* vpart;                   // its partial sums
  unsigned* ticket;
  float* d_eta;
  float* val_loss;
};

// [X | y]^T [X | y] of every batch: one workgroup per 32 x 32 output tile on or
// above the diagonal, whose 16 waves take every 16th group of four rows; the
// v_mfma_f32_16x16x4_f32 operands are read straight from the rows (lane: column
// lane % 16 of row lane / 16, 64-byte runs), so no LDS staging is needed.  The
// waves' sums are added in wave order in float64 and rounded once.
__global__ void __launch_bounds__(GR_THREADS) linreg_gram_kernel(GramArgs a) {
  __shared__ float part[GR_WAVES][32 * 33];
  const int b = blockIdx.y;
  const int nt = a.nr / 32;
  int p = blockIdx.x, ti = 0;
  while (p >= nt - ti) {
    p -= nt - ti;
    ++ti;
  }
  const int tj = ti + p;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (blockIdx.x == 0 && b == 0 && tid == 0) *a.ticket = 0u;
  const float* X = a.xs[b];
  const float* y = a.ys[b];
  const int rows = b < a.T ? a.rows : a.vrows;
  // four columns per lane: two of the tile's rows, two of its columns
  const float* base[4];
  unsigned stride[4];
  bool in[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = (q < 2 ? ti : tj) * 32 + (q & 1) * 16 + (lane & 15);
    base[q] = c < a.d ? X + c : y;
    stride[q] = c < a.d ? a.d : 1;
    in[q] = c <= a.d;
  }
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int UN = 4;   // steps whose loads are in flight together
  const int steps = (rows + 4 * GR_WAVES - 1) / (4 * GR_WAVES);
  for (int s0 = 0; s0 < steps; s0 += UN) {
    float v[UN][4];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int r = (s0 + u) * 4 * GR_WAVES + 4 * w + (lane >> 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[u][q] = base[q][(unsigned)min(r, rows - 1) * stride[q]];
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int r = (s0 + u) * 4 * GR_WAVES + 4 * w + (lane >> 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[u][q] = in[q] && r < rows ? v[u][q] : 0.0f;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[u][i], v[u][2 + j], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        part[w][(i * 16 + (lane >> 4) * 4 + r) * 33 + j * 16 + (lane & 15)] = acc[i][j][r];
  __syncthreads();
  float* G = a.G + (long)b * a.nr * a.ldg;
  {
    const int r = tid >> 5, c = tid & 31;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < GR_WAVES; ++k) s += (double)part[k][r * 33 + c];
    const float g = (float)s;
    const int gr = ti * 32 + r, gc = tj * 32 + c;
    if (gc < a.ldg) G[(long)gr * a.ldg + gc] = g;
    if (ti != tj) part[0][r * 33 + c] = g;   // each thread rewrites the entry only it read
  }
  if (ti == tj) return;
  __syncthreads();
  const int r = tid >> 5, c = tid & 31;   // the mirrored tile
  const int gr = tj * 32 + r, gc = ti * 32 + c;
  if (gc < a.ldg) G[(long)gr * a.ldg + gc] = part[0][c * 33 + r];
}

__device__ __forceinline__ float quad_sum(float v) {   // over the four lanes of a quad
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true));
  return v;
}

// The sweep: T inner steps, the seed at theta_T, T reverse steps, on W waves.  A
// row of G takes LPR lanes of 16 bytes, so the workgroup reads W * 64 / LPR rows
// per step and all d in NS steps, each thread holding its NS pieces in registers;
// the next phase's pieces are requested as soon as this phase's are used.  The
// column sums go over the row slots of a wave, then over the W waves through LDS
// (four lanes per column), in a fixed order.
template <int W, int LPR, int NS, bool SAVE_LDS>
__global__ void __launch_bounds__(W * 64) linreg_sweep_kernel(GramArgs a) {
  constexpr int RPW = 64 / LPR;            // rows per wave and step
  constexpr int RPS = W * RPW;
  __shared__ float x[NS * RPS];            // the vector of this phase, zero past d
  __shared__ __attribute__((aligned(16))) float part[W][LPR * 4];
  __shared__ float gs[SAVE_LDS ? GR_SAVE : 1];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int d = a.d, T = a.T;
  const int row0 = w * RPW + lane / LPR, cg = (lane % LPR) * 4;
  float4 g[NS];
  const unsigned off = (unsigned)(row0 * a.ldg + min(cg, a.ldg - 4)) * 4u;
  auto load = [&](int b) {   // NS * RPS <= a.nr
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const float* G = a.G + ((long)b * a.nr + s * RPS) * a.ldg;
      g[s] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(G) + off);
    }
  };
  // W * 16 columns at a time: thread 4 j + q works on column j
  static_assert(W * 16 >= LPR * 4 || W * 32 >= LPR * 4, "one or two columns per thread");
  constexpr int NC = W * 16 >= LPR * 4 ? 1 : 2;
  const int q = tid & 3;
  int j[NC];
  bool own[NC];
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    const int col = (tid >> 2) + n * W * 16;
    j[n] = min(col, d - 1);
    own[n] = col < d && q == 0;
  }
  load(0);
  float c[NC], th[NC], tb[NC], eb[NC], lam[NC], u[NC];
  auto rhs = [&](int b) {   // c_b
#pragma unroll
    for (int n = 0; n < NC; ++n) c[n] = a.G[((long)b * a.nr + d) * a.ldg + j[n]];
  };
  rhs(0);
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    th[n] = a.theta0[j[n]];
    lam[n] = a.eta[j[n]];
    eb[n] = 0.0f;
  }
  for (int i = tid; i < NS * RPS; i += W * 64) x[i] = 0.0f;
  __syncthreads();
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    lam[n] = expf(lam[n]);
    if (own[n]) x[j[n]] = th[n];
  }
  __syncthreads();
  // u = G_b x; requests G of batch nb meanwhile
  auto matvec = [&](int nb) {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const float xk = x[k * RPS + row0];
      s.x = fmaf(g[k].x, xk, s.x);
      s.y = fmaf(g[k].y, xk, s.y);
      s.z = fmaf(g[k].z, xk, s.z);
      s.w = fmaf(g[k].w, xk, s.w);
    }
    // from NS = 28 on, loads moved up between the products would not fit the registers
    if (NS >= 28) __builtin_amdgcn_sched_barrier(0);
    if (nb >= 0) load(nb);
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      s.x += __shfl_xor(s.x, o, 64);
      s.y += __shfl_xor(s.y, o, 64);
      s.z += __shfl_xor(s.z, o, 64);
      s.w += __shfl_xor(s.w, o, 64);
    }
    if (lane < LPR) *reinterpret_cast<float4*>(&part[w][cg]) = s;
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      float t = 0.0f;
#pragma unroll
      for (int k = 0; k < W / 4; ++k) t += part[q * (W / 4) + k][j[n]];
      u[n] = quad_sum(t);
    }
  };
  const float inv = 2.0f / (float)a.rows, invv = 2.0f / (float)a.vrows;
  for (int t = 0; t < T; ++t) {
    matvec(t + 1);
    float gr[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) gr[n] = inv * (u[n] - c[n]);
    rhs(t + 1);
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      th[n] -= lam[n] * gr[n];
      if (own[n]) {
        x[j[n]] = th[n];
        if (SAVE_LDS) gs[t * d + j[n]] = gr[n];
        else a.gsave[(long)t * d + j[n]] = gr[n];
      }
    }
    __syncthreads();
  }
  if (a.val_loss) {   // for linreg_val_kernel
#pragma unroll
    for (int n = 0; n < NC; ++n)
      if (own[n]) a.thetaT[j[n]] = th[n];
  }
  // Seed: bar theta_T = dV/dtheta_T.  x is rewritten once every wave has passed the
  // barrier after its last read of it.
  matvec(T - 1);
#pragma unroll
  for (int n = 0; n < NC; ++n) {
    tb[n] = invv * (u[n] - c[n]);
    if (own[n]) x[j[n]] = -lam[n] * tb[n];
  }
  __syncthreads();
  for (int i = T - 1; i >= 0; --i) {
    float gr[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) {   // by the lane that saved it
      gr[n] = 0.0f;
      if (own[n]) gr[n] = SAVE_LDS ? gs[i * d + j[n]] : a.gsave[(long)i * d + j[n]];
    }
    matvec(i - 1);
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      eb[n] = fmaf(-lam[n] * gr[n], tb[n], eb[n]);
      tb[n] += inv * u[n];
      if (own[n]) x[j[n]] = -lam[n] * tb[n];
    }
    __syncthreads();
  }
#pragma unroll
  for (int n = 0; n < NC; ++n)
    if (own[n]) a.d_eta[j[n]] = eb[n];
}

// The validation loss: one wave per row, the workgroups' sums added in order by the
// last one to finish.  A launch of its own also for small batches: held in the
// sweep's registers from its start the batch made the sweep longer by more (64 x
// 256: 22 us against 14 and 8), its unrolled code running once.
__global__ void __launch_bounds__(256) linreg_val_kernel(GramArgs a) {
  __shared__ float x[GR_MAXD];
  __shared__ float red[4];
  __shared__ bool last;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float* X = a.xs[a.T];
  const float* y = a.ys[a.T];
  if (tid < a.d) x[tid] = a.thetaT[tid];
  __syncthreads();
  float ls = 0.0f;
  for (int r = blockIdx.x * 4 + w; r < a.vrows; r += gridDim.x * 4) {
    constexpr int NV = GR_MAXD / 64;
    float xr[NV], s = 0.0f;
    const float t = y[r];
#pragma unroll
    for (int n = 0; n < NV; ++n) xr[n] = X[(long)r * a.d + min(lane + 64 * n, a.d - 1)];
#pragma unroll
    for (int n = 0; n < NV; ++n)
      if (lane + 64 * n < a.d) s = fmaf(xr[n], x[lane + 64 * n], s);
    const float e = wave_sum(s) - t;
    ls = fmaf(e, e, ls);
  }
  if (lane == 0) red[w] = ls;
  __syncthreads();
  if (tid == 0) {
    __hip_atomic_store(a.vpart + blockIdx.x, (red[0] + red[1]) + (red[2] + red[3]),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence();
    last = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
           gridDim.x - 1;
  }
  __syncthreads();
  if (!last || w != 0) return;
  __threadfence();
  float s = 0.0f;
  for (int k = lane; k < (int)gridDim.x; k += 64)
    s += __hip_atomic_load(a.vpart + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  s = wave_sum(s);
  if (lane == 0) *a.val_loss = s / (float)a.vrows;
}

constexpr int GR_VAL_BLOCKS = 256;

template <int W, int LPR, int NS>
void launch_sweep(const GramArgs& a, hipStream_t s) {
  if ((long)a.T * a.d <= GR_SAVE)
    hipLaunchKernelGGL((linreg_sweep_kernel<W, LPR, NS, true>), dim3(1), dim3(W * 64), 0, s, a);
  else
    hipLaunchKernelGGL((linreg_sweep_kernel<W, LPR, NS, false>), dim3(1), dim3(W * 64), 0, s, a);
}

inline long rup4(long n) { return (n + 3) / 4 * 4; }
// Rows of G: d + 1 in whole 32-row tiles, and at least the 64 of the sweep's
// smallest step, so that the sweep reads zeros and not past the end.
inline int gram_rows(int d) { return std::max(64, (d + 1 + 31) / 32 * 32); }

}  // namespace

static bool gram_fits(int T, int rows, int vrows, int d) {
  return T >= 1 && T <= GR_MAXT && d >= 1 && d <= GR_MAXD && rows >= 1 && rows <= GR_MAXR &&
         vrows >= 1 && vrows <= GR_MAXR;
}

long linreg_scratch_floats(int T, int d) {   // covers the (T + 1) d of the other forms
  return (T + 1) * (long)gram_rows(d) * rup4(d + 1) + rup4((long)T * d) + rup4(d) + GR_VAL_BLOCKS + 4;
}

hipError_t linreg_gram_meta_grad(const float* theta0, const float* eta, const float* const* xs,
                                 const float* const* ys, int T, int rows, int d, const float* vx,
                                 const float* vy, int vrows, float* d_eta, float* val_loss,
                                 float* scratch, hipStream_t s) {
  if (!gram_fits(T, rows, vrows, d)) return hipErrorInvalidValue;
  GramArgs a = {};
  for (int t = 0; t < T; ++t) {
    a.xs[t] = xs[t];
    a.ys[t] = ys[t];
  }
  a.xs[T] = vx;
  a.ys[T] = vy;
  a.T = T; a.rows = rows; a.vrows = vrows; a.d = d;
  a.n = d + 1;
  a.nr = gram_rows(d);
  a.ldg = (int)rup4(a.n);
  a.G = scratch;
  a.gsave = a.G + (long)(T + 1) * a.nr * a.ldg;
  a.thetaT = a.gsave + rup4((long)T * d);
  a.vpart = a.thetaT + rup4(d);
  a.theta0 = theta0; a.eta = eta; a.d_eta = d_eta; a.val_loss = val_loss;
  a.ticket = reinterpret_cast<unsigned*>(a.vpart + GR_VAL_BLOCKS);
  const int nt = a.nr / 32;
  hipLaunchKernelGGL(linreg_gram_kernel, dim3(nt * (nt + 1) / 2, T + 1), dim3(GR_THREADS), 0, s, a);
  // waves, lanes per row of G, steps over its rows (steps x waves x 64 / lanes <=
  // gram_rows)
  if (d <= 64) launch_sweep<4, 16, 4>(a, s);
  else if (d <= 96) launch_sweep<16, 32, 3>(a, s);
  else if (d <= 128) launch_sweep<16, 32, 4>(a, s);
  else if (d <= 160) launch_sweep<8, 64, 20>(a, s);
  else if (d <= 192) launch_sweep<8, 64, 24>(a, s);
  else if (d <= 224) launch_sweep<8, 64, 28>(a, s);
  else launch_sweep<8, 64, 32>(a, s);
  if (val_loss)
    hipLaunchKernelGGL(linreg_val_kernel, dim3(std::min((vrows + 3) / 4, GR_VAL_BLOCKS)),
                       dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace mfmg
