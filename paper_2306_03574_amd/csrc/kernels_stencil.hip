// Stencil and vector kernels of the ABAC MINRES path:
//   * Y T x matvec (eqs. (1.2), (1.4)) as an HBM sweep that marches over time levels
//     from both ends at once, so that <Y T z, z> pairs level k of T z with level
//     nt-1-k of z without a second read of z;
//   * the explicit residual ||f - T u|| used to confirm convergence;
//   * right-hand side assembly of eq. (1.2);
//   * solve set-up, forming the iterate from the resident basis, and the scalar steps
//     (Givens QR of the Lanczos tridiagonal matrix, stopping test) run by one block per
//     right-hand side.
#include "abac_internal.h"
#include "minres_device.h"
#include "stencil_device.h"

namespace abac {

namespace {


// One kernel per mode and coefficient kind, so each gets the registers its own path
// needs.  SPLIT: the block marches over several chunks and leaves a partial of each.  The
// others get no third wave per SIMD, which 166 registers would allow: their chunks are made
// for two (511^2 x 512: 504 us with three, as 1024 blocks then run as 768 and 256, 431 with two).
constexpr bool stencil_sums(int mode) { return mode != STENCIL_PLAIN && mode != STENCIL_T; }
template <int MODE, bool VAR, bool SPLIT>
__global__ void __launch_bounds__(kStencilThreads)
__attribute__((amdgpu_waves_per_eu(1, stencil_sums(MODE) && !VAR && !SPLIT ? 2 : 8)))
k_stencil(DevPlan P, const double* __restrict__ xin, double* __restrict__ yout, const double* __restrict__ fref) {
  const int b = blockIdx.y;
  MinresState* st = P.st + b;
  const double* x = xin;
  double* y = yout;
  if (MODE == STENCIL_MINRES) {
    if (!rhs_active(st)) return;
    const int j = st->iter + 1;
    x = P.Z[zslot(j)];
    y = P.V[(j + 1) % 3];
  } else if (MODE == STENCIL_RESIDUAL) {
    // explicit residual only when the form kernel asked for a check
    if (st->state != ST_RUNNING || !st->need_check) return;
  }
  x += (size_t)b * P.N;
  if (y) y += (size_t)b * P.N;
  const double* f = fref ? fref + (size_t)b * P.N : nullptr;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  if (MODE == STENCIL_PLAIN) {
    stencil_run<VAR, OUT_REV, false>(P, x, y, f, lb, P.st_march, threadIdx.x);
    return;
  }
  if (MODE == STENCIL_T) {
    stencil_run<VAR, OUT_NAT, false>(P, x, y, f, lb, P.st_march, threadIdx.x);
    return;
  }
  __shared__ double red[kStencilMarch][kStencilThreads / 64];
  auto emit = [&](int q, double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = v;
  };
  double acc;
  if (MODE == STENCIL_RESIDUAL && st->want_r)
    acc = stencil_run<VAR, OUT_RESREV, false, SPLIT>(P, x, P.R + (size_t)b * P.N, f, lb, P.st_march, threadIdx.x, emit);
  else if (MODE == STENCIL_MINRES)
    acc = stencil_run<VAR, OUT_REV, true, SPLIT>(P, x, y, f, lb, P.st_march, threadIdx.x, emit);
  else if (MODE == STENCIL_RESVEC)
    acc = stencil_run<VAR, OUT_RESVEC, false, SPLIT>(P, x, y, f, lb, P.st_march, threadIdx.x, emit);
  else
    acc = stencil_run<VAR, OUT_RESNORM, false, SPLIT>(P, x, y, f, lb, P.st_march, threadIdx.x, emit);
  if (!SPLIT) emit(0, acc);
  __syncthreads();
  // the partial of a chunk: its waves in order, at the chunk's place whatever the march
  const int tiles = stencil_tiles(P), q = threadIdx.x, chunk = lb / tiles * P.st_march + q;
  if (q < P.st_march && chunk * tiles < stencil_parts(P)) {
    double s = 0.0;
    for (int w = 0; w < (int)blockDim.x / 64; ++w) s += red[q][w];
    part_slot(P, MODE == STENCIL_MINRES ? PART_DELTA : PART_RES, b)[chunk * tiles + lb % tiles] = s;
  }
}

// f_1 = tau^2 src_0 / 2 + tau psi1 + psi0; f_2 = tau^2 src_1 - L psi0; f_k = tau^2 src_{k-1}
__global__ void __launch_bounds__(kVecThreads)
k_rhs(DevPlan P, const double* __restrict__ src, const double* __restrict__ psi0,
      const double* __restrict__ psi1, double* __restrict__ f) {
  const size_t total = (size_t)P.B * P.N;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const size_t b = e / P.N;
    const size_t r = e - b * P.N;
    const int k = (int)(r / P.m);
    const int i = (int)(r - (size_t)k * P.m);
    const double s = src[e];
    double v = P.tau2 * s;
    if (k == 0) {
      v = 0.5 * P.tau2 * s + P.tau * psi1[b * P.m + i] + psi0[b * P.m + i];
    } else if (k == 1) {
      v -= apply_L(l_coef(P, i % P.nx, i / P.nx), psi0 + b * P.m, i);
    }
    f[e] = v;
  }
}

// Set-up of a solve: b = Y f into V_1, zero u; ||b||^2 partials.  (v_0 is never read, and
// the w vectors are written by the flush of the resident basis before they are first
// read.)  Memory bounds it (24 bytes per element): a thread has four pairs in flight and
// steps through the levels without divisions, the blocks take turns.  With one element at a
// time 511^2 x 512 took 718 us, 64 x 127^2 x 128 630; now 647 to 657 and 551 to 565.
__global__ void __launch_bounds__(kVecThreads)
k_init(DevPlan P, const double* __restrict__ f, double* __restrict__ u) {
  const int b = blockIdx.y;
  const size_t off = (size_t)b * P.N;
  f += off;
  u += off;
  double* __restrict__ v1 = P.V[1] + off;
  const size_t m = P.m, stride = 2 * (size_t)gridDim.x * kVecThreads, dk = stride / m, di = stride - dk * m;
  size_t e = 2 * ((size_t)blockIdx.x * kVecThreads + threadIdx.x), k = e / m, i = e - k * m;
  double acc = 0.0;
  constexpr int U = 4;
  while (e < (size_t)P.N) {
    dpair v[U];
    size_t at[U];
    bool live[U];
    // element i of level k and the next one, which may open level k + 1
#pragma unroll
    for (int q = 0; q < U; ++q) {
      live[q] = e < (size_t)P.N;
      at[q] = e;
      const size_t g = live[q] ? (P.nt - 1 - k) * m + i : 0;
      v[q].x = f[g];
      v[q].y = f[!live[q] ? 0 : i + 1 < m ? g + 1 : g - i - m];
      e += stride;
      k += dk;
      i += di;
      if (i >= m) {
        i -= m;
        ++k;
      }
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (!live[q]) continue;
      *reinterpret_cast<dpair*>(v1 + at[q]) = v[q];
      *reinterpret_cast<dpair*>(u + at[q]) = dpair{0.0, 0.0};
      acc += v[q].x * v[q].x + v[q].y * v[q].y;
    }
  }
  const double bs = block_sum(acc);
  if (threadIdx.x == 0) part_slot(P, PART_RNORM, b)[blockIdx.x] = bs;
}

// Forms u (and at the flush w_j, w_{j-1}) from the resident basis for the right-hand
// sides whose scalar step (FIN_GAMMA_ITER or FIN_FINAL) set form_now; the others return at
// once.  Writes no solve state.
__global__ void __launch_bounds__(kVecThreads)
k_form(DevPlan P, double* __restrict__ u) {
  const int b = blockIdx.y;
  const MinresState* st = P.st + b;
  if (!st->form_now) return;
  const int nb = st->nbasis;
  if (st->flush_now) form_dispatch<true>(P, b, nb, u, blockIdx.x, gridDim.x);
  else form_dispatch<false>(P, b, nb, u, blockIdx.x, gridDim.x);
}

// Identity preconditioner (MINRES-I): z = q, with the Lanczos step fused in.
__global__ void __launch_bounds__(kVecThreads)
k_identity(DevPlan P, int mode, const double* __restrict__ in, double* __restrict__ out) {
  const int b = blockIdx.y;
  const size_t off = (size_t)b * P.N;
  const int nblk = gridDim.x;
  const size_t per = ((size_t)P.N + nblk - 1) / nblk;
  const size_t lo = (size_t)blockIdx.x * per;
  const size_t hi = lo + per < (size_t)P.N ? lo + per : (size_t)P.N;
  if (mode == INV_PLAIN) {
    for (size_t e = lo + threadIdx.x; e < hi; e += blockDim.x) out[off + e] = in[off + e];
    return;
  }
  const MinresState* st = P.st + b;
  if (!rhs_active(st)) return;
  double acc = 0.0;
  if (mode == INV_GAMMA_INIT) {
    const double* __restrict__ q = P.V[1] + off;
    double* __restrict__ z = P.Z[zslot(1)] + off;
    for (size_t e = lo + threadIdx.x; e < hi; e += blockDim.x) {
      const double v = q[e];
      z[e] = v;
      acc += v * v;
    }
  } else {
    const int j = st->iter + 1;
    double* __restrict__ q = P.V[(j + 1) % 3] + off;
    const double* __restrict__ vj = P.V[j % 3] + off;
    const double* __restrict__ vjm1 = P.V[j == 1 ? j % 3 : (j + 2) % 3] + off;   // v_0 has weight 0 at j = 1
    double* __restrict__ z = P.Z[zslot(j + 1)] + off;
    const double cA = st->sig, cB = st->delta * st->sig, cC = st->gamma * st->sig_prev;
    for (size_t e = lo + threadIdx.x; e < hi; e += blockDim.x) {
      const double v = cA * q[e] - cB * vj[e] - cC * vjm1[e];
      q[e] = v;
      z[e] = v;
      acc += v * v;
    }
  }
  const double bs = block_sum(acc);
  if (threadIdx.x == 0) part_slot(P, PART_GAMMA, b)[blockIdx.x] = bs;
}

__global__ void __launch_bounds__(kFinThreads)
k_fin(DevPlan P, int kind, int nparts, DotParts ndots, FinArgs a) {
  const int b = blockIdx.x;
  fin_step(P, b, kind, a, [&](Dots3* dots) {
    if (kind == FIN_GAMMA_ITER) *dots = sum_dots(P, b, ndots);
    if (kind == FIN_DELTA) return threadIdx.x < 64 ? delta_sum(P, b) : 0.0;
    return sum_parts(part_slot(P, fin_part_kind(kind), b), nparts);
  });
}

}  // namespace

int update_blocks(const DevPlan& P) {
  long long want = (P.N + (long long)kVecThreads * kVecPerThread - 1) / ((long long)kVecThreads * kVecPerThread);
  if (want > kVecMaxBlocks) want = kVecMaxBlocks;
  if (want < 1) want = 1;
  return (int)want;
}

hipError_t launch_stencil(const DevPlan& plan, int mode, const double* x, double* y, const double* f, hipStream_t s) {
  DevPlan P = plan;
  // the one-column tile marches its columns one after the other: its sums take a chunk at a time
  if (stencil_sums(mode) && (P.coef_x || P.st_cols != 2)) P.st_march = 1;
  const dim3 grid(stencil_blocks(P, P.st_march * P.st_chunk), P.B);
  const dim3 block(P.st_threads);
#define ABAC_STENCIL_CASE(M)                                                                           \
  case M:                                                                                              \
    if (P.coef_x)                                                                                      \
      hipLaunchKernelGGL((k_stencil<M, true, false>), grid, block, 0, s, P, x, y, f);                  \
    else if (stencil_sums(M) && P.st_march > 1)                                                        \
      hipLaunchKernelGGL((k_stencil<M, false, stencil_sums(M)>), grid, block, 0, s, P, x, y, f);       \
    else                                                                                               \
      hipLaunchKernelGGL((k_stencil<M, false, false>), grid, block, 0, s, P, x, y, f);                 \
    break;
  switch (mode) {
    ABAC_STENCIL_CASE(STENCIL_PLAIN)
    ABAC_STENCIL_CASE(STENCIL_MINRES)
    ABAC_STENCIL_CASE(STENCIL_RESIDUAL)
    ABAC_STENCIL_CASE(STENCIL_REPORT)
    ABAC_STENCIL_CASE(STENCIL_T)
    ABAC_STENCIL_CASE(STENCIL_RESVEC)
    default: return hipErrorInvalidValue;
  }
#undef ABAC_STENCIL_CASE
  return hipGetLastError();
}

hipError_t launch_rhs(const DevPlan& P, const double* src, const double* psi0, const double* psi1, double* f,
                      hipStream_t s) {
  long long total = (long long)P.B * P.N;
  long long blocks = (total + kVecThreads - 1) / kVecThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_rhs, dim3((unsigned)blocks), dim3(kVecThreads), 0, s, P, src, psi0, psi1, f);
  return hipGetLastError();
}

hipError_t launch_init(const DevPlan& P, const double* f, double* u, double tol, int maxit, int epoch, hipStream_t s) {
  dim3 grid(update_blocks(P), P.B);
  hipLaunchKernelGGL(k_init, grid, dim3(kVecThreads), 0, s, P, f, u);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  FinArgs a;
  a.tol = tol;
  a.maxit = maxit;
  a.epoch = epoch;
  return launch_fin(P, FIN_BNORM, a, s);
}

hipError_t launch_form(const DevPlan& P, double* u, hipStream_t s) {
  dim3 grid(update_blocks(P), P.B);
  hipLaunchKernelGGL(k_form, grid, dim3(kVecThreads), 0, s, P, u);
  return hipGetLastError();
}

hipError_t launch_identity(const DevPlan& P, int mode, const double* in, double* out, hipStream_t s) {
  dim3 grid(update_blocks(P), P.B);
  hipLaunchKernelGGL(k_identity, grid, dim3(kVecThreads), 0, s, P, mode, in, out);
  return hipGetLastError();
}

hipError_t launch_fin(const DevPlan& P, int kind, const FinArgs& a, hipStream_t s) {
  int nparts;
  switch (kind) {
    case FIN_BNORM: nparts = update_blocks(P); break;
    case FIN_GAMMA_INIT:
    case FIN_GAMMA_ITER: nparts = P.gamma_nparts; break;
    default: nparts = stencil_parts(P); break;
  }
  const DotParts ndots = kind == FIN_GAMMA_ITER && P.prec != 2 ? dot_parts(P, P.wg_x) : DotParts{0, 2};
  hipLaunchKernelGGL(k_fin, dim3(P.B), dim3(kFinThreads), 0, s, P, kind, nparts, ndots, a);
  return hipGetLastError();
}

}  // namespace abac
