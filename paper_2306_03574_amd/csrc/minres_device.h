// Device code of the MINRES steps (Section 3's solver; Paige-Saunders recurrences in
// the P^{-1} inner product): forming the iterate from the resident Krylov basis, and the
// per-right-hand-side scalar steps (sums of partials, Givens QR, bounds on the residual
// norm, stopping test, snapshots).  Shared by the separate kernels and the fused
// small-problem iteration.
#pragma once
#include "abac_internal.h"

namespace abac {
namespace {

constexpr int kFormTrips = kVecPerThread / 2;
constexpr int kFinThreads = 1024;   // threads of a scalar step

// u = [u +] sum_l xm_l z_l over the NB vectors of the current cycle, plus the two carried
// w vectors of a later cycle; with FLUSH also W[0] = w_j and W[1] = w_{j-1} from their
// coefficients.  The nparts blocks of right-hand side b take turns
// of kFormTrips trips: 32 KB of each vector in a row per block, and the chip sweeps all of
// them front to back.  Memory bounds it.  Against one range per block (1 MB at 511^2 x 512):
// 2400 -> 2285 us there (10 iterations, 5.1 TB/s), 238 -> 202 us at 255^2 x 256; turns of
// 4 KB 1866 us at 64 x 127^2 x 128, where a range is one turn and takes 1790 to 1810 us.
template <int NB, bool FLUSH>
__device__ __forceinline__ void form_from_basis(const DevPlan& P, int b, double* __restrict__ u, int part,
                                                int nparts) {
  const size_t off = (size_t)b * P.N;
  const MinresState* st = P.st + b;
  const double* kc = minres_ext(P, b)->kc;
  const int base = st->cbase;
  const bool add = st->u_valid != 0, carry = base != 0;
  double cx[NB], c1[NB], c2[NB];
  const double* zs[NB];
#pragma unroll
  for (int l = 0; l < NB; ++l) {
    cx[l] = kc[l];
    c1[l] = FLUSH ? kc[kCoefs + l] : 0.0;
    c2[l] = FLUSH ? kc[2 * kCoefs + l] : 0.0;
    zs[l] = P.Z[zslot(base + l + 1)] + off;
  }
  double* X = u + off;
  double* W1 = P.W[0] + off;
  double* W2 = P.W[1] + off;
  // a pair of elements per trip (N is even, since nt is): NB 16-byte loads in flight, past
  // the caches at every size (each z is read once, and after all else of the iteration: 1 us
  // slower or less where a vector takes 2 to 16 MB, 51.5 -> 46.1 us at 255 x 127 x 128, 105 -> 85
  // at 255^2 x 128)
  const auto pair = [](const double* p) { return stream_load<true>(reinterpret_cast<const dpair*>(p)); };
  const auto store = [](double* p, dpair v) { *reinterpret_cast<dpair*>(p) = v; };
  const size_t step = 2 * (size_t)blockDim.x, chunk = kFormTrips * step;
  size_t e = part * chunk + 2 * threadIdx.x;
  for (int trip = 1; e < (size_t)P.N; e += trip % kFormTrips ? step : step + (nparts - 1) * chunk, ++trip) {
    dpair z[NB];
#pragma unroll
    for (int l = 0; l < NB; ++l) z[l] = pair(zs[l] + e);
    dpair ax{0.0, 0.0}, a1{0.0, 0.0}, a2{0.0, 0.0};
    if (add) ax = *reinterpret_cast<const dpair*>(X + e);
    if (carry) {
      const dpair p = *reinterpret_cast<const dpair*>(W1 + e), q = *reinterpret_cast<const dpair*>(W2 + e);
      ax += kc[kBasis] * p + kc[kBasis + 1] * q;
      if (FLUSH) {
        a1 = kc[kCoefs + kBasis] * p + kc[kCoefs + kBasis + 1] * q;
        a2 = kc[2 * kCoefs + kBasis] * p + kc[2 * kCoefs + kBasis + 1] * q;
      }
    }
#pragma unroll
    for (int l = 0; l < NB; ++l) {
      ax += cx[l] * z[l];
      if (FLUSH) {
        a1 += c1[l] * z[l];
        a2 += c2[l] * z[l];
      }
    }
    store(X + e, ax);
    if (FLUSH) {
      store(W1 + e, a1);
      store(W2 + e, a2);
    }
  }
}

template <bool FLUSH>
__device__ __forceinline__ void form_dispatch(const DevPlan& P, int b, int nb, double* u, int part, int nparts) {
  if constexpr (FLUSH) {
    form_from_basis<kBasis, true>(P, b, u, part, nparts);   // a flush ends a full cycle
  } else {
    switch (nb) {
#define ABAC_FORM_CASE(K) \
    case K: form_from_basis<K, false>(P, b, u, part, nparts); break;
      ABAC_FORM_CASE(1) ABAC_FORM_CASE(2) ABAC_FORM_CASE(3) ABAC_FORM_CASE(4) ABAC_FORM_CASE(5) ABAC_FORM_CASE(6)
      ABAC_FORM_CASE(7) ABAC_FORM_CASE(8) ABAC_FORM_CASE(9) ABAC_FORM_CASE(10) ABAC_FORM_CASE(11) ABAC_FORM_CASE(12)
#undef ABAC_FORM_CASE
      default: break;
    }
  }
}
static_assert(kBasis == 12, "form_dispatch lists one case per basis size");

// The coefficients after a form step wrote the iterate to u: x adds to u from zero again,
// and after a flush the next cycle's w recurrences start from the two w vectors.
__device__ __forceinline__ void form_done(MinresState* st, MinresExt* x) {
  double* xm = x->kc;
  double* m1 = x->kc + kCoefs;
  double* m2 = x->kc + 2 * kCoefs;
  for (int l = 0; l < kCoefs; ++l) xm[l] = 0.0;
  if (st->flush_now) {
    for (int l = 0; l < kCoefs; ++l) m1[l] = m2[l] = 0.0;
    m1[kBasis] = 1.0;
    m2[kBasis + 1] = 1.0;
    st->cbase += st->nbasis;
    st->nbasis = 0;
  }
  st->u_valid = 1;
  st->basis_dirty = 0;
  st->form_now = 0;
  st->flush_now = 0;
}

// Bounds on ||r_j|| after the Givens step of iteration j (st->iter), from the inner
// products of the first transform pass (see MinresExt); returns the estimate of
// ||r_j||^2.  The unrolled sums carry a relative rounding slack of 1e-13 of their terms; the
// tracked vector's norm is compared as it is, as an explicit one would be.
__device__ __forceinline__ double residual_bounds(MinresState* st, MinresExt* x, const Dots3& d, bool identity,
                                                  double* lo, double* hi) {
  const double r1 = st->r1, r2 = st->r2;
  double est2, tail = 0.0, slack = 0.0;
  if (identity) {
    est2 = st->eta * st->eta;   // P = I: ||r_j|| = |eta_j|
  } else if (st->track) {
    est2 = r1 * r1 * d.c + 2.0 * r1 * r2 * d.b + r2 * r2 * d.a;
  } else {
    const double ra = r1 * x->rb, rb = r1 * x->rc, rc = r2;
    const double ta = ra * ra * x->n0, tb = rb * rb * x->n1, tc = rc * rc * d.a;
    est2 = ta + tb + tc + 2.0 * (ra * rb * x->d01 + rb * rc * d.b + ra * rc * d.c);
    slack = 1e-13 * (ta + tb + tc);
    if (st->iter >= 3) tail = r1 * x->r1p[0] * x->r1p[1] * x->hi[2];
    x->rb = rb;
    x->rc = rc;
    x->n0 = x->n1;
    x->n1 = d.a;
    x->d01 = d.b;
  }
  x->r1p[1] = x->r1p[0];
  x->r1p[0] = r1;
  *lo = sqrt(fmax(est2 - slack, 0.0)) - tail;
  *hi = sqrt(fmax(est2 + slack, 0.0)) + tail;
  if (!(est2 == est2)) *lo = *hi = est2;   // NaN: no bound
  x->hi[2] = x->hi[1];
  x->hi[1] = x->hi[0];
  x->hi[0] = *hi;
  return est2;
}

// Lanczos coefficient gamma_{j+1}, the Givens QR update of iteration j, and the stopping
// test on the bounds of ||r_j||: an explicit check where they do not exclude
// convergence.  The step of the w and x recurrences is left to step_coefs.
__device__ void step_gamma_iter(MinresState* st, MinresExt* x, double g2, const Dots3& dots, bool identity) {
  const double gn = sqrt(g2);
  const double gam = st->gamma, del = st->delta;
  const double eps = st->s2 * gam;
  const double dbar = st->c2 * gam;
  const double dp = st->c1 * dbar + st->s1 * del;
  const double t2 = -st->s1 * dbar + st->c1 * del;
  const double rho = hypot(t2, gn);
  if (!(g2 >= 0.0) || !(g2 < 1e300) || !(rho > 0.0) || !(rho < 1e300)) {
    st->state = ST_DONE;
    st->status = -5;  // ABAC_EBREAKDOWN
    st->iter += 1;
    st->need_check = 0;
    st->form_now = st->basis_dirty;   // u gets the last iterate
    st->flush_now = 0;
    st->hold = st->form_now;
    x->step = 0.0;
    return;
  }
  const double c = t2 / rho, s = gn / rho;
  x->wa = st->sig / rho;
  x->wb = dp / rho;
  x->wc = eps / rho;
  x->xc = c * st->eta;
  x->step = 1.0;
  st->r1 = s * s;
  st->r2 = gn > 0.0 ? -s * c * st->eta / gn : 0.0;
  st->eta = -s * st->eta;
  st->c2 = st->c1; st->c1 = c;
  st->s2 = st->s1; st->s1 = s;
  st->sig_prev = st->sig;
  st->sig = gn > 0.0 ? 1.0 / gn : 0.0;
  st->gamma = gn;
  st->iter += 1;
  if (gn == 0.0) st->lucky = 1;
  const int j = st->iter;
  st->nbasis += 1;
  st->basis_dirty = 1;
  double lo, hi;
  st->rnorm2 = residual_bounds(st, x, dots, identity, &lo, &hi);
  const double thr = sqrt(st->tol2 * st->bnorm2);
  const int need = !(lo > thr) || st->explicit_mode || j >= st->maxit || st->lucky;
  st->need_check = need;
  // bounds too wide to decide (slow convergence): keep the residual vector from here on
  st->want_r = need && !identity && !st->track && !st->explicit_mode && hi > thr && !(hi < 1.25 * lo);
  st->flush_now = st->nbasis == kBasis;
  st->form_now = need || st->flush_now;
  st->hold = st->tail = st->form_now;
}

// The w and x recurrences of the last Givens step on the coefficient vectors over the basis
// (kc: x, w_j, w_{j-1}), a coefficient per thread (behind a barrier).
__device__ __forceinline__ void step_coefs(const MinresState* st, MinresExt* x) {
  const int l = threadIdx.x;
  if (l >= kCoefs || x->step == 0.0) return;
  double* xm = x->kc + l;
  double* m1 = xm + kCoefs;
  double* m2 = m1 + kCoefs;
  const double w = (l == st->nbasis - 1 ? x->wa : 0.0) - x->wb * *m1 - x->wc * *m2;
  *m2 = *m1;
  *m1 = w;
  *xm += x->xc * w;
}

__device__ __forceinline__ void post_snapshot(const DevPlan& P, int b, MinresState* st) {
  const int seq = st->snap;
  st->snap = seq + 1;
  write_snapshot(P, b, seq, snap_word(st->epoch, seq, st->state, st->hold), st->state != ST_RUNNING, st->status, st->iter,
                 st->rnorm2, st->bnorm2, st->res2, st->tol2);
}

// First half of a scalar step of right-hand side b: the flag updates of the step kind
// (by thread 0 of the calling workgroup) and whether the step folds a sum into the
// state.  A skipped step that posts a snapshot still does.  Every thread returns the same
// answer.
__device__ __forceinline__ bool fin_posts(int kind, const FinArgs& a) {
  return a.post >= 0 && (kind == FIN_GAMMA_INIT || kind == FIN_RES || (kind == FIN_GAMMA_ITER && a.post));
}

__device__ __forceinline__ bool fin_begin(const DevPlan& P, int b, MinresState* st, MinresExt* x, int kind,
                                          const FinArgs& a) {
  const bool posts = fin_posts(kind, a);
  if (kind == FIN_RES || kind == FIN_REPORT) {
    if (threadIdx.x == 0) {
      if (st->form_now) form_done(st, x);
      st->hold = 0;
    }
  } else if ((kind == FIN_DELTA || kind == FIN_GAMMA_ITER) && st->hold) {
    if (posts && threadIdx.x == 0) post_snapshot(P, b, st);
    return false;
  }
  if (kind == FIN_FINAL) {
    // the end of a solve with a stale u forms it from the basis
    if (threadIdx.x == 0) {
      st->form_now = st->basis_dirty;
      st->flush_now = 0;
    }
    return false;
  }
  if ((kind != FIN_BNORM && kind != FIN_REPORT && st->state != ST_RUNNING) || (kind == FIN_RES && !st->need_check)) {
    if (posts && threadIdx.x == 0) post_snapshot(P, b, st);
    return false;
  }
  return true;
}

// Which partial sums a scalar step folds in.
__device__ __forceinline__ int fin_part_kind(int kind) {
  switch (kind) {
    case FIN_BNORM: return PART_RNORM;
    case FIN_DELTA: return PART_DELTA;
    case FIN_GAMMA_INIT:
    case FIN_GAMMA_ITER: return PART_GAMMA;
    default: return PART_RES;
  }
}

// Sums of the partials of the first transform pass's inner products; valid in thread 0.  In the
// order of kFinThreads threads, whatever the block has (a divisor of them, whole waves), so
// that every kernel's scalar step gets the same bits.
__device__ __forceinline__ Dots3 sum_dots(const DevPlan& P, int b, DotParts parts) {
  __shared__ double red[kFinThreads / 64][3];
  const double* const part[3] = {dot_slot(P, 0, b), dot_slot(P, 1, b), dot_slot(P, 2, b)};
  auto sum = [&](auto pairs) {
    for (int t = threadIdx.x; t < kFinThreads; t += blockDim.x)
      dots_reduce(group_share<decltype(pairs)::value>(part, parts.n, parts.group / 8, t, kFinThreads), red[t >> 6]);
  };
  if (parts.group >= 8) sum(std::integral_constant<int, 4>{});
  else if (parts.group == 4) sum(std::integral_constant<int, 2>{});
  else sum(std::integral_constant<int, 1>{});
  __syncthreads();
  Dots3 t{0.0, 0.0, 0.0};
  if (threadIdx.x == 0) {
    for (int w = 0; w < kFinThreads / 64; ++w) {
      t.a += red[w][0];
      t.b += red[w][1];
      t.c += red[w][2];
    }
  }
  __syncthreads();
  return t;
}

// Second half, thread 0 only: fold the sum `tot` (and for FIN_GAMMA_ITER the inner
// products of the first transform pass) into the state of right-hand side b (Givens QR,
// stopping test, ...) and post the snapshot at the end of an iteration.
__device__ __forceinline__ void fin_scalar(const DevPlan& P, int b, MinresState* st, MinresExt* x, int kind, double tot,
                                           const Dots3& dots, const FinArgs& a) {
  switch (kind) {
    case FIN_BNORM:
      st->bnorm2 = tot;
      st->tol2 = a.tol * a.tol;
      st->maxit = a.maxit;
      st->epoch = a.epoch;
      st->hold = 0;
      st->tail = 0;
      st->iter = 0;
      st->explicit_mode = 0;
      st->need_check = 0;
      st->lucky = 0;
      st->snap = 0;
      st->cbase = 0;
      st->nbasis = 0;
      st->u_valid = 0;
      st->track = 0;
      st->want_r = 0;
      st->basis_dirty = 0;   // u = 0 = x_0
      st->form_now = 0;
      st->flush_now = 0;
      st->rnorm2 = tot;
      st->res2 = tot;
      st->status = 0;
      if (tot == 0.0) {
        st->state = ST_DONE;   // u = 0 is exact
      } else if (!(tot == tot) || tot > 1e300) {
        st->state = ST_DONE;
        st->status = -5;
      } else {
        st->state = ST_RUNNING;
      }
      break;
    case FIN_DELTA:
      st->delta = tot * st->sig * st->sig;
      break;
    case FIN_GAMMA_INIT:
      if (!(tot > 0.0) || !(tot < 1e300)) {
        st->state = ST_DONE;
        st->status = -5;
        break;
      }
      st->gamma = sqrt(tot);
      st->sig = 1.0 / st->gamma;
      st->sig_prev = 0.0;
      st->eta = st->gamma;
      st->c1 = 1.0; st->c2 = 1.0;
      st->s1 = 0.0; st->s2 = 0.0;
      st->iter = 0;
      for (int l = 0; l < 3 * kCoefs; ++l) x->kc[l] = 0.0;
      x->rb = 0.0;   // r_0 = V_1
      x->rc = 1.0;
      x->n0 = 0.0;
      x->n1 = st->bnorm2;
      x->d01 = 0.0;
      x->r1p[0] = x->r1p[1] = 0.0;
      x->hi[0] = x->hi[1] = x->hi[2] = sqrt(st->bnorm2);
      break;
    case FIN_GAMMA_ITER:
      step_gamma_iter(st, x, tot, dots, P.prec == 2);
      break;
    case FIN_RES:
      st->res2 = tot;
      if (tot <= st->tol2 * st->bnorm2) {
        st->state = ST_DONE;
        st->status = 0;
      } else if (!(tot == tot) || tot > 1e300) {
        st->state = ST_DONE;
        st->status = -5;
      } else if (st->iter >= st->maxit) {
        st->state = ST_DONE;
        st->status = -4;  // ABAC_ENOTCONV
      } else if (st->want_r) {
        // undecided and not converged: P.R now holds r_j, so the next first pass must not
        // add the recurrence's last step again
        st->track = 1;
        st->r1 = 1.0;
        st->r2 = 0.0;
      } else {
        if (!(x->hi[0] * x->hi[0] > st->tol2 * st->bnorm2)) st->explicit_mode = 1;   // the recurrence was optimistic
        x->hi[0] = sqrt(tot);
      }
      st->need_check = 0;
      st->want_r = 0;
      break;
    case FIN_REPORT:
      st->res2 = tot;
      break;
  }
  if (fin_posts(kind, a)) post_snapshot(P, b, st);
}

// The scalar state of a right-hand side, in LDS for the length of a scalar step: the step
// is a chain of dependent reads and writes of it, which costs a trip to L2 each in global
// memory (63^2 x 64: 10.6 -> 8.3 us per Givens step).
struct ScalarState {
  MinresState st;
  MinresExt x;
};
template <bool IN>
__device__ __forceinline__ void move_state(const DevPlan& P, int b, ScalarState& s) {
  static_assert(sizeof(MinresState) % 8 == 0 && sizeof(MinresExt) % 8 == 0, "moved in doubles");
  constexpr int n1 = sizeof(MinresState) / 8, n2 = sizeof(MinresExt) / 8;
  double *g1 = reinterpret_cast<double*>(P.st + b), *g2 = reinterpret_cast<double*>(minres_ext(P, b));
  double *l1 = reinterpret_cast<double*>(&s.st), *l2 = reinterpret_cast<double*>(&s.x);
  for (int i = threadIdx.x; i < n1 + n2; i += blockDim.x) {
    double* g = i < n1 ? g1 + i : g2 + (i - n1);
    double* l = i < n1 ? l1 + i : l2 + (i - n1);
    if (IN) *l = *g;
    else *g = *l;
  }
}

// A scalar step of right-hand side b by the calling workgroup; `sums` gives the step's sum
// of partials and, for FIN_GAMMA_ITER, the inner products (both valid in thread 0).
template <typename Sums>
__device__ __forceinline__ void fin_step(const DevPlan& P, int b, int kind, const FinArgs& a, Sums&& sums) {
  __shared__ ScalarState s;
  move_state<true>(P, b, s);
  __syncthreads();
  const bool go = fin_begin(P, b, &s.st, &s.x, kind, a);
  if (go) {
    Dots3 dots{0.0, 0.0, 0.0};
    const double tot = sums(&dots);
    if (threadIdx.x == 0) fin_scalar(P, b, &s.st, &s.x, kind, tot, dots, a);
  }
  __syncthreads();
  if (go && kind == FIN_GAMMA_ITER) {
    step_coefs(&s.st, &s.x);
    __syncthreads();
  }
  move_state<false>(P, b, s);
}

}  // namespace
}  // namespace abac
