// Fused MINRES set-up, iteration and whole solve for small 1D problems (N = nt * nx <= 4096
// unknowns).
//
// At these sizes an iteration of the separate kernels is bound by the latency of its
// launches and of their global accesses, not by memory.  Here one workgroup per right-hand
// side runs the whole iteration, and what one step hands to the next stays in LDS: z_j
// (read by the matvec), the transform scratch (read by the next pass in another order) and
// the scalar state.  Every thread owns the elements tid + 512 i of a vector, so the
// elementwise steps (matvec, Lanczos step, forming the iterate) pass their values on in
// registers; the Lanczos vectors and the basis go to global memory for later iterations,
// written by the thread that reads them back.  The spectral weights of a thread's mode pair
// are computed once per launch.  63 x 64 FP64, 6 iterations: 294 us per solve when the
// steps went through global memory tile by tile, 159 us now.
//
// The transforms are the separate kernels' (fft_seq, time_core, the same staging and
// scaling), the scalar steps are theirs (minres_device.h), in the same order and under the
// same conditions; the order of the partial sums does not depend on the batch.
#include "../../include/abac.h"
#include "abac_internal.h"
#include "minres_device.h"
#include "stencil_device.h"
#include "transform_device.h"

namespace abac {

namespace {

constexpr int kSmallWG = 512;

// Sizes and LDS regions of a small problem (x-DST length L, nt = NT).
template <typename T, int L, int NT>
struct Small {
  using C = cplx<T>;
  static constexpr int Mx = L / 2, nx = Mx - 1, N = NT * nx;
  static constexpr int E = (N + kSmallWG - 1) / kSmallWG;   // elements of a thread
  static constexpr int LD = Mx + 1;                         // scratch row stride: odd, so rows spread over the banks
  // x pass: RX row pairs side by side, TX threads each; time pass: NP mode pairs, TT threads
  // each.  Both put whole idle waves at the end, which only take the barriers.
  static constexpr int TX = fft_tps<T, L>(), RX = kSmallWG / TX < NT / 2 ? kSmallWG / TX : NT / 2;
  static constexpr int TT = fft_tps<T, NT>(), NP = Mx / 2;
  static constexpr int G = TT >= 8 ? 8 : TT;
  static constexpr size_t align(size_t v) { return (v + 15) / 16 * 16; }
  static constexpr size_t exch = 0;   // FFT exchange
  static constexpr size_t exch_x = (size_t)RX * L * sizeof(C), exch_t = (size_t)NP * NT * sizeof(C);
  static constexpr size_t scratch = align(exch_x > exch_t ? exch_x : exch_t);
  static constexpr size_t z = scratch + align((size_t)NT * LD * sizeof(T));
  static constexpr size_t twx = z + align((size_t)N * sizeof(double));
  static constexpr size_t twt = twx + align(L * sizeof(C));
  static constexpr size_t abk = twt + align(NT * sizeof(C));
  static constexpr size_t sc = abk + align(2 * NT * sizeof(C));
  static constexpr size_t sci = sc + align(NT * sizeof(T));
  static constexpr size_t red = sci + align(NT * sizeof(T));
  static constexpr size_t parts = red + align((size_t)(NP * TT + NP * TT / G) * sizeof(double));
  static constexpr size_t total = parts + align((size_t)NP * sizeof(double));
  static constexpr bool ok =
      N <= 4096 && (sizeof(T) == 4 || NT <= 128) && NP * TT <= kSmallWG && (NT / 2) % RX == 0 && total <= kMaxTransformLds;
};

// One right-hand side's workgroup.
template <typename T, int L, int NT>
struct SmallRun {
  using M = Small<T, L, NT>;
  using C = cplx<T>;
  const DevPlan& P;
  const int b;
  const size_t off;
  C *exch, *twx, *twt;
  T *scr, *sc, *sci;
  double *z, *red, *parts;
  ScalarState& S;
  double (*dred)[3];
  SpectralWeights<T, NT> W;   // of this thread's mode pair

  __device__ __forceinline__ SmallRun(const DevPlan& P_, ScalarState& S_, double (*dred_)[3], unsigned char* lds)
      : P(P_), b(blockIdx.x), off((size_t)blockIdx.x * P_.N), S(S_), dred(dred_) {
    exch = reinterpret_cast<C*>(lds + M::exch);
    scr = reinterpret_cast<T*>(lds + M::scratch);
    z = reinterpret_cast<double*>(lds + M::z);
    twx = reinterpret_cast<C*>(lds + M::twx);
    twt = reinterpret_cast<C*>(lds + M::twt);
    sc = reinterpret_cast<T*>(lds + M::sc);
    sci = reinterpret_cast<T*>(lds + M::sci);
    red = reinterpret_cast<double*>(lds + M::red);
    parts = reinterpret_cast<double*>(lds + M::parts);
    C* abk = reinterpret_cast<C*>(lds + M::abk);
    move_state<true>(P, b, S);
    stage_table(twx, reinterpret_cast<const C*>(P.twx), L);
    stage_table(twt, reinterpret_cast<const C*>(P.twt), NT);
    stage_table(abk, reinterpret_cast<const C*>(P.abk), 2 * NT);
    stage_table(sc, reinterpret_cast<const T*>(P.sc), NT);
    stage_table(sci, reinterpret_cast<const T*>(P.sci), NT);
    __syncthreads();
    const int tid = threadIdx.x, s = tid % M::NP, j = tid / M::NP;
    if (j < M::TT) {
      const T* beta = reinterpret_cast<const T*>(P.beta);
      spectral_weights<T, NT>(W, j, abk, beta[2 * s], beta[2 * s + 1], (T)(0.5 / NT), 0);
    }
  }

  // The thread index, opaque to the compiler: otherwise it hoists every step's element
  // indices, stencil weights and LDS addresses out of the iteration loop, 300 spilled
  // registers at 63 x 64.
  static __device__ __forceinline__ int thread() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  }

  // Write the state back.
  __device__ __forceinline__ void leave() {
    __syncthreads();
    move_state<false>(P, b, S);
  }

  // Sine transform along x of every row of the scratch: in place, or with INV the result in
  // FP64 to z.  Ends with a barrier.
  template <bool INV>
  __device__ __forceinline__ void x_pass() {
    constexpr int R = FftShape<T, L>::R, TPS = M::TX, Mx = M::Mx, LD = M::LD;
    const int tid = thread(), s = tid % M::RX, j = tid / M::RX;
    const bool act = j < TPS;
    for (int p0 = 0; p0 < NT / 2; p0 += M::RX) {
      const int ra = 2 * (p0 + s), rb = ra + 1;
      C v[R];
      if (act) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const int t = j + i * TPS;
          const int src = t < Mx ? max(t - 1, 0) : min(2 * Mx - t - 1, Mx - 2);
          const T a = scr[ra * LD + src], c = scr[rb * LD + src];
          const bool zero = t == 0 || t == Mx, neg = t > Mx;
          v[i] = C{zero ? (T)0 : (neg ? -a : a), zero ? (T)0 : (neg ? -c : c)};
        }
      }
      if (p0) __syncthreads();   // the exchange region is free
      fft_seq<T, L, false>(v, j, exch + s, M::RX, twx, act);
      if (!act) continue;
      if constexpr (INV) {
        const double scl = 1.0 / sqrt((double)L);
#pragma unroll
        for (int i = 0; i < R / 2; ++i) {
          const int k = j + i * TPS;
          if (i > 0 || k > 0) {
            z[ra * M::nx + k - 1] = -(double)v[i].y * scl;
            z[rb * M::nx + k - 1] = (double)v[i].x * scl;
          }
        }
      } else {
        const T scl = (T)(1.0 / sqrt((double)L));
#pragma unroll
        for (int i = 0; i <= R / 2; ++i) {
          const int k = j + i * TPS;
          if (k == 0 || k > Mx) continue;
          scr[ra * LD + k - 1] = k == Mx ? (T)0 : -v[i].y * scl;
          scr[rb * LD + k - 1] = k == Mx ? (T)0 : v[i].x * scl;
        }
      }
    }
    __syncthreads();
  }

  // K Y K Y of every mode pair of the scratch, in place; returns <q, P^{-1} q> (thread 0).
  __device__ __forceinline__ double time_pass() {
    constexpr int R = FftShape<T, NT>::R, TPS = M::TT, LD = M::LD;
    const int tid = thread(), s = tid % M::NP, j = tid / M::NP;
    const bool act = j < TPS;
    C v[R];
    if (act) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int t = j + i * TPS;
        const T* g = scr + (NT - 1 - t) * LD + 2 * s;
        v[i] = cscale(C{g[0], g[1]}, sc[t]);
      }
    }
    const double gsum = time_core<T, NT>(v, j, s, exch + s, M::NP, twt, sc, sci, W, 0, 1, red, red + M::NP * TPS, act);
    if (act) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int t = (j + i * TPS - 1) & (NT - 1);
        const C o = cscale(v[i], sci[t]);
        scr[t * LD + 2 * s] = o.x;
        scr[t * LD + 2 * s + 1] = o.y;
      }
      if (j == 0) parts[s] = gsum;
    }
    __syncthreads();
    return sum_parts(parts, M::NP);
  }

  // (T v)_k at grid point x, v in LDS.
  __device__ __forceinline__ double apply_T_at(const double* v, int k, int x) const {
    const LCoef q = l_coef(P, x, 0);
    const double* lvl = v + k * M::nx;
    double out = apply_L(q, lvl, x);
    if (k >= 2) out += apply_L(q, lvl - 2 * M::nx, x);
    if (k >= 1) out -= 2.0 * lvl[x - M::nx];
    return out;
  }

  // The basis slot of z_{j}, from z in LDS.
  __device__ __forceinline__ void store_z(int j) {
    const int tid = thread();
    double* slot = P.Z[zslot(j)] + off;
#pragma unroll
    for (int i = 0; i < M::E; ++i) {
      const int e = tid + i * kSmallWG;
      if (e < M::N) slot[e] = z[e];
    }
  }
  __device__ __forceinline__ void load_z(int j) {
    const int tid = thread();
    const double* slot = P.Z[zslot(j)] + off;
#pragma unroll
    for (int i = 0; i < M::E; ++i) {
      const int e = tid + i * kSmallWG;
      if (e < M::N) z[e] = slot[e];
    }
    __syncthreads();
  }

  // Set-up: b = Y f into v_1, u = 0, ||b||^2, then z_1 = P^{-1} b (left in z) and gamma_1.
  __device__ __forceinline__ void setup(const double* __restrict__ f, double* __restrict__ u, const FinArgs& a) {
    const int tid = thread();
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < M::E; ++i) {
      const int e = tid + i * kSmallWG;
      if (e < M::N) {
        const int k = e / M::nx, x = e - k * M::nx;
        const double v = f[off + (NT - 1 - k) * M::nx + x];
        P.V[1][off + e] = v;
        u[off + e] = 0.0;
        scr[k * M::LD + x] = (T)v;
        acc += v * v;
      }
    }
    double tot = block_sum(acc);
    if (tid == 0) fin_scalar(P, b, &S.st, &S.x, FIN_BNORM, tot, Dots3{}, a);
    __syncthreads();
    if (S.st.state == ST_RUNNING) {
      x_pass<false>();
      tot = time_pass();
      x_pass<true>();
      store_z(1);
    }
    if (fin_begin(P, b, &S.st, &S.x, FIN_GAMMA_INIT, a) && tid == 0)
      fin_scalar(P, b, &S.st, &S.x, FIN_GAMMA_INIT, tot, Dots3{}, a);
    __syncthreads();
  }

  // One MINRES iteration; z holds z_j and, unless the solve stops, z_{j+1} afterwards.  Every
  // branch is uniform (the state is read behind a barrier).
  __device__ __forceinline__ void iterate(const double* __restrict__ f, double* __restrict__ u, const FinArgs& a) {
    const int tid = thread();
    if (S.st.state == ST_RUNNING) {
      const int j = S.st.iter + 1;
      double* q = P.V[(j + 1) % 3] + off;
      const double* vj = P.V[j % 3] + off;
      const double* vjm1 = P.V[j == 1 ? j % 3 : (j + 2) % 3] + off;   // v_0 has weight 0 at j = 1
      double* r = P.R + off;
      const bool track = S.st.track != 0;
      // matvec A z_j = Y T z_j with <A z_j, z_j>; the Lanczos vectors' loads go out first
      double az[M::E], bv[M::E], cv[M::E];
#pragma unroll
      for (int i = 0; i < M::E; ++i) {
        const int e = min(tid + i * kSmallWG, M::N - 1);
        bv[i] = vj[e];
        cv[i] = vjm1[e];
      }
      double acc = 0.0;
#pragma unroll
      for (int i = 0; i < M::E; ++i) {
        const int e = tid + i * kSmallWG;
        az[i] = 0.0;
        if (e < M::N) {
          const int k = e / M::nx;
          az[i] = apply_T_at(z, NT - 1 - k, e - k * M::nx);
          acc += az[i] * z[e];
        }
      }
      double tot = block_sum(acc);
      if (tid == 0) fin_scalar(P, b, &S.st, &S.x, FIN_DELTA, tot, Dots3{}, FinArgs{});
      __syncthreads();
      // Lanczos step (see LanczosStep), its result staged for the first transform
      const double cA = S.st.sig, cB = S.st.delta * S.st.sig, cC = S.st.gamma * S.st.sig_prev;
      Dots3 d{0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < M::E; ++i) {
        const int e = tid + i * kSmallWG;
        if (e < M::N) {
          const double v = cA * az[i] - cB * bv[i] - cC * cv[i];
          q[e] = v;
          const int k = e / M::nx;
          scr[k * M::LD + e - k * M::nx] = (T)v;
          d.a += v * v;
          if (track) {
            const double rn = S.st.r1 * r[e] + S.st.r2 * bv[i];
            r[e] = rn;
            d.b += v * rn;
            d.c += rn * rn;
          } else {
            d.b += v * bv[i];
            d.c += v * cv[i];
          }
        }
      }
      dots_reduce(d, dred[tid >> 6]);
      __syncthreads();
      x_pass<false>();
      tot = time_pass();
      // gamma_{j+1}, Givens step, stopping test
      if (tid == 0) {
        Dots3 dots{0.0, 0.0, 0.0};
        for (int w = 0; w < kSmallWG / 64; ++w) {
          dots.a += dred[w][0];
          dots.b += dred[w][1];
          dots.c += dred[w][2];
        }
        fin_scalar(P, b, &S.st, &S.x, FIN_GAMMA_ITER, tot, dots, FinArgs{});
      }
      __syncthreads();
      step_coefs(&S.st, &S.x);
      __syncthreads();
    }
    // the iterate from the resident basis when a check, a stop or the flush needs it; it
    // takes the place of z_j for the check
    if (S.st.form_now) {
      form(u);
      __syncthreads();
    }
    // explicit residual check, end of the scalar steps (snapshot)
    double tot = 0.0;
    if (S.st.state == ST_RUNNING && S.st.need_check) {
      double acc = 0.0;
#pragma unroll
      for (int i = 0; i < M::E; ++i) {
        const int e = tid + i * kSmallWG;
        if (e < M::N) {
          const int k = e / M::nx, x = e - k * M::nx;
          const double rv = f[off + e] - apply_T_at(z, k, x);
          acc += rv * rv;
          if (S.st.want_r) P.R[off + (NT - 1 - k) * M::nx + x] = rv;
        }
      }
      tot = block_sum(acc);
    }
    if (fin_begin(P, b, &S.st, &S.x, FIN_RES, a) && tid == 0)
      fin_scalar(P, b, &S.st, &S.x, FIN_RES, tot, Dots3{}, a);
    __syncthreads();
    // the second half of z_{j+1}
    if (S.st.state == ST_RUNNING) {
      x_pass<true>();
      store_z(S.st.iter + 1);
    }
  }

  // u = [u +] sum_l xm_l z_l over the current cycle of the basis and the carried w vectors
  // (with flush also the two w vectors from their coefficients); u also to z.
  __device__ void form(double* __restrict__ u) {
    const int tid = thread();
    const double* kc = S.x.kc;
    const int nb = S.st.nbasis, base = S.st.cbase;
    const bool flush = S.st.flush_now != 0, add = S.st.u_valid != 0;
    double* X = u + off;
    double* W1 = P.W[0] + off;
    double* W2 = P.W[1] + off;
    double ax[M::E], a1[M::E], a2[M::E];
#pragma unroll
    for (int i = 0; i < M::E; ++i) {
      const int e = min(tid + i * kSmallWG, M::N - 1);
      ax[i] = add ? X[e] : 0.0;
      a1[i] = a2[i] = 0.0;
      if (base) {
        const double p = W1[e], q = W2[e];
        ax[i] += kc[kBasis] * p + kc[kBasis + 1] * q;
        a1[i] = kc[kCoefs + kBasis] * p + kc[kCoefs + kBasis + 1] * q;
        a2[i] = kc[2 * kCoefs + kBasis] * p + kc[2 * kCoefs + kBasis + 1] * q;
      }
    }
    for (int l = 0; l < nb; ++l) {
      const double* zl = P.Z[zslot(base + l + 1)] + off;
      const double c0 = kc[l], c1 = kc[kCoefs + l], c2 = kc[2 * kCoefs + l];
      double v[M::E];
#pragma unroll
      for (int i = 0; i < M::E; ++i) v[i] = zl[min(tid + i * kSmallWG, M::N - 1)];
#pragma unroll
      for (int i = 0; i < M::E; ++i) {
        ax[i] += c0 * v[i];
        a1[i] += c1 * v[i];
        a2[i] += c2 * v[i];
      }
    }
#pragma unroll
    for (int i = 0; i < M::E; ++i) {
      const int e = tid + i * kSmallWG;
      if (e < M::N) {
        X[e] = ax[i];
        z[e] = ax[i];
        if (flush) {
          W1[e] = a1[i];
          W2[e] = a2[i];
        }
      }
    }
  }
};

template <typename T, int L, int NT>
__global__ void __launch_bounds__(kSmallWG)
k_iter_small(DevPlan P, const double* __restrict__ f, double* __restrict__ u) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ ScalarState S;
  __shared__ double dred[16][3];
  SmallRun<T, L, NT> run(P, S, dred, smem);
  if (S.st.state == ST_RUNNING) run.load_z(S.st.iter + 1);
  run.iterate(f, u, FinArgs{});
  run.leave();
}

template <typename T, int L, int NT>
__global__ void __launch_bounds__(kSmallWG)
k_setup_small(DevPlan P, const double* __restrict__ f, double* __restrict__ u, FinArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ ScalarState S;
  __shared__ double dred[16][3];
  SmallRun<T, L, NT> run(P, S, dred, smem);
  run.setup(f, u, a);
  run.leave();
}

// A whole solve in one launch: the set-up, then iterations until the right-hand side
// stops (at most maxit + 1, a safety net: the state machine stops it by maxit), and one
// snapshot at the end.
template <typename T, int L, int NT>
__global__ void __launch_bounds__(kSmallWG)
k_solve_small(DevPlan P, const double* __restrict__ f, double* __restrict__ u, FinArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ ScalarState S;
  __shared__ double dred[16][3];
  a.post = -1;
  SmallRun<T, L, NT> run(P, S, dred, smem);
  run.setup(f, u, a);
  for (int it = 0; it <= a.maxit && S.st.state == ST_RUNNING; ++it) {
    run.iterate(f, u, a);
    __syncthreads();   // z_{j+1} and the state are visible to every thread
  }
  if (threadIdx.x == 0) {
    S.st.snap = 0;
    post_snapshot(P, blockIdx.x, &S.st);
  }
  run.leave();
}

// what: 0 one iteration, 1 the set-up, 2 a whole solve (set-up and iterations)
template <typename T, int L, int NT>
hipError_t launch_small_t(const DevPlan& P, const double* f, double* u, hipStream_t s, int what,
                          const FinArgs& a) {
  if constexpr (!Small<T, L, NT>::ok) {
    return hipErrorInvalidValue;
  } else {
    constexpr size_t lds = Small<T, L, NT>::total;
    if (what == 1)
      hipLaunchKernelGGL((k_setup_small<T, L, NT>), dim3(P.B), dim3(kSmallWG), lds, s, P, f, u, a);
    else if (what == 2)
      hipLaunchKernelGGL((k_solve_small<T, L, NT>), dim3(P.B), dim3(kSmallWG), lds, s, P, f, u, a);
    else
      hipLaunchKernelGGL((k_iter_small<T, L, NT>), dim3(P.B), dim3(kSmallWG), lds, s, P, f, u);
    return hipGetLastError();
  }
}

#define ABAC_SMALL_NT(LL, CALL)               \
  switch (P.nt) {                             \
    case 8: return CALL(LL, 8);               \
    case 16: return CALL(LL, 16);             \
    case 32: return CALL(LL, 32);             \
    case 64: return CALL(LL, 64);             \
    case 128: return CALL(LL, 128);           \
    case 256: return CALL(LL, 256);           \
    default: return hipErrorInvalidValue;     \
  }

template <typename T>
hipError_t small_dispatch(const DevPlan& P, const double* f, double* u, hipStream_t s, int what,
                          const FinArgs& a) {
#define CALL(LL, NN) launch_small_t<T, LL, NN>(P, f, u, s, what, a)
  switch (2 * P.Mx) {
    case 16: ABAC_SMALL_NT(16, CALL)
    case 32: ABAC_SMALL_NT(32, CALL)
    case 64: ABAC_SMALL_NT(64, CALL)
    case 128: ABAC_SMALL_NT(128, CALL)
    default: return hipErrorInvalidValue;
  }
#undef CALL
}

template <typename T>
bool small_valid_t(int L, int nt) {
#define CALL(LL, NN) Small<T, LL, NN>::ok
  switch (L) {
#define ABAC_SMALL_NT_OK(LL)                                                                            \
  case LL:                                                                                             \
    switch (nt) {                                                                                      \
      case 8: return CALL(LL, 8);                                                                      \
      case 16: return CALL(LL, 16);                                                                    \
      case 32: return CALL(LL, 32);                                                                    \
      case 64: return CALL(LL, 64);                                                                    \
      case 128: return CALL(LL, 128);                                                                  \
      case 256: return CALL(LL, 256);                                                                  \
      default: return false;                                                                           \
    }
    ABAC_SMALL_NT_OK(16) ABAC_SMALL_NT_OK(32) ABAC_SMALL_NT_OK(64) ABAC_SMALL_NT_OK(128)
#undef ABAC_SMALL_NT_OK
    default: return false;
  }
#undef CALL
}

}  // namespace

hipError_t launch_iter_small(const DevPlan& P, int prec, const double* f, double* u, hipStream_t s) {
  return prec ? small_dispatch<float>(P, f, u, s, 0, FinArgs{}) : small_dispatch<double>(P, f, u, s, 0, FinArgs{});
}

hipError_t launch_setup_small(const DevPlan& P, int prec, const double* f, double* u, const FinArgs& a, hipStream_t s) {
  return prec ? small_dispatch<float>(P, f, u, s, 1, a) : small_dispatch<double>(P, f, u, s, 1, a);
}

hipError_t launch_solve_small(const DevPlan& P, int prec, const double* f, double* u, const FinArgs& a, hipStream_t s) {
  return prec ? small_dispatch<float>(P, f, u, s, 2, a) : small_dispatch<double>(P, f, u, s, 2, a);
}

bool small_path_valid(int nx, int ny, int nt, int prec) {
  if (ny || prec == ABAC_PREC_NONE) return false;
  const int L = 2 * (nx + 1);
  return prec ? small_valid_t<float>(L, nt) : small_valid_t<double>(L, nt);
}

}  // namespace abac
