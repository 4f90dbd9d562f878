// Internal definitions shared by the HIP translation units of the ABAC library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fft_device.h"

namespace abac {

// Solve state of one right-hand side, resident in device memory.  Every scalar of
// the MINRES recurrence lives here; kernels read what they need at entry and the
// last block of a reduction writes the new values.
enum : int { ST_IDLE = 0, ST_RUNNING = 1, ST_DONE = 2 };
constexpr int kSnapRing = 16;   // host snapshot slots per right-hand side
constexpr size_t kMaxTransformLds = 152 * 1024;   // dynamic LDS per transform block (gfx950: 160 KB per workgroup, 8 KB kept for static LDS)

// Resident Krylov basis: the z vectors live in a ring of slots, and the w and x
// recurrences run on coefficient vectors over the kBasis newest of them (a cycle) and
// over the two w vectors the cycle started from.  The iterate is formed only when a
// residual check, a breakdown or the end of the solve needs it, and every kBasis
// iterations a flush forms x and the two newest w and starts the next cycle; no other
// step of an iteration touches x or w.  z_{j+1} is written while the cycle of z_j is
// still needed, so the ring holds more than kBasis slots.
constexpr int kBasis = 12;
constexpr int kZSlots = kBasis + 2;
constexpr int kCoefs = kBasis + 2;   // basis coefficients of a vector: the cycle's z, then the two carried w
__host__ __device__ inline int zslot(int j) { return (j - 1) % kZSlots; }

struct MinresState {
  double gamma;     // gamma_j, current Lanczos off-diagonal
  double sig;       // 1/gamma_j: scale of the stored (unnormalised) v_j and z_j
  double sig_prev;  // 1/gamma_{j-1}: scale of the stored v_{j-1} (0 at j = 1)
  double delta;     // delta_j = <A z_j, z_j>
  double c1, c2;    // Givens cosines c_{j-1}, c_{j-2}
  double s1, s2;    // Givens sines s_{j-1}, s_{j-2}
  double eta;       // running right-hand side of the rotated least-squares problem
  double r1, r2;    // r_j = r1 * r_{j-1} + r2 * Vslot_{j+1}
  double rnorm2;    // ||r_j||^2 from the recurrence (an estimate unless `track`)
  double bnorm2;    // ||b||^2
  double tol2;      // tol^2
  double res2;      // last explicit ||b - A x||^2
  int iter;         // completed iterations
  int maxit;
  int state;        // ST_*
  int status;       // abac_status of this right-hand side
  int explicit_mode;
  int need_check;   // the recurrence cannot exclude convergence: confirm it explicitly
  int lucky;        // gamma_{j+1} == 0: the Krylov space is invariant
  int snap;         // sequence number of the next host snapshot
  int cbase;        // iterations before the current cycle of the basis
  int nbasis;       // z vectors of the current cycle with coefficients
  int u_valid;      // u holds the iterate the coefficients add to (0: they start from x = 0)
  int basis_dirty;  // u does not yet hold the iterate of the basis coefficients
  int form_now;     // this iteration forms u from the basis (flush: also w_j, w_{j-1})
  int flush_now;
  int track;        // P.R holds the residual vector, updated by the first transform pass
  int want_r;       // the explicit check also writes the residual vector to P.R
  int hold;         // the stopping test asked for a form or check step: nothing else runs before it
  int tail;         // the inverse transforms of the last iteration were held back
  int epoch;        // which solve of the plan this is (tags its snapshots)
};
// An iteration's kernels skip a right-hand side that stopped or waits for a check.
__device__ __forceinline__ bool rhs_active(const MinresState* st) { return st->state == ST_RUNNING && !st->hold; }
// How a transform pass decides that: 0 always run; CHECK_ACTIVE; CHECK_RESUME the inverse
// passes after a check, only where they were held back.
enum PassCheck : int { CHECK_NONE = 0, CHECK_ACTIVE = 1, CHECK_RESUME = 2 };
__device__ __forceinline__ bool pass_runs(const MinresState* st, int check) {
  return check == CHECK_NONE || (rhs_active(st) && (check == CHECK_ACTIVE || st->tail));
}

// What the host sees of a right-hand side after the set-up and after the scalar steps of
// an iteration, in host-mapped memory.  `word` is written last and names the snapshot, so
// the host needs no event to know that a snapshot is complete: epoch (16 bits), sequence
// number + 1 (24), Arnoldi column (GMRES, bits 3-7), hold (bit 2), state (bits 0-1).
struct Snapshot {
  unsigned long long word;
  int status, iter;
  double rnorm2, bnorm2, res2, tol2;
  double pad_[2];
};
static_assert(sizeof(Snapshot) == 64, "one line of host memory per snapshot");
__host__ __device__ inline unsigned long long snap_word(int epoch, long long seq, int state, int hold, int column = 0) {
  return (unsigned long long)(epoch & 0xffff) << 48 | (unsigned long long)((seq + 1) & 0xffffff) << 24 |
         (unsigned long long)column << 3 | (unsigned long long)(hold ? 4 : 0) | (unsigned long long)state;
}
__host__ __device__ inline unsigned long long snap_name(unsigned long long word) { return word >> 24; }
__host__ __device__ inline int snap_state(unsigned long long word) { return (int)(word & 3); }
__host__ __device__ inline bool snap_hold(unsigned long long word) { return (word & 4) != 0; }
__host__ __device__ inline int snap_column(unsigned long long word) { return (int)(word >> 3 & 31); }

// More per right-hand side state of a MINRES solve, kept in the right-hand side's GMRES
// state (the two solvers never run on one plan together).
//
// The residual vector r_j = r1 r_{j-1} + r2 V_{j+1} is not stored: its norm decides when
// to stop, and the first transform pass has V_{j+1}, V_j and V_{j-1} in registers, whose
// pairwise inner products cost no memory traffic.  Unrolled three steps,
//   r_j = E + ra V_{j-1} + rb V_j + rc V_{j+1},  E = r1_j r1_{j-1} r1_{j-2} r_{j-3},
// so ||r_j|| lies within ||E|| of the norm of the last three terms, and ||E|| is at
// most the product of the r1 (squared sines, small where the iteration converges) and
// the bound on ||r_{j-3}||.  Convergence is only tested explicitly where that interval
// reaches the tolerance.  Where it is too wide to decide (slow convergence) the explicit
// test leaves the residual vector in P.R and the first pass updates it from there on,
// 16 bytes per unknown.  Against a separate update pass of 24 bytes per unknown and
// iteration, whole solves (with the inverse passes of the last iteration skipped):
// 511^2 x 512 FP32 transforms 38.5 -> 32.0 ms, 255^2 x 256 FP64 5.56 -> 4.81 ms,
// 64 x 127^2 x 128 FP64 37.3 -> 32.2 ms, 63^2 x 64 FP32 0.79 -> 0.71 ms.
struct MinresExt {
  double kc[3 * kCoefs];    // coefficients of x_j - u, w_j, w_{j-1}
  double rb, rc;            // r_j's coefficients on V_j and V_{j+1}
  double n0, n1, d01;       // ||V_j||^2, ||V_{j+1}||^2, <V_j, V_{j+1}> of the last step
  double hi[3];             // upper bounds on ||r_j||, ||r_{j-1}||, ||r_{j-2}||
  double r1p[2];            // r1 of the last two steps
  double wa, wb, wc, xc;    // w_j = wa z_j - wb w_{j-1} - wc w_{j-2}; x_j = x_{j-1} + xc w_j
  double step;              // 1: the coefficients kc wait for that step
};

// vector kernels: 256 threads, about 16 elements per thread, at most 1024 blocks per
// right-hand side (update_blocks)
constexpr int kVecThreads = 256;
constexpr int kVecPerThread = 16;
constexpr int kVecMaxBlocks = 1024;

// Restarted GMRES (right preconditioning with C_alpha^{-1}) on T u = f: per right-hand
// side state.  The Arnoldi basis v_0 .. v_restart lives in the plan's Krylov vector
// slots (so restart <= kGmresMax), H is the rotated Hessenberg matrix, column-major.
constexpr int kGmresMax = 15;
struct GmresState {
  double H[(kGmresMax + 1) * kGmresMax];   // H[c * (kGmresMax + 1) + l]: row l, column c
  double cs[kGmresMax], sn[kGmresMax];     // Givens rotations
  double g[kGmresMax + 1];                 // rotated beta e_1
  double y[kGmresMax];                     // least-squares solution (when forming u)
  double h1[kGmresMax + 1], h2[kGmresMax + 1];   // the two Gram-Schmidt passes of a column
  double sig[kGmresMax + 1];                 // v_l = sig_l * (slot l): slots hold unnormalised vectors
  double bnorm2, tol2, scale, res2, resid2;
  int iter, k, maxit, restart, state, status, need, explicit_mode, restart_now;
  int reorth;   // the current column needs the second Gram-Schmidt pass
  int epoch, snap;   // this solve's tag; the number of the next snapshot
};
static_assert(sizeof(MinresExt) <= sizeof(GmresState), "the MINRES state shares the GMRES state's memory");
// Everything a kernel needs about a plan, passed by value.
struct DevPlan {
  int nx, ny, nt, B;   // ny = 0 in 1D
  int ny1;             // max(ny, 1): rows per level
  int Mx, My;          // nx+1, ny+1 (My = 1 in 1D)
  int m;               // nx * ny1: unknowns per level
  int ms;              // Mx * ny1: scratch modes per level (one zero pad column)
  int stream;          // vectors too large for the caches: see stream_branch
  int fold;            // the first transform pass forms delta_j from the matvec's partials
  long long N;         // nt * m: unknowns per right-hand side
  long long NS;        // nt * ms: scratch values per right-hand side
  double c0, cx, cy;   // (L s)_i = c0 s_i - cx (s_{i-1} + s_{i+1}) - cy (s_{i-nx} + s_{i+nx})
  double tau, tau2;
  // variable coefficient a(x) of div(a grad u) (eq. (3.2)); both NULL for a = 1.
  // coef_x: ny1 rows of Mx face weights (tau^2/2) a(x_{i+1/2}, y_j) / hx^2, i = 0..nx;
  // coef_y (2D): My rows of nx face weights (tau^2/2) a(x_i, y_{j+1/2}) / hy^2, j = 0..ny.
  const double* coef_x;
  const double* coef_y;
  // spectral tables, stored in the transform precision
  const void* twx;     // 2*Mx complex twiddles exp(-2 pi i e/(2 Mx))
  const void* twy;     // 2*My complex twiddles (2D)
  const void* twt;     // nt complex twiddles exp(-2 pi i e/nt)
  const void* beta;    // ms real: (tau^2/2) * eigenvalue of -Laplace_h of each scratch mode
  const void* abk;     // 2*nt complex: (A_k, B_k), mu_k(beta) = A_k + beta * B_k
  const void* sc;      // nt real: a^t,  a = alpha^{1/nt}
  const void* sci;     // nt real: a^{-t}
  void* scratch;       // B * NS transform values
  // MINRES vectors, each B * N doubles
  double* V[3];
  double* Z[kZSlots];  // slot zslot(j) holds the stored z_j
  double* W[2];
  GmresState* gst;     // B entries (GMRES solves; MINRES solves keep their MinresExt there)
  double* gparts;      // B x (kGmresMax + 1) x kVecMaxBlocks partial dot products
  double* R;           // MINRES: the residual vector while it is tracked; GMRES: the cycle's first iterate
  double* dot3;        // third inner product of the first transform pass, one partial per block
  long long dot3_stride;   // doubles per right-hand side
  MinresState* st;     // B entries
  double* partials;    // PART_KINDS * B * maxparts
  Snapshot* host_ring;     // device view of the host-mapped snapshot ring (kSnapRing * B)
  int maxparts;
  // workgroup sizes of the transform kernels (chosen by the plan's autotuner)
  int wg_x, wg_xi, wg_y, wg_t;
  int wg_s;            // fused 2D passes (0: separate x and y passes)
  int small;           // 1: one workgroup per right-hand side runs a whole iteration
  int st_chunk;        // forward time levels per partial sum of the matvec
  int st_march;        // chunks a matvec block marches over
  int st_threads;      // threads per matvec block
  int st_cols;         // columns per matvec thread (2, or 1 for a one-column grid)
  int st_rows;         // grid rows per matvec block (1 in 1D)
  int gamma_nparts;    // partial sums of <q, P^{-1} q> per right-hand side
  int prec;            // 0 FP64 transforms, 1 FP32 transforms, 2 no preconditioner
};

// ---------------------------------------------------------------------------
// deterministic reductions: every block of a reducing kernel writes one partial
// (fixed-order block sum) into its own slot; a later kernel sums the slots in index
// order.  Kernel boundaries provide the visibility, so no fences or atomics are used.
// ---------------------------------------------------------------------------
enum PartKind : int { PART_DELTA = 0, PART_GAMMA = 1, PART_RNORM = 2, PART_RES = 3, PART_KINDS = 4 };

__device__ __forceinline__ double* part_slot(const DevPlan& P, int kind, int b) {
  return P.partials + ((size_t)kind * P.B + b) * P.maxparts;
}

__device__ __forceinline__ MinresExt* minres_ext(const DevPlan& P, int b) {
  return reinterpret_cast<MinresExt*>(P.gst + b);
}

// The inner products a block of the first transform pass forms for the stopping test
// (see MinresExt): <q, q>, then <q, V_j> and <q, V_{j-1}>, or with the residual tracked
// <q, r_{j-1}> and ||r_{j-1}||^2.  They are summed in one order, whatever the tile, so that
// tuned, batched and grouped solves take the same decisions: a wave sums a unit of 64 / TPS row
// pairs (TPS threads to a sequence; TPS / 64 waves a unit of one row pair where TPS > 64),
// units are added two by two up to a group of twice those of a 1024-thread block, partly by
// the block, which leaves one partial of the units it has, partly by the scalar step, which
// then sums the groups.  In the fused x-y passes the unit is a level, the group two of them.
// Partials per block summed as they come, so that the tile decides, take the scalar step as
// long at 255^2 x 256 FP64 (10.5 us), 5 us less at 511^2 x 512 FP32 (25 and 20 us).
__host__ __device__ constexpr int dot_group_units(int tps) { return 2048 / (tps > 64 ? tps : 64); }
struct Dots3 {
  double a, b, c;
};
__device__ __forceinline__ double* dot_slot(const DevPlan& P, int which, int b) {
  return which == 0 ? part_slot(P, PART_RNORM, b) : which == 1 ? part_slot(P, PART_RES, b) : P.dot3 + b * P.dot3_stride;
}

template <int N>
__device__ __forceinline__ double tree_sum(double* v) {
#pragma unroll
  for (int d = 1; d < N; d *= 2)
#pragma unroll
    for (int i = 0; i < N; i += 2 * d) v[i] += v[i + d];
  return v[0];
}

// Every wave leaves its sums of three values in `red` (the caller places the barrier).
__device__ __forceinline__ void dots_reduce(Dots3 d, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    d.a += __shfl_down(d.a, off, 64);
    d.b += __shfl_down(d.b, off, 64);
    d.c += __shfl_down(d.c, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0] = d.a;
    red[1] = d.b;
    red[2] = d.c;
  }
}
// Where partial i of n in groups of `group` lies: the pairs of a group `groups` apart, so that
// consecutive threads of the scalar step read consecutive groups.
__device__ __forceinline__ int dot_place(int i, int n, int group) {
  const int groups = (n + group - 1) / group, g = i / group, j = i - g * group;
  return ((j >> 1) * groups + g) * 2 + (j & 1);
}

// The partial of block blk of n, from the sums of UNITS units of WAVES waves each.
template <int UNITS, int WAVES>
__device__ __forceinline__ void dots_store(const DevPlan& P, int b, int blk, int n, int group, const double (*red)[3]) {
  if (threadIdx.x < 3) {
    double s[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      s[u] = red[u * WAVES][threadIdx.x];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) s[u] += red[u * WAVES + w][threadIdx.x];
    }
    dot_slot(P, threadIdx.x, b)[dot_place(blk, n, group)] = tree_sum<UNITS>(s);
  }
}

// Sum of v over the block; the result is valid in thread 0.  Ends with a barrier so
// the shared buffer can be reused.
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double red_ws[16];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red_ws[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) s += red_ws[i];
  }
  __syncthreads();
  return s;
}

// Fixed-order sum of n partials by the whole block (pairs per thread, then the block
// tree); result valid in thread 0.  `part` is 16-byte aligned.
//
// A thread's share of that sum, for thread t of a block of nt threads.  Its loads go out in
// batches before any is added: one load at a time costs an L2 trip each (255^2 x 256:
// 32 k partials over 1024 threads and three sums of 16 k, the Givens step 24 -> 16 us).
__device__ __forceinline__ double parts_share(const double* __restrict__ part, int n, int t, int nt) {
  constexpr int BATCH = 8;
  const double2* p2 = reinterpret_cast<const double2*>(part);
  const int n2 = n >> 1;
  double s = 0.0;
  for (int i0 = t; i0 < n2; i0 += BATCH * nt) {
    double2 v[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = p2[min(i0 + u * nt, n2 - 1)];
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (i0 + u * nt < n2) s += v[u].x + v[u].y;
  }
  if ((n & 1) && t == 0) s += part[n - 1];
  return s;
}

// The same of three times n partials in groups of 2 H = 2 Q steps (dot_place; what is missing of
// the last group counts as 0), four pairs of each at a time: of 4 / Q groups, or with Q = 4 a
// whole, a half or a quarter of one (steps 1, 2 or 4).
template <int Q>
__device__ __forceinline__ Dots3 group_share(const double* const (&part)[3], int n, int steps, int t, int nt) {
  const int H = Q < 4 ? Q : 4 * steps, groups = (n + 2 * H - 1) / (2 * H);
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
  for (int g0 = t; g0 < groups; g0 += 4 / Q * nt) {
    double even[3], half[3];
#pragma unroll 1
    for (int st = 0; st < (Q < 4 ? 1 : steps); ++st) {
      double2 v[3][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned at = (st * Q + q % Q) * groups + min(g0 + q / Q * nt, groups - 1);
#pragma unroll
        for (int r = 0; r < 3; ++r) v[r][q] = reinterpret_cast<const double2*>(part[r])[at];
      }
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        double w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = 2 * ((g0 + q / Q * nt) * H + st * Q + q % Q);
          w[q] = (i < n ? v[r][q].x : 0.0) + (i + 1 < n ? v[r][q].y : 0.0);
        }
        if constexpr (Q < 4) {
#pragma unroll
          for (int u = 0; u < 4 / Q; ++u)
            if (g0 + u * nt < groups) s[r] += tree_sum<Q>(w + u * Q);
        } else {
          double x = tree_sum<4>(w);
          if (st & 1) x += even[r];
          if (st == 3) x += half[r];
          if (st == steps - 1) s[r] += x;
          else if (st & 1) half[r] = x;
          else even[r] = x;
        }
      }
    }
  }
  return {s[0], s[1], s[2]};
}

__device__ __forceinline__ double sum_parts(const double* __restrict__ part, int n) {
  return block_sum(parts_share(part, n, threadIdx.x, blockDim.x));
}

// Accesses of vectors that no kernel reads again before as much other data has passed (the
// Lanczos vectors, the basis, an apply's input and output): marked non-temporal they leave
// the caches to what the next pass reads, the transform scratch and the matvec's output.
// Three read streams and one written one of 133 MB: 5.6 TB/s plain, 6.8 with such loads;
// of 1 GiB 5.7 and 6.3.  Loads of the scratch itself (y and time passes) are faster plain:
// 255^2 x 256 FP64 4.04 ms per solve against 4.12 to 4.17 with them marked.
//
// They are marked only where the vectors of the batch take 64 MB, twice the L2s (P.stream): the
// next pass finds a smaller vector there.  Whole solves with the marks against without:
// 1.01 to 1.06 of the time at 16 MB, 1.01 to 1.04 at 32, 1.01 to 1.02 at 47, 0.98 to 1.01 at 62 to
// 64, 0.96 to 1.00 at 79 to 95, 0.90 to 0.93 at 127.  The iterate's reads of the basis are marked
// at every size (form_from_basis).  stream_branch makes the choice outside a sweep's loops; its
// marked branch holds an empty asm statement, since the compiler merges two branches that
// differ in the marks alone into one of plain accesses.
template <bool STREAM, typename V>
__device__ __forceinline__ V stream_load(const V* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool STREAM, typename V>
__device__ __forceinline__ void stream_store(V* p, V v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <typename F>
__device__ __forceinline__ void stream_branch(int stream, F&& sweep) {
  if (stream) {
    asm volatile("");
    sweep(std::true_type{});
  } else {
    sweep(std::false_type{});
  }
}

// Write snapshot `seq` of right-hand side b to the host-mapped ring (by one thread).  Every
// store goes past the caches (system scope).  Of a solve that has stopped, the word that
// names the snapshot is stored once the others have been acknowledged (a system-scope fence
// would also write the whole L2 back); while it runs, the others are hints, and the step
// does not wait for host memory.
__device__ __forceinline__ void write_snapshot(const DevPlan& P, int b, int seq, unsigned long long word, bool stopped,
                                               int status, int iter, double rnorm2, double bnorm2, double res2,
                                               double tol2) {
  if (!P.host_ring) return;
  Snapshot* s = P.host_ring + (size_t)(seq % kSnapRing) * P.B + b;
#define ABAC_PUT(field, value) __hip_atomic_store(&s->field, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)
  ABAC_PUT(status, status);
  ABAC_PUT(iter, iter);
  ABAC_PUT(rnorm2, rnorm2);
  ABAC_PUT(bnorm2, bnorm2);
  ABAC_PUT(res2, res2);
  ABAC_PUT(tol2, tol2);
  if (stopped) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  ABAC_PUT(word, word);
#undef ABAC_PUT
}

// Workgroups are dispatched round-robin over the 8 XCDs; remap the hardware block
// index so each XCD receives a contiguous range of logical blocks (shared halo
// rows then hit the same L2).
__device__ __forceinline__ int xcd_remap(int w, int n) {
  const int q = n >> 3, rem = n & 7;
  const int x = w & 7, slot = w >> 3;
  return x * q + (x < rem ? x : rem) + slot;
}

// ---------------------------------------------------------------------------
// host-side launchers (defined in the kernel translation units)
// ---------------------------------------------------------------------------
// PLAIN: y = Y T x; MINRES: the Lanczos matvec with <Y T z, z>; RESIDUAL: ||f - T u||^2
// when the solve asked for a check; REPORT: ||f - T u||^2 always; T: y = T x (natural
// time order); RESVEC: y = f - T x and its squared norm (partials in PART_RES)
enum StencilMode : int {
  STENCIL_PLAIN = 0, STENCIL_MINRES = 1, STENCIL_RESIDUAL = 2, STENCIL_REPORT = 3, STENCIL_T = 4, STENCIL_RESVEC = 5
};
enum FwdMode : int { FWD_PLAIN = 0, FWD_LANCZOS = 1 };
// last pass: INV_PLAIN writes out; the MINRES set-up and iteration modes write z_1 /
// z_{j+1} into its basis slot.  The identity preconditioner (GAMMA modes) also forms the
// partial sums of <q, z>; elsewhere the time pass forms <q, P^{-1} q>.
enum InvMode : int { INV_PLAIN = 0, INV_GAMMA_INIT = 1, INV_GAMMA_ITER = 2, INV_Z_INIT = 3, INV_Z_ITER = 4 };
enum FinKind : int {
  FIN_BNORM = 0, FIN_DELTA = 1, FIN_GAMMA_INIT = 2,
  FIN_GAMMA_ITER = 3,   // Givens step and stopping test of an iteration; decides forming u
  FIN_RES = 4, FIN_REPORT = 5,
  FIN_FINAL = 6    // end of a solve: form u if it is stale
};

// matvec decomposition: a tile is a band of st_rows grid rows times st_threads * st_cols
// columns; a block covers a tile and st_march chunks of st_chunk forward time levels (plus
// their mirrors), and leaves one partial sum per chunk
// two doubles moved by one 16-byte access; 8-byte alignment suffices on gfx950 (rows of
// odd length start at odd 8-byte offsets)
typedef double dpair __attribute__((ext_vector_type(2), aligned(8)));

constexpr int kStencilThreads = 256;
constexpr int kStencilMarch = 4;      // most chunks of a block: 8 levels in chunks of 2
constexpr int kStencilWaves = 2048;   // 2 waves per SIMD on 256 CUs x 4 SIMDs
__host__ __device__ inline int stencil_tiles(const DevPlan& P) {
  const int cols = P.st_threads * P.st_cols;
  return ((P.ny1 + P.st_rows - 1) / P.st_rows) * ((P.nx + cols - 1) / cols);
}
__host__ __device__ inline int stencil_blocks(const DevPlan& P, int levels) {
  return stencil_tiles(P) * ((P.nt / 2 + levels - 1) / levels);
}
// partial sums per right-hand side
__host__ __device__ inline int stencil_parts(const DevPlan& P) { return stencil_blocks(P, P.st_chunk); }
// The longest chunk of 64/32/16/8/4/2 levels whose blocks fill the GPU once at the matvec's
// occupancy: those of one right-hand side down to 8 levels, of `rhs` of them below.  (More
// than 8 levels where a batch fills the GPU with them gained nothing: 64 x 63^2 x 64.)
inline int stencil_chunk(const DevPlan& P, int rhs) {
  int c = 64;
  while (c > 2 && (long long)stencil_blocks(P, c) * (c > 8 ? 1 : rhs) * (P.st_threads / 64) < kStencilWaves) c /= 2;
  return c;
}
// <A z_j, z_j> from the matvec's partials, by each wave that calls it, in one order: the
// scalar step and the first transform pass (DevPlan::fold) get the same bits, so that a
// batch whose vectors are too large to fold equals its right-hand sides on their own.
__device__ __forceinline__ double delta_sum(const DevPlan& P, int b) {
  double s = parts_share(part_slot(P, PART_DELTA, b), stencil_parts(P), threadIdx.x & 63, 64);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  return s;
}

int update_blocks(const DevPlan& P);
// the first pass's partials of an inner product per right-hand side with tiles of wg threads,
// and how many of them make a group
struct DotParts {
  int n, group;
};
DotParts dot_parts(const DevPlan& P, int wg);

hipError_t launch_stencil(const DevPlan& P, int mode, const double* x, double* y, const double* f, hipStream_t s);
hipError_t launch_rhs(const DevPlan& P, const double* src, const double* psi0, const double* psi1, double* f,
                      hipStream_t s);
hipError_t launch_init(const DevPlan& P, const double* f, double* u, double tol, int maxit, int epoch, hipStream_t s);
// identity preconditioner: z = r (mode 0), or the MINRES set-up / Lanczos step with
// z = q and the partials of <q, q> (modes INV_GAMMA_INIT / INV_GAMMA_ITER)
hipError_t launch_identity(const DevPlan& P, int mode, const double* in, double* out, hipStream_t s);

// GMRES steps (kernels_gmres.hip); gslot(l) is the vector slot of Arnoldi vector v_l
enum GmresFin : int { G_INIT = 0, G_DOTS1 = 1, G_DOTS2 = 2, G_NORM = 3, G_CHECK = 4 };
hipError_t launch_ginit(const DevPlan& P, const double* f, double* u, hipStream_t s);
hipError_t launch_gdots(const DevPlan& P, int j, const double* w, hipStream_t s);
hipError_t launch_gaxpy(const DevPlan& P, int j, int pass, double* w, hipStream_t s);
hipError_t launch_gbase(const DevPlan& P, const double* src, const double* u, int restart_step, hipStream_t s);
hipError_t launch_gcomb(const DevPlan& P, int j, double* t, hipStream_t s);
hipError_t launch_gaddx(const DevPlan& P, double* u, const double* z, hipStream_t s);
__host__ __device__ inline double* gslot(const DevPlan& P, int l) { return l < kZSlots ? P.Z[l] : P.W[l - kZSlots]; }
static_assert(kGmresMax + 1 <= kZSlots + 2, "the Arnoldi basis must fit the Z and W slots");
// u (and at the flush w_j, w_{j-1}) from the resident basis, for right-hand sides whose
// scalar step set form_now
hipError_t launch_form(const DevPlan& P, double* u, hipStream_t s);
// one block per right-hand side: fixed-order sum of the partials of a reduction and
// the scalar step that consumes it
struct FinArgs {
  double tol = 0.0;            // FIN_BNORM
  int maxit = 0, epoch = 0;
  int post = 0;                // 1: FIN_GAMMA_ITER posts a snapshot, as the set-up and FIN_RES do; -1: none does
};
hipError_t launch_fin(const DevPlan& P, int kind, const FinArgs& a, hipStream_t s);
hipError_t launch_gfin(const DevPlan& P, int kind, const FinArgs& a, int restart, hipStream_t s);

// check: which right-hand sides the pass skips (PassCheck)
hipError_t launch_dstx_fwd(const DevPlan& P, int prec, int mode, int check, const double* in, hipStream_t s);
hipError_t launch_dsty(const DevPlan& P, int prec, int check, hipStream_t s);
// inv1 = 1: the single time pass of C_alpha^{-1} (mu^{-1}, no time reversal); with check
// (and inv1 = 0) the pass also writes the partials of <q, P^{-1} q> (PART_GAMMA, one
// per mode pair)
hipError_t launch_time(const DevPlan& P, int prec, int check, hipStream_t s, int inv1 = 0);
hipError_t launch_dstx_inv(const DevPlan& P, int prec, int mode, int check, double* out, hipStream_t s);
// fused 2D first / last pass (square grids whose level fits in LDS; P.wg_s != 0)
hipError_t launch_dst2_fwd(const DevPlan& P, int prec, int mode, int check, const double* in, hipStream_t s);
hipError_t launch_dst2_inv(const DevPlan& P, int prec, int mode, int check, double* out, hipStream_t s);
int slab_wg(int nx, int ny, int prec, int maxlds, size_t margin);
// dynamic LDS bytes of the fused 2D passes with workgroup wg (0 if not legal)
size_t slab_lds_bytes(int L, int wg, int prec);
// fused small-problem iteration (1D, nt * nx <= 4096; P.small != 0)
hipError_t launch_iter_small(const DevPlan& P, int prec, const double* f, double* u, hipStream_t s);
hipError_t launch_setup_small(const DevPlan& P, int prec, const double* f, double* u, const FinArgs& a, hipStream_t s);
hipError_t launch_solve_small(const DevPlan& P, int prec, const double* f, double* u, const FinArgs& a, hipStream_t s);
bool small_path_valid(int nx, int ny, int nt, int prec);
// transform kernel kinds (tile validity and LDS size differ per kind)
enum TransformKind : int { TK_XFWD = 0, TK_XINV = 1, TK_Y = 2, TK_TIME = 3 };
// dynamic LDS bytes of one workgroup (0 if the tile is not legal)
size_t transform_lds_bytes(int kind, int L, int wg, int prec);
bool transform_tile_valid(int kind, int L, int wg, int prec);
int transform_tps(int L, int prec);   // threads per sequence of length L (prec 1: FP32)

}  // namespace abac
