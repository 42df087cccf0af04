// rs_qp.hpp -- barrier-certificate QP of one environment, solved exactly by
// the lane group that owns it.
//
// Problem (control barrier certificate of JaxRobotarium Sec. 4.1, with the
// cubic class-K pairwise rows and wall rows defined in robostep.h):
//     min |u - u_nom|^2   s.t.  -2 D_ij.u_i + 2 D_ij.u_j <= gamma h_ij^3  (i<j)
//                               lo_i <= u_i <= hi_i                     (per coordinate)
// The minimiser is the Euclidean projection of u_nom onto a polytope, hence
// unique. It is found with a dual active-set method in the style of Goldfarb
// and Idnani (1983) specialised to the identity Hessian:
//   * bound rows are unit rows, so an active bound simply fixes its coordinate;
//     with up to four active pairwise rows S the Gram system over the free
//     coordinates, G_S = C_S^free C_S^free^T, is factored by Cholesky in
//     registers; beyond that the inverse Gram matrix of all active rows, bounds
//     among them, is kept in LDS (and what that does not solve is solved again
//     with the free coordinates' Gram system, factored in LDS);
//   * the start point clips u_nom to the box, which is exactly the state after
//     adding every violated bound (they are mutually orthogonal);
//   * each iteration adds the most violated row (normalised violation),
//     stepping along its component z orthogonal to the active set and
//     dropping an active row whose multiplier would turn negative.
// Rows that no point of the speed box can violate (4 v_max (|Dx|+|Dy|) <= b)
// are never examined: they are implied by the box, so the solution is
// unchanged.
//
// Work split inside the group: lane i owns robot i (its u, bounds, fixed
// flags and bound multipliers) and the pairs (i, i+k mod N), k = 1..N/2
// (k = N/2 only for i < N/2), so every pair has exactly one owner and the
// violation scan costs ceil((N-1)/2) rounds. The register loop's algebra is
// done identically by every lane of the group from group-uniform data; the
// general solver gives each lane two rows of the inverse.
#pragma once

#include <cstddef>

#include "rs_device.hpp"

namespace rs {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// One active row of the general solver, as a vector so that a lane reads it
// with one LDS access: {id, cx, cy, r}. Its coefficients are (-cx, -cy) at
// robot ra and (cx, cy) at robot rb, id = ra | rb << 8 (held as a number). A
// pair row has ra < rb and (cx, cy) = 2 D; an active bound has no second robot
// (rb = kNoRobot) and (cx, cy) = minus its unit normal. r is a work column:
// Gram products, then the multiplier direction.
template <typename T> struct QPRow {
  typedef T vec __attribute__((ext_vector_type(4)));
};
constexpr int kNoRobot = 255;
constexpr int kQR = 4;  // active rows that the register-resident solver holds

template <typename T, int G> struct alignas(4 * sizeof(T)) QPScratch {
  typename QPRow<T>::vec row[2 * G];  // active rows
  T lam[2 * G];                       // multipliers (objective 1/2 |u - u_nom|^2)
  T H[(2 * G) * (2 * G + 1) / 2];     // inverse Gram matrix of the rows (packed lower)
  T px[G], py[G];                     // projection points, for the out-of-line solvers
};
// The scratch as an LDS pointer: an out-of-line function that took a generic
// one would reach it by flat accesses, which also wait for the wavefront's
// outstanding global stores.
template <typename T, int G>
using LdsScratch = __attribute__((address_space(3))) QPScratch<T, G>;

__device__ __forceinline__ int tri(int a, int b) { return (a * (a + 1)) / 2 + b; }

// Index of pair (a, b), a < b, in lexicographic order.
__device__ __forceinline__ int pair_index(int a, int b, int N) {
  return a * (2 * N - a - 1) / 2 + (b - a - 1);
}

// min / max / |.| as single instructions (operands are never NaN here).
__device__ __forceinline__ float tmax(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ float tmin(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ double tmax(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ double tmin(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ float tfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double tfma(double a, double b, double c) { return __builtin_fma(a, b, c); }
// clamp to [lo, hi] with lo <= hi: one median-of-three in FP32
__device__ __forceinline__ float tclamp(float x, float lo, float hi) {
  return __builtin_amdgcn_fmed3f(x, lo, hi);
}
__device__ __forceinline__ double tclamp(double x, double lo, double hi) {
  return __builtin_fmin(__builtin_fmax(x, lo), hi);
}
__device__ __forceinline__ float tabs(float a) { return __builtin_fabsf(a); }
__device__ __forceinline__ double tabs(double a) { return __builtin_fabs(a); }
// Quotient used by the step-length and ratio tests of the solver: in FP32 a
// reciprocal (1 ulp) times the numerator, in FP64 the correctly rounded
// division.
__device__ __forceinline__ float qdiv(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ double qdiv(double a, double b) { return a / b; }
template <typename T> __device__ __forceinline__ T eps_v();  // spacing of the numbers at 1
template <> __device__ __forceinline__ float eps_v<float>() { return 1.1920929e-7f; }
template <> __device__ __forceinline__ double eps_v<double>() { return 2.220446049250313e-16; }
template <typename T> __device__ __forceinline__ T big_v();
template <> __device__ __forceinline__ float big_v<float>() { return 3.0e38f; }
template <> __device__ __forceinline__ double big_v<double>() { return 1.0e300; }

// Per-coordinate bounds: speed box intersected with the wall certificates of
// the projection point (walls pulled in by r_s / 2, gain c_b gamma, cubic).
template <typename T, typename CS>
__device__ __forceinline__ void wall_bounds(const CS &C, T px, T py, T &lox, T &hix,
                                            T &loy, T &hiy) {
  const T mxh = C.xwh - px, mxl = px - C.xwl;
  const T myh = C.ywh - py, myl = py - C.ywl;
  hix = tmin(C.vmax, C.kb * (mxh * mxh * mxh));
  lox = tmax(-C.vmax, -(C.kb * (mxl * mxl * mxl)));
  hiy = tmin(C.vmax, C.kb * (myh * myh * myh));
  loy = tmax(-C.vmax, -(C.kb * (myl * myl * myl)));
}

// Stage of the solver that produced the command.
enum : int {
  kStBox = 0,        // no row violated at the box clip u0
  kStOneRow = 1,     // one violated row: closed-form projection
  kStTwoRows = 2,    // two violated rows on four distinct robots
  kStShared = 3,     // two or three rows through shared robots (Gram system, no bound)
  kStActiveSet = 4,  // register-resident active-set loop
  kStGeneral = 5     // general active-set solver with its rows in LDS
};

struct QPInfo {
  int status;  // 0 solved, 1 infeasible, 2 iteration cap / numerical failure
  int iters;   // active-set iterations
  int q;       // active pairwise rows at exit
  int in_lds;  // nonzero: the general solver ran
  int stage;   // kSt*: the stage that produced the command
};

// Per-env certificate statistics (the qp_stats outputs): slots 0..5 count
// solves by the stage that produced the command, slot 6 infeasible solves,
// slot 7 solves stopped by the iteration cap or a numerical failure (neither
// of the last two is counted in 0..5), slot 8 the active-set iterations of
// the solves that ran the loop.
constexpr int kQPStats = 9;
__device__ __forceinline__ int qp_stat_slot(const QPInfo &q) {
  return q.status == 1 ? 6 : (q.status == 2 ? 7 : q.stage);
}
// Adds one solve to an env's counters (one lane of the group calls it).
__device__ __forceinline__ void qp_stats_add(int32_t *q, const QPInfo &info) {
  q[qp_stat_slot(info)] += 1;
  if (info.stage >= kStActiveSet) q[8] += info.iters;
}
// Always-on failure counters of a context: [0] infeasible, [1] capped.
__device__ __forceinline__ void qp_fail_count(unsigned long long *fail, const QPInfo &info) {
  if (fail && info.status != 0) atomicAdd(fail + (info.status - 1), 1ull);
}

// ---------------------------------------------------------------------------
// Register-resident solver (the hot path):
//  * the active pairwise rows live in kQR group-uniform register slots, so
//    the q x q Gram/Cholesky algebra is straight-line code on registers;
//  * a lane owns the pairs (i, (i+K) mod G), K = 1..G/2 (K = G/2 only for
//    i < G/2), whose geometry (D, b, 1/|c|) is computed once per solve from
//    DPP rotations of the projection points;
//  * every cross-lane quantity (argmax with the row's data as payload, |z|^2,
//    the violation of the entering row, the blocking step) is a DPP butterfly
//    over the group: no LDS traffic at all.
// When a row must enter while all slots are taken, the general solver carries
// on from there; when the Gram system loses positive definiteness, it starts
// again from the box clip.
// ---------------------------------------------------------------------------
template <typename T> struct QPActive {
  int q;
  int rows_in_lds;  // 1: the rows are in sh->row / sh->lam (active-set loops)
  int sa[kQR], sb[kQR];
  T slam[kQR];
};

template <int G, typename T>
__device__ __forceinline__ void gargmax_payload(T &v, int &id, T &p0, T &p1, T &p2) {
  auto step = [&](auto cc) {
    constexpr int CT = decltype(cc)::value;
    const T w = dpp<CT>(v), q0 = dpp<CT>(p0), q1 = dpp<CT>(p1), q2 = dpp<CT>(p2);
    const int j = dpp<CT>(id);
    if (w > v || (w == v && j < id)) { v = w; id = j; p0 = q0; p1 = q1; p2 = q2; }
  };
  step(std::integral_constant<int, 0xB1>{});
  if constexpr (G >= 4) step(std::integral_constant<int, 0x4E>{});
  if constexpr (G >= 8) step(std::integral_constant<int, 0x141>{});
  if constexpr (G >= 16) step(std::integral_constant<int, 0x140>{});
}

template <int G, typename T> __device__ __forceinline__ void gargmax(T &v, int &id) {
  auto step = [&](auto cc) {
    constexpr int CT = decltype(cc)::value;
    const T w = dpp<CT>(v);
    const int j = dpp<CT>(id);
    if (w > v || (w == v && j < id)) { v = w; id = j; }
  };
  step(std::integral_constant<int, 0xB1>{});
  if constexpr (G >= 4) step(std::integral_constant<int, 0x4E>{});
  if constexpr (G >= 8) step(std::integral_constant<int, 0x141>{});
  if constexpr (G >= 16) step(std::integral_constant<int, 0x140>{});
}

template <int G, typename T> __device__ __forceinline__ void gargmin(T &v, int &id) {
  auto step = [&](auto cc) {
    constexpr int CT = decltype(cc)::value;
    const T w = dpp<CT>(v);
    const int j = dpp<CT>(id);
    if (w < v || (w == v && j < id)) { v = w; id = j; }
  };
  step(std::integral_constant<int, 0xB1>{});
  if constexpr (G >= 4) step(std::integral_constant<int, 0x4E>{});
  if constexpr (G >= 8) step(std::integral_constant<int, 0x141>{});
  if constexpr (G >= 16) step(std::integral_constant<int, 0x140>{});
}

// Lane of the group holding the largest positive score (ties: smaller lane),
// or -1 if no lane has one. A non-negative float orders like its bit pattern
// read as an unsigned integer, so the score's bits, truncated by one byte,
// carry 255 - lane in the low byte and a single unsigned-max butterfly
// decides; the caller then reads the winner's payload from its lane.
template <int G, typename T>
__device__ __forceinline__ int group_argmax_lane(T score, bool has, int i) {
  const uint32_t key0 =
      has ? ((__float_as_uint((float)score) & 0xFFFFFF00u) | (uint32_t)(255 - i)) : 0u;
  const int key = gred<G>((int)key0, [](int a, int b) { return (uint32_t)a > (uint32_t)b ? a : b; });
  return key == 0 ? -1 : 255 - (key & 255);
}

// Owner lane and rotation of pair (a, b), a < b, under the mod-G ownership.
template <int G> __device__ __forceinline__ void pair_owner_g(int a, int b, int &owner, int &k) {
  const int d = b - a;
  if (2 * d <= G) { owner = a; k = d; }
  else { owner = b; k = G - d; }
}

// Result of the active-set loop: six values, so that it comes back in
// registers (a larger result would travel through scratch memory, and
// reading it back would wait for every outstanding store of the wavefront).
template <typename T> struct QPLoopOut {
  T ux, uy;
  int status, iters, q;
  int in_lds;  // the general solver ran: 1 from the clip, 2 from the loop's active set,
               // 3 without an answer
};

// General solver: the dual active-set method for any number of active rows,
// bounds and pairs alike (at most 2N rows are independent). The inverse H of
// the active rows' Gram matrix is kept explicitly in LDS (packed symmetric):
// lane i of the group owns slots i and i + G, so the multiplier direction
// r = H (C c_p) is one row product per lane with no serial substitution, a row
// entering is a rank-one update of H (its Schur complement is |z|^2) and a row
// leaving another; the last slot then moves into the gap. It is bound by the
// latency of its few hundred instructions and six LDS round trips a step, in
// the few wavefronts that need it. Refactoring the Gram system serially on
// every step instead, from scratch, took 1.53 ms for one env_step of 16384
// envs x 16 robots, a dense eighth of them, and 0.32 ms for 8192 x 12
// certificates; this takes 0.19 and 0.06 ms.
//
// Explicit updates of H lose digits over many steps, so once no row is
// violated the command and the multipliers are formed again from the active
// rows (one residual correction with H, which leaves rounding of the residual
// itself) and scanned again; a correction that does not close the residual
// rebuilds H from the rows.
//
// Entry (handover, written by the register loop): the problem and the
// active bounds of every lane, and with `carry` the loop's q0 pair rows, the
// entering row and its multiplier; (ux, uy) is the command of that active
// set. Without `carry` it starts from the box clip. `iters` counts on from the
// caller's. Every lane of the group calls it together; the rows stay in
// sh->row / sh->lam.
// What the register loop leaves in the group's scratch for the general solver:
// ten values per lane at the end of H (value c of lane i at c * G + i) beside
// the projection points and, ahead of them, rows 0..3 {id, cx, cy,
// multiplier}, row 4 the entering row {id, cx, cy, rhs} and its multiplier. With the problem in LDS the register
// loop can end in a tail call of the general solver, which leaves it a leaf
// function: as an ordinary caller it saved more registers on every entry (1%
// of the headline rollout's time), and a second call site in the step loop
// cost that loop 2 to 4%.
// The general solver leaves the first six of them for qp_factored in the same
// way, clear of all rows.
constexpr int kHandover = 10, kHandback = 6;
template <int VALUES, typename T, int G>
__device__ __forceinline__ __attribute__((address_space(3))) T *handover(LdsScratch<T, G> *sh) {
  typedef QPScratch<T, G> Scratch;
  constexpr int end = offsetof(Scratch, px) / sizeof(T);
  static_assert(end >= VALUES * G && (G == 2 || end >= 24 + VALUES * G), "row 5 stays clear");
  static_assert(VALUES > kHandback || end >= (2 * G) * 4 + VALUES * G, "all rows stay clear");
  return (__attribute__((address_space(3))) T *)sh->px - VALUES * G;
}

template <typename T, int G>
__device__ __forceinline__ void qp_general_solve(LdsScratch<T, G> *sh, int lane, int N, bool carry,
                                                 QPLoopOut<T> &out, T rs2, T gamma, T vmax4,
                                                 T tol_add, T eps_z, T eps_r, int qp_cap,
                                                 typename QPRow<T>::vec &enter) {
  constexpr int KH = G / 2;
  constexpr int S = 2;  // slots per lane: i and i + G
  const T BIG = big_v<T>();
  typedef typename QPRow<T>::vec Row;
  typedef __attribute__((address_space(3))) Row LdsRow;
  typedef __attribute__((address_space(3))) T LdsT;
  LdsRow *rows = sh->row;
  LdsT *lam = sh->lam, *H = sh->H;
  auto work = [&](int k) -> LdsT & { return ((LdsT *)(rows + k))[3]; };
  const int i = lane & (G - 1);
  const bool on = i < N;
  const int gbase = lane & ~(G - 1);
  const int cap = qp_cap > 0 ? qp_cap : 8 * N + 32;
  // --- what the register loop left ---------------------------------------------
  const LdsT *hv = handover<kHandover>(sh) + i;
  const T px = sh->px[i], py = sh->py[i], uhx = hv[0], uhy = hv[G];
  const T lox = hv[2 * G], hix = hv[3 * G], loy = hv[4 * G], hiy = hv[5 * G];
  int fx = (int)hv[6 * G], fy = (int)hv[7 * G];
  T mux = hv[8 * G], muy = hv[9 * G];
  Row p = (Row){T(0), T(0), T(0), T(0)};  // the entering row
  T lam_p = T(0), hl = T(0);              // its multiplier; lane k < 4: row k's
  if constexpr (G > 2) {
    if (carry) {
      p = rows[kQR];
      lam_p = ((LdsT *)(rows + kQR + 1))[0];
      hl = work(i & (kQR - 1));
    }
  }
  T ux = out.ux, uy = out.uy;
  int q0 = out.q;
  const int iters0 = carry ? 0 : out.iters;  // of the abandoned attempt
  out.iters -= iters0;
  if (!carry) {  // the box clip, its active bounds fixing their coordinate
    q0 = 0;
    ux = uhx;
    uy = uhy;
    fx = fy = 0;
    mux = muy = T(0);
    if (on) {
      if (uhx > hix) { ux = hix; fx = 1; mux = uhx - hix; }
      else if (uhx < lox) { ux = lox; fx = -1; mux = lox - uhx; }
      if (uhy > hiy) { uy = hiy; fy = 1; muy = uhy - hiy; }
      else if (uhy < loy) { uy = loy; fy = -1; muy = loy - uhy; }
    }
  }
  wave_lds_fence();
  if (i < q0) lam[i] = hl;
  // --- geometry of the owned pairs (the scan's formulas) ----------------------
  T cdx[KH], cdy[KH], cb[KH], crn[KH];
  uint32_t open_k = 0;  // bit K: my rotation-K pair can be violated and is not active
  static_for<1, KH + 1>([&](auto kc) {
    constexpr int K = decltype(kc)::value;
    const T pxj = grot<G, K>(px, lane), pyj = grot<G, K>(py, lane);
    const int j = (i + K) & (G - 1);
    const bool valid = on && j < N && !(2 * K == G && i >= KH);
    const bool ia = i < j;
    const T dx = ia ? px - pxj : pxj - px;
    const T dy = ia ? py - pyj : pyj - py;
    const T d2 = dx * dx + dy * dy;
    const T h = d2 - rs2;
    const T bb = gamma * (h * h * h);
    const bool cand = valid && (vmax4 * (tabs(dx) + tabs(dy)) > bb);
    cdx[K - 1] = dx;
    cdy[K - 1] = dy;
    cb[K - 1] = bb;
    crn[K - 1] = d2 > T(0) ? T(0.35355339059327373) * rsqrt_t(d2) : T(0);
    if (cand && d2 > T(0)) open_k |= 1u << K;
  });

  // --- active bounds into the slots after the pairs, then H row by row --------
  int q;
  {
    const uint32_t bx = group_bits<G>(__ballot(fx != 0), lane);
    const uint32_t by = group_bits<G>(__ballot(fy != 0), lane);
    const uint32_t below = (1u << i) - 1u;
    const int qx = q0 + __popc(bx);
    const int sx = q0 + __popc(bx & below), sy = qx + __popc(by & below);
    q = qx + __popc(by);
    if (fx != 0 && q <= 2 * G) {
      rows[sx] = (Row){T(i | kNoRobot << 8), T(-fx), T(0), T(0)};
      lam[sx] = mux;
    }
    if (fy != 0 && q <= 2 * G) {
      rows[sy] = (Row){T(i | kNoRobot << 8), T(0), T(-fy), T(0)};
      lam[sy] = muy;
    }
    wave_lds_fence();
    for (int s = 0; s < q0; ++s) {
      const int id = (int)rows[s].x;
      int owner, kk;
      pair_owner_g<G>(id & 255, id >> 8, owner, kk);
      if (i == owner) open_k &= ~(1u << kk);
    }
  }
  // product of H's row k with the work column of the first n rows
  auto hdot = [&](int k, int n) {
    T acc = T(0);
    int idx = tri(k, 0);
#pragma unroll 4
    for (int b = 0; b < n; ++b) {
      acc += H[idx] * work(b);
      idx += b < k ? 1 : b + 1;
    }
    return acc;
  };
  // r = H (C c) over the first n rows for the row (ra, rb, cx, cy); r is left
  // in the work column and, for my slots, in rk; (zx, zy): the part of the
  // row orthogonal to them at my robot, zz = |z|^2
  T rk[S];
  auto direction = [&](int n, int ra, int rb, T cx, T cy, T &zx, T &zy, T &zz) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = i + s * G;
      if (k < n) {
        const Row w = rows[k];
        const int wa = (int)w.x & 255, wb = (int)w.x >> 8;
        const int m = (wa == ra) - (wa == rb) - (wb == ra) + ((wb == rb) & (wb != kNoRobot));
        work(k) = T(m) * (w.y * cx + w.z * cy);
      }
    }
    wave_lds_fence();
#pragma unroll
    for (int s = 0; s < S; ++s) rk[s] = i + s * G < n ? hdot(i + s * G, n) : T(0);
    wave_lds_fence();
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (i + s * G < n) work(i + s * G) = rk[s];
    wave_lds_fence();
    const int sg = (i == rb) - (i == ra);
    zx = T(sg) * cx;
    zy = T(sg) * cy;
#pragma unroll 4
    for (int a = 0; a < n; ++a) {
      const Row w = rows[a];
      const T f = T((i == ((int)w.x >> 8)) - (i == ((int)w.x & 255))) * w.w;
      zx -= f * w.y;
      zy -= f * w.z;
    }
    zz = gsum<G>(zx * zx + zy * zy);
  };
  // H of n rows -> n + 1 rows, from r (rk, work column) and zz of the new one
  auto grow = [&](int n, T zz) {
    const T iz = T(1) / zz;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = i + s * G;
      if (k < n) {
        const T f = rk[s] * iz;
#pragma unroll 4
        for (int b = 0; b <= k; ++b) H[tri(k, b)] += f * work(b);
        H[tri(n, k)] = -f;
      }
    }
    if (i == 0) H[tri(n, n)] = iz;
    wave_lds_fence();
  };
  // H of the first n rows of the table; false when one depends on the others
  auto rebuild = [&](int n) {
    bool indep = true;
    for (int s = 0; s < n && indep; ++s) {
      const Row w = rows[s];
      const int wb = (int)w.x >> 8;
      T zx, zy, zz;
      direction(s, (int)w.x & 255, wb, w.y, w.z, zx, zy, zz);
      const T n2 = (wb == kNoRobot ? T(1) : T(2)) * (w.y * w.y + w.z * w.z);
      indep = zz > T(0.01) * eps_z * n2;
      if (indep) grow(s, zz);
    }
    return indep;
  };
  // command and multipliers from the active rows: one correction of the
  // multipliers by H times the rows' residuals. Returns the largest residual
  // over its row's norm that was left after it, and in `size` the largest sum
  // of magnitudes that a robot's command was formed from: a residual cannot
  // fall below its rounding, in whatever unit the speeds are. (One sum, formed
  // beside the command: the solver's registers are counted. Beyond 194 of them
  // at 8 lanes the Predator-Prey rollouts spill more in their step loop, 200
  // took 6% off 16384 x 6; beyond 256 at 16 lanes a SIMD holds one wavefront,
  // which took 50% off 16384 x 16 steps.)
  auto refine = [&](T &size) {
    T left = T(0);
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (i + s * G < q) work(i + s * G) = lam[i + s * G];
      wave_lds_fence();
      T vx = uhx, vy = uhy, mag = tabs(uhx) + tabs(uhy);
#pragma unroll 4
      for (int a = 0; a < q; ++a) {
        const Row w = rows[a];
        const T f = T((i == ((int)w.x >> 8)) - (i == ((int)w.x & 255))) * w.w;
        vx -= f * w.y;
        vy -= f * w.z;
        mag += tabs(f) * (tabs(w.y) + tabs(w.z));
      }
      size = on ? mag : T(0);
      ux = on ? vx : ux;
      uy = on ? vy : uy;
      const T bx = fx > 0 ? hix : lox, by = fy > 0 ? hiy : loy;
      T e[S], worst = T(0);
      wave_lds_fence();
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int k = i + s * G;
        const Row w = rows[k < q ? k : 0];
        const int ra = (int)w.x & 255, rb = (int)w.x >> 8;
        const bool bound = rb == kNoRobot;
        const int la = gbase + (ra & (G - 1)), lb = gbase + (rb & (G - 1));
        const T uax = __shfl(ux, la, 64), uay = __shfl(uy, la, 64);
        const T ubx = __shfl(ux, lb, 64), uby = __shfl(uy, lb, 64);
        const T bax = __shfl(bx, la, 64), bay = __shfl(by, la, 64);
        const T d2 = T(0.25) * (w.y * w.y + w.z * w.z);
        const T h = d2 - rs2;
        const T beta = gamma * (h * h * h);
        e[s] = bound ? w.y * (bax - uax) + w.z * (bay - uay)
                     : w.y * (ubx - uax) + w.z * (uby - uay) - beta;
        e[s] = k < q ? e[s] : T(0);
        const T rn = bound ? T(1) : T(0.35355339059327373) * rsqrt_t(d2);  // 1 / |c|
        worst = tmax(worst, k < q ? tabs(e[s]) * rn : T(0));
      }
      left = gmax<G>(worst);
      if (pass == 1) break;
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (i + s * G < q) work(i + s * G) = e[s];
      wave_lds_fence();
      T dl[S];
#pragma unroll
      for (int s = 0; s < S; ++s) dl[s] = i + s * G < q ? hdot(i + s * G, q) : T(0);
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (i + s * G < q) lam[i + s * G] += dl[s];
      wave_lds_fence();
    }
    if (fx != 0) ux = fx > 0 ? hix : lox;
    if (fy != 0) uy = fy > 0 ? hiy : loy;
    size = gmax<G>(size);
    return left;
  };

  bool dead = false;
  bool settled = false;  // the command was formed from the rows since they last changed
  // H has to be formed from the rows: at entry, and when a correction did not
  // close the residual (again: it was formed for that). One place each for
  // rebuild() and refine(): the solver is called from kernels that fill the
  // instruction cache, and its size shows in their time.
  bool stale = true, again = false;
  // the entering row (its id as the table holds it): a pair or a bound
  bool pend = carry;
  int rid = (int)p.x;
  T cx = p.y, cy = p.z, rhs = p.w;
  while (true) {
    if (stale) {
      if (q > 2 * G || !rebuild(q)) { out.status = 2; break; }
      stale = false;
    }
    if (!pend) {
      // --- most violated row (normalised), its data as the argmax's payload ---
      T best = tol_add, bcx = T(0), bcy = T(0), bb = T(0);
      int bid = -1;  // pair: a << 4 | b; bound: 256 + 4 robot + 2 coordinate + lower
      if (on) {
        if (fx == 0) {
          const T su = ux - hix, sl = lox - ux;
          if (su > best) { best = su; bid = 256 + 4 * i; }
          else if (sl > best) { best = sl; bid = 256 + 4 * i + 1; }
        }
        if (fy == 0) {
          const T su = uy - hiy, sl = loy - uy;
          if (su > best) { best = su; bid = 256 + 4 * i + 2; }
          else if (sl > best) { best = sl; bid = 256 + 4 * i + 3; }
        }
        if (bid >= 0) {
          const T sg = (bid & 1) ? T(1) : T(-1);  // minus the unit normal
          bcx = (bid & 2) ? T(0) : sg;
          bcy = (bid & 2) ? sg : T(0);
          bb = (bid & 2) ? ((bid & 1) ? -loy : hiy) : ((bid & 1) ? -lox : hix);
        }
      }
      int bk = 0;
      static_for<1, KH + 1>([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        const T uxj = grot<G, K>(ux, lane), uyj = grot<G, K>(uy, lane);
        if ((open_k >> K) & 1u) {
          const bool ia = i < ((i + K) & (G - 1));
          const T dux = ia ? uxj - ux : ux - uxj;
          const T duy = ia ? uyj - uy : uy - uyj;
          const T sn = (T(2) * (cdx[K - 1] * dux + cdy[K - 1] * duy) - cb[K - 1]) * crn[K - 1];
          if (sn > best) {
            best = sn;
            bk = K;
            bcx = T(2) * cdx[K - 1];
            bcy = T(2) * cdy[K - 1];
            bb = cb[K - 1];
          }
        }
      });
      if (bk > 0) {
        const int j = (i + bk) & (G - 1);
        bid = min(i, j) << 4 | max(i, j);
      }
      gargmax_payload<G>(best, bid, bcx, bcy, bb);
      if (bid < 0) {
        // a command that is not finite violates no row either, and leaves no
        // residual that a maximum shows
        if (group_any<G>(!(tabs(ux) + tabs(uy) < BIG), lane)) { out.status = 2; break; }
        if (settled) break;  // optimal
        T size;
        const T left = refine(size);
        const T close = tol_add + T(8) * eps_v<T>() * size;
        settled = left <= (again ? T(8) * close : close);
        if (!settled && again) { out.status = 2; break; }
        stale = again = !settled;
        continue;
      }
      if (++out.iters > cap) { out.status = 2; break; }
      rid = bid < 256 ? bid >> 4 | (bid & 15) << 8 : (bid - 256) >> 2 | kNoRobot << 8;
      cx = bcx;
      cy = bcy;
      rhs = bb;
      lam_p = T(0);
      pend = true;
    }
    // --- one step toward the entering row -------------------------------------
    const int ra = rid & 255, rb = rid >> 8;
    const bool p_pair = rb != kNoRobot;
    T zx, zy, zz;
    direction(q, ra, rb, cx, cy, zx, zy, zz);
    const int sg = (i == rb) - (i == ra);
    const T sp = gsum<G>(on ? T(sg) * (cx * ux + cy * uy) : T(0)) - rhs;
    // blocking row: the first active multiplier to reach zero
    T t1 = BIG;
    int drop = -1;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = i + s * G;
      const T ratio = k < q ? qdiv(lam[k], rk[s]) : T(0);
      const bool ok = k < q && rk[s] > eps_r && ratio < t1;
      t1 = ok ? ratio : t1;
      drop = ok ? k : drop;
    }
    gargmin<G>(t1, drop);
    const T n2 = (p_pair ? T(2) : T(1)) * (cx * cx + cy * cy);
    const bool z_ok = zz > eps_z * n2;
    const T t2 = z_ok ? qdiv(sp, zz) : BIG;
    if (drop < 0 && !z_ok) { dead = true; break; }  // no step can restore the row
    const bool full = z_ok && (drop < 0 || t2 <= t1);
    const T t = full ? t2 : t1;
    if (full && q == 2 * G) { out.status = 2; break; }
    if (z_ok) {
      ux -= t * zx;
      uy -= t * zy;
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (i + s * G < q) lam[i + s * G] -= t * rk[s];
    lam_p += t;
    settled = again = false;
    if (full) {
      grow(q, zz);
      if (i == 0) {
        rows[q] = (Row){T(rid), cx, cy, T(0)};
        lam[q] = lam_p;
      }
      wave_lds_fence();
      ++q;
      if (p_pair) {
        int owner, kk;
        pair_owner_g<G>(ra, rb, owner, kk);
        if (i == owner) open_k &= ~(1u << kk);
      } else if (i == ra) {
        // (cx, cy) is minus the normal: negative at an upper bound
        if (cx != T(0)) { fx = cx < T(0) ? 1 : -1; ux = cx < T(0) ? hix : lox; }
        else { fy = cy < T(0) ? 1 : -1; uy = cy < T(0) ? hiy : loy; }
      }
      pend = false;
    } else {
      // --- release slot `drop`; the last slot takes its place ------------------
      const Row w = rows[drop];
      const int wa = (int)w.x & 255, wb = (int)w.x >> 8;
      if (wb == kNoRobot) {
        if (i == wa) {
          if (w.y != T(0)) fx = 0; else fy = 0;
        }
      } else {
        int owner, kk;
        pair_owner_g<G>(wa, wb, owner, kk);
        if (i == owner) open_k |= 1u << kk;
      }
      const int last = q - 1;
      const T ihd = T(1) / H[tri(drop, drop)];
      T hk[S];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int k = i + s * G;
        hk[s] = k < q ? H[k >= drop ? tri(k, drop) : tri(drop, k)] : T(0);
      }
      wave_lds_fence();
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (i + s * G < q) work(i + s * G) = hk[s];
      wave_lds_fence();
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int k = i + s * G;
        if (k < q) {
          const T f = hk[s] * ihd;
#pragma unroll 4
          for (int b = 0; b <= k; ++b) H[tri(k, b)] -= f * work(b);
        }
      }
      wave_lds_fence();
      if (drop != last) {
        T mv[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int k = i + s * G;
          mv[s] = k < last ? H[k == drop ? tri(last, last) : tri(last, k)] : T(0);
        }
        wave_lds_fence();
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int k = i + s * G;
          if (k < last) H[k >= drop ? tri(k, drop) : tri(drop, k)] = mv[s];
        }
        if (i == 0) {
          rows[drop] = rows[last];
          lam[drop] = lam[last];
        }
        wave_lds_fence();
      }
      q = last;
    }
    if (++out.iters > cap) { out.status = 2; break; }
  }

  if (dead) {
    out.status = 1;
    if (on) {
      ux = lox <= hix ? tmin(tmax(uhx, lox), hix) : T(0.5) * (lox + hix);
      uy = loy <= hiy ? tmin(tmax(uhy, loy), hiy) : T(0.5) * (loy + hiy);
    }
  }
  if (out.status != 0) {  // for qp_factored to confirm
    LdsT *hw = handover<kHandback>(sh) + i;
    wave_lds_fence();
    const T v[kHandback] = {uhx, uhy, lox, hix, loy, hiy};
#pragma unroll
    for (int c = 0; c < kHandback; ++c) hw[c * G] = v[c];
    wave_lds_fence();
    out.in_lds = 3;
    enter = (Row){T(rid), cx, cy, T(0)};
  }
  out.ux = ux;
  out.uy = uy;
  out.q = q;
  out.iters += iters0;
}

// The dual active-set method once more, from the box clip, with the Gram system
// of the active pair rows over the coordinates that no active bound fixes,
// factored anew on every step (column by column, each lane two rows): for what
// the general solver did not solve. Its inverse holds the bounds as rows
// of their own, so a pair row of which the bounds leave only a sliver (two
// robots held along their line of centres, met by the small component across
// it) is too close to dependent on them; without the bounds it is an ordinary
// row. An overlapping pair held at the walls, met by 4e-6 m/s across: called
// infeasible in FP32 below 3e-5 rad off the axis without this.
// A verdict of "infeasible" stands unless such a row (free in less of its squared
// norm than some hundred units of rounding) is among the active ones or
// entering; "not solved" never does. It is bound by the latency of a solve's
// 50 to 100 steps, each of q^2 / 2 fused products and 3q LDS round trips (6000
// strewn envs of 16 robots, FP32, with a few such solves among them: 1.16 ms,
// 2.73 with every lane factoring the whole system). Signature and `packed` as qp_general;
// groups whose in_lds is not 3 pass through. fpb, fdx, fdy: the row that could
// not enter.
template <typename T, int G>
__device__ __noinline__ QPLoopOut<T> qp_factored(LdsScratch<T, G> *sh, int lane, int packed, int N,
                                                 bool on, T px, T py, T ux, T uy, T lox, T hix,
                                                 T loy, T hiy, bool seed, int iters, int fpb, T fl1,
                                                 T fdx, T fdy, T rs2, T gamma, T vmax4, T tol_add,
                                                 T eps_z, T eps_r, int qp_cap, bool want_rows) {
  typedef typename QPRow<T>::vec Row;
  typedef __attribute__((address_space(3))) Row LdsRow;
  typedef __attribute__((address_space(3))) T LdsT;
  constexpr int S = 2;  // rows per lane: i and i + G
  const T BIG = big_v<T>();
  LdsRow *rows = sh->row;
  LdsT *lam = sh->lam, *L = sh->H;
  auto work = [&](int k) -> LdsT & { return ((LdsT *)(rows + k))[3]; };
  const int i = lane & (G - 1), base = lane & ~(G - 1);
  const int cap = qp_cap > 0 ? qp_cap : 8 * N + 32;
  on = i < N;
  QPLoopOut<T> out{ux, uy, (packed >> 8) & 255, iters, packed >> 16, packed & 255};
  bool solve = out.in_lds == 3;
  // the part of robot r's (xx, yy) along the coordinates whose bits are set
  auto over = [](uint32_t x, uint32_t y, int r, T xx, T yy) {
    return ((x >> r) & 1u ? xx : T(0)) + ((y >> r) & 1u ? yy : T(0));
  };
  if (solve && out.status == 1) {
    uint32_t freex = ~0u, freey = ~0u;
    auto row = [&](int k) { return k < out.q ? rows[k] : (Row){T(fpb), fdx, fdy, T(0)}; };
    for (int k = 0; k <= out.q; ++k) {
      const Row w = row(k);
      if ((int)w.x >> 8 == kNoRobot) {
        const uint32_t bit = ~(1u << ((int)w.x & 255));
        if (w.y != T(0)) freex &= bit;
        else freey &= bit;
      }
    }
    solve = false;
    for (int k = 0; k <= out.q; ++k) {
      const Row w = row(k);
      if ((int)w.x >> 8 == kNoRobot) continue;
      const T xx = w.y * w.y, yy = w.z * w.z;
      const T left = over(freex, freey, (int)w.x & 255, xx, yy) +
                     over(freex, freey, (int)w.x >> 8, xx, yy);
      solve = solve || (left > T(0) && left < T(200) * eps_v<T>() * (xx + yy));  // |c|^2 / 2
    }
    out.q = 0;
  }
  if (solve) {
    const LdsT *hv = handover<kHandback>(sh) + i;
    px = sh->px[i];
    py = sh->py[i];
    const T uhx = hv[0], uhy = hv[G];
    lox = hv[2 * G]; hix = hv[3 * G]; loy = hv[4 * G]; hiy = hv[5 * G];
    wave_lds_fence();
    int fx = 0, fy = 0;  // +1 fixed at upper, -1 fixed at lower
    T mux = T(0), muy = T(0);
    ux = uhx;
    uy = uhy;
    if (on) {
      if (uhx > hix) { ux = hix; fx = 1; mux = uhx - hix; }
      else if (uhx < lox) { ux = lox; fx = -1; mux = lox - uhx; }
      if (uhy > hiy) { uy = hiy; fy = 1; muy = uhy - hiy; }
      else if (uhy < loy) { uy = loy; fy = -1; muy = loy - uhy; }
    }
    int q = 0, steps = 0, status = 0;
    uint32_t own_act = 0;  // bit K: my rotation-K pair is active
    bool dead = false;
    while (!dead && status == 0) {
      // --- most violated row (normalised) --------------------------------------
      T best = tol_add;
      int bid = -1;  // pair: a << 4 | b; bound: 256 + 4 robot + 2 coordinate + lower
      if (on) {
        if (fx == 0) {
          const T su = ux - hix, sl = lox - ux;
          if (su > best) { best = su; bid = 256 + 4 * i; }
          else if (sl > best) { best = sl; bid = 256 + 4 * i + 1; }
        }
        if (fy == 0) {
          const T su = uy - hiy, sl = loy - uy;
          if (su > best) { best = su; bid = 256 + 4 * i + 2; }
          else if (sl > best) { best = sl; bid = 256 + 4 * i + 3; }
        }
      }
      for (int K = 1; K <= G / 2; ++K) {
        const int j = (i + K) & (G - 1);
        const T pxj = __shfl(px, base + j, 64), pyj = __shfl(py, base + j, 64);
        const T uxj = __shfl(ux, base + j, 64), uyj = __shfl(uy, base + j, 64);
        if (on && j < N && !(2 * K == G && i >= K) && !((own_act >> K) & 1u)) {
          const bool ia = i < j;
          const T dx = ia ? px - pxj : pxj - px, dy = ia ? py - pyj : pyj - py;
          const T d2 = dx * dx + dy * dy;
          const T h = d2 - rs2;
          const T bb = gamma * (h * h * h);
          if (d2 > T(0) && vmax4 * (tabs(dx) + tabs(dy)) > bb) {
            const T dux = ia ? uxj - ux : ux - uxj, duy = ia ? uyj - uy : uy - uyj;
            const T sn = (T(2) * (dx * dux + dy * duy) - bb) * (T(0.35355339059327373) * rsqrt_t(d2));
            if (sn > best) { best = sn; bid = min(i, j) << 4 | max(i, j); }
          }
        }
      }
      gargmax<G>(best, bid);
      if (bid < 0) {  // optimal
        if (group_any<G>(!(tabs(ux) + tabs(uy) < BIG), lane)) status = 2;
        break;
      }
      if (++steps > cap) { status = 2; break; }
      // the entering row: coefficients (-cx, -cy) at robot pa, (cx, cy) at pb; a
      // bound: minus its unit normal, pb = kNoRobot
      const bool pair = bid < 256;
      const int pa = pair ? bid >> 4 : (bid - 256) >> 2, pb = pair ? bid & 15 : kNoRobot;
      T cx, cy, rhs;
      {
        const int jb = base + (pair ? pb : pa);
        const T dx = __shfl(px, base + pa, 64) - __shfl(px, jb, 64);
        const T dy = __shfl(py, base + pa, 64) - __shfl(py, jb, 64);
        const T h = dx * dx + dy * dy - rs2;
        const T lim = (bid & 2) ? ((bid & 1) ? -loy : hiy) : ((bid & 1) ? -lox : hix);
        const T blim = __shfl(lim, base + pa, 64);
        const T sg = (bid & 1) ? T(1) : T(-1);
        cx = pair ? T(2) * dx : ((bid & 2) ? T(0) : sg);
        cy = pair ? T(2) * dy : ((bid & 2) ? sg : T(0));
        rhs = pair ? gamma * (h * h * h) : blim;
      }
      T lam_p = T(0);
      bool added = false;
      while (!added) {
        const uint32_t freex = ~group_bits<G>(__ballot(fx != 0), lane);
        const uint32_t freey = ~group_bits<G>(__ballot(fy != 0), lane);
        // product of two rows over the free coordinates
        auto gram = [&](Row s, int ta, int tb, T tx, T ty) {
          const int sa = (int)s.x & 255, sb = (int)s.x >> 8;
          const T xx = s.y * tx, yy = s.z * ty;
          T acc = T(0);
          if (sa == ta) acc += over(freex, freey, sa, xx, yy);
          if (sa == tb) acc -= over(freex, freey, sa, xx, yy);
          if (sb == ta) acc -= over(freex, freey, sb, xx, yy);
          if (sb == tb) acc += over(freex, freey, sb, xx, yy);
          return acc;
        };
        // Cholesky factor of the active rows, column by column, my rows i and i + G
        bool chol_ok = true;
        for (int b = 0; b < q && chol_ok; ++b) {
          const Row w = rows[b];
          T v[S], d = T(0);
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const int a = i + s * G;
            v[s] = T(0);
            if (a >= b && a < q) {
              v[s] = gram(rows[a], (int)w.x & 255, (int)w.x >> 8, w.y, w.z);
              for (int k = 0; k < b; ++k) v[s] -= L[tri(a, k)] * L[tri(b, k)];
            }
            d = b / G == s ? v[s] : d;
          }
          d = __shfl(d, base + (b & (G - 1)), 64);
          chol_ok = d > T(0);
          const T root = sqrt_t(d);
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const int a = i + s * G;
            if (a >= b && a < q) L[tri(a, b)] = a == b ? root : v[s] / root;
          }
          wave_lds_fence();
        }
        if (!chol_ok) { status = 2; break; }
        // r = G^-1 (C c): my rows' values in g, the solved one passed round; r is
        // left in the work column
        T g[S];
#pragma unroll
        for (int s = 0; s < S; ++s)
          g[s] = i + s * G < q ? gram(rows[i + s * G], pa, pb, cx, cy) : T(0);
        auto solved = [&](int a) {
          return __shfl(a < G ? g[0] : g[S - 1], base + (a & (G - 1)), 64) / L[tri(a, a)];
        };
        for (int a = 0; a < q; ++a) {
          const T x = solved(a);
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const int k = i + s * G;
            if (k == a) g[s] = x;
            else if (k > a && k < q) g[s] -= L[tri(k, a)] * x;
          }
        }
        for (int a = q - 1; a >= 0; --a) {
          const T x = solved(a);
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const int k = i + s * G;
            if (k == a) g[s] = x;
            else if (k < a) g[s] -= L[tri(a, k)] * x;
          }
        }
        wave_lds_fence();
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (i + s * G < q) work(i + s * G) = g[s];
        wave_lds_fence();
        // the row less its part in the active ones, at my robot: along free
        // coordinates the step, along fixed ones the change of my bounds
        const int sg = (i == pb) - (i == pa);
        T zx = T(sg) * cx, zy = T(sg) * cy;
        for (int a = 0; a < q; ++a) {
          const Row w = rows[a];
          const T f = T((i == ((int)w.x >> 8)) - (i == ((int)w.x & 255))) * w.w;
          zx -= f * w.y;
          zy -= f * w.z;
        }
        if (!on) zx = zy = T(0);
        const T rfx = T(fx) * zx, rfy = T(fy) * zy;
        zx = fx == 0 ? zx : T(0);
        zy = fy == 0 ? zy : T(0);
        const T zz = gsum<G>(zx * zx + zy * zy);
        const T xx = cx * cx, yy = cy * cy;
        const T n2 = over(freex, freey, pa, xx, yy) + (pair ? over(freex, freey, pb, xx, yy) : T(0));
        const T sp = gsum<G>(on ? T(sg) * (cx * ux + cy * uy) : T(0)) - rhs;
        // blocking row: the first active multiplier to reach zero
        T t1 = BIG;
        int drop = -1;  // pair slot, or 1024 + 2 robot + coordinate
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int k = i + s * G;
          const T ratio = k < q ? qdiv(lam[k], g[s]) : T(0);
          if (k < q && g[s] > eps_r && ratio < t1) { t1 = ratio; drop = k; }
        }
        if (rfx > eps_r) {
          const T ratio = qdiv(mux, rfx);
          if (ratio < t1) { t1 = ratio; drop = 1024 + 2 * i; }
        }
        if (rfy > eps_r) {
          const T ratio = qdiv(muy, rfy);
          if (ratio < t1) { t1 = ratio; drop = 1024 + 2 * i + 1; }
        }
        gargmin<G>(t1, drop);
        const bool z_ok = zz > eps_z * n2;
        const T t2 = z_ok ? qdiv(sp, zz) : BIG;
        if (drop < 0 && !z_ok) { dead = true; break; }  // no step can restore the row
        const bool full = z_ok && (drop < 0 || t2 <= t1);
        const T t = full ? t2 : t1;
        if (full && pair && q == 2 * G) { status = 2; break; }
        if (z_ok) {
          ux -= t * zx;
          uy -= t * zy;
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (i + s * G < q) lam[i + s * G] -= t * g[s];
        wave_lds_fence();
        mux -= t * rfx;
        muy -= t * rfy;
        lam_p += t;
        if (full) {
          if (pair) {
            if (i == 0) {
              rows[q] = (Row){T(pa | pb << 8), cx, cy, T(0)};
              lam[q] = lam_p;
            }
            ++q;
            int owner, kk;
            pair_owner_g<G>(pa, pb, owner, kk);
            if (i == owner) own_act |= 1u << kk;
          } else if (i == pa) {
            // (cx, cy) is minus the normal: negative at an upper bound
            if (cx != T(0)) { fx = cx < T(0) ? 1 : -1; mux = lam_p; ux = cx < T(0) ? hix : lox; }
            else { fy = cy < T(0) ? 1 : -1; muy = lam_p; uy = cy < T(0) ? hiy : loy; }
          }
          added = true;
        } else if (drop >= 1024) {
          if (i == (drop - 1024) >> 1) {
            if (drop & 1) { fy = 0; muy = T(0); }
            else { fx = 0; mux = T(0); }
          }
        } else {
          const int id = (int)rows[drop].x;
          int owner, kk;
          pair_owner_g<G>(id & 255, id >> 8, owner, kk);
          if (i == owner) own_act &= ~(1u << kk);
          --q;
          if (i == 0 && drop != q) {  // the last row takes its place
            rows[drop] = rows[q];
            lam[drop] = lam[q];
          }
        }
        wave_lds_fence();
        if (++steps > cap) { status = 2; break; }
      }
    }
    if (dead) {
      status = 1;
      q = 0;
      if (on) {
        ux = tmin(tmax(uhx, lox), hix);
        uy = tmin(tmax(uhy, loy), hiy);
      }
    }
    wave_lds_fence();
    out = QPLoopOut<T>{ux, uy, status, out.iters + steps, q, 3};
  }
  __builtin_amdgcn_s_setprio(0);
  return out;
}

// Tail of the register loop for a wavefront in which some group needs the
// general solver; the others' results pass through.
// It has the register loop's signature (what a tail call needs here) and takes
// the result so far in uhx, uhy (command), i (in_lds, status and rows, a byte
// each) and fpa (iterations).
template <typename T, int G>
__device__ __noinline__ QPLoopOut<T> qp_general(LdsScratch<T, G> *sh, int lane, int packed, int N,
                                                bool on, T px, T py, T ux, T uy, T lox, T hix,
                                                T loy, T hiy, bool seed, int iters, int fpb, T fl1,
                                                T fdx, T fdy, T rs2, T gamma, T vmax4, T tol_add,
                                                T eps_z, T eps_r, int qp_cap, bool want_rows) {
  QPLoopOut<T> out;
  typename QPRow<T>::vec p{};
  const int run = packed & 255;
  if (run != 0) {
    out = QPLoopOut<T>{ux, uy, 0, iters, packed >> 16, run};
    qp_general_solve<T, G>(sh, lane, N, run == 2, out, rs2, gamma, vmax4, tol_add, eps_z, eps_r,
                           qp_cap, p);
  } else {
    out = QPLoopOut<T>{ux, uy, (packed >> 8) & 255, iters, packed >> 16, 0};
  }
  if (__ballot(out.in_lds == 3) != 0)  // wavefront-uniform: a tail call
    [[clang::musttail]] return qp_factored<T, G>(
        sh, lane, out.in_lds | out.status << 8 | out.q << 16, N, true, T(0), T(0), out.ux, out.uy,
        T(0), T(0), T(0), T(0), false, out.iters, (int)p.x, T(0), p.y, p.z, rs2, gamma, vmax4,
        tol_add, eps_z, eps_r, qp_cap, false);
  __builtin_amdgcn_s_setprio(0);
  return out;
}

// The active-set loop, kept out of line: it runs for the few environments the
// closed-form stages leave, and inlined its registers would weigh on every
// step. It rebuilds the pair geometry and the box clip from the arguments and
// starts from the box clip or, with `seed`, from the one-row solution of row
// (fpa, fpb) with multiplier fl1 (fdx, fdy = p_a - p_b). Every lane of the
// group calls it together. Only scalars cross the call. With want_rows the
// active rows and their multipliers are left in sh->row / sh->lam (as the
// general solver leaves them) for the caller to read.
template <typename T, int G>
__device__ __noinline__ QPLoopOut<T> qp_active_set(LdsScratch<T, G> *sh, int lane, int i, int N,
                                                   bool on, T px, T py, T uhx, T uhy, T lox,
                                                   T hix, T loy, T hiy, bool seed, int fpa,
                                                   int fpb, T fl1, T fdx, T fdy, T rs2, T gamma,
                                                   T vmax4, T tol_add, T eps_z, T eps_r,
                                                   int qp_cap, bool want_rows) {
  constexpr int KH = G / 2;
  const T BIG = big_v<T>();
  SimConst<T> C{};
  C.rs2 = rs2;
  C.gamma = gamma;
  C.vmax4 = vmax4;
  C.tol_add = tol_add;
  C.eps_z = eps_z;
  C.eps_r = eps_r;
  C.qp_cap = qp_cap;
  // the wavefronts in this loop are the slowest of a launch: give them the
  // first claim on issue slots over the other wavefront of their SIMD
  __builtin_amdgcn_s_setprio(1);
  QPInfo info{0, 0, 0, 0, kStBox};
  bool dead = false;
  T ux, uy;
  // --- geometry of the owned pairs ------------------------------------------
  T cdx[KH], cdy[KH], cb[KH], crn[KH];
  int cpid[KH];
  static_for<1, KH + 1>([&](auto kc) {
    constexpr int K = decltype(kc)::value;
    const T pxj = grot<G, K>(px, lane), pyj = grot<G, K>(py, lane);
    const int j = (i + K) & (G - 1);
    const bool valid = on && j < N && !(2 * K == G && i >= KH);
    const bool ia = i < j;
    const T dx = ia ? px - pxj : pxj - px;
    const T dy = ia ? py - pyj : pyj - py;
    const T d2 = dx * dx + dy * dy;
    const T h = d2 - C.rs2;
    const T bb = C.gamma * (h * h * h);
    const bool cand = valid && (C.vmax4 * (tabs(dx) + tabs(dy)) > bb);
    cdx[K - 1] = dx;
    cdy[K - 1] = dy;
    cb[K - 1] = bb;
    crn[K - 1] = d2 > T(0) ? T(0.35355339059327373) * rsqrt_t(d2) : T(0);
    cpid[K - 1] = (cand && d2 > T(0)) ? ((ia ? i : j) << 4 | (ia ? j : i)) : -1;
  });
  // the projection points are not needed again here: out of the registers
  sh->px[i] = px;
  sh->py[i] = py;
  // --- start: clip to the box; active bounds fix their coordinate ----------
  int fx = 0, fy = 0;
  T mux = T(0), muy = T(0);
  ux = uhx;
  uy = uhy;
  if (on) {
    if (uhx > hix) { ux = hix; fx = 1; mux = uhx - hix; }
    else if (uhx < lox) { ux = lox; fx = -1; mux = lox - uhx; }
    if (uhy > hiy) { uy = hiy; fy = 1; muy = uhy - hiy; }
    else if (uhy < loy) { uy = loy; fy = -1; muy = loy - uhy; }
  }

  const int cap = C.qp_cap > 0 ? C.qp_cap : 8 * N + 32;
  // Active pairwise rows: group-uniform slots (robots, multiplier) and, per
  // lane, the row's coefficients at the lane's robot (zero unless the robot is
  // one of the row's two ends). Gram entries and the products with the
  // entering row are then one butterfly sum each.
  int q = 0;
  int sa[kQR], sb[kQR];
  T slam[kQR], ccx[kQR], ccy[kQR];
  // Cholesky factor of the Gram system over the free coordinates, kept across
  // iterations: a row entering by a full step appends [w, |z|] (since
  // |z|^2 = c_p^T c_p - |L^-1 g|^2); any change of the free set or a dropped
  // row refactors.
  T L[kQR * (kQR + 1) / 2], Linv[kQR];
  bool lvalid = true;
#pragma unroll
  for (int a = 0; a < kQR; ++a) {
    sa[a] = sb[a] = -1;
    slam[a] = ccx[a] = ccy[a] = T(0);
    Linv[a] = T(0);
#pragma unroll
    for (int b = 0; b <= a; ++b) L[tri(a, b)] = T(0);
  }
  uint32_t own_act = 0;
  bool restart = false, carry = false;  // carry: restart from this state, p entering

  if (seed) {
    // row (fpa, fpb) active with multiplier fl1; its robots' coordinates are
    // free or clipped at that multiplier, and the clipped ones are fixed with
    // the bound multiplier that makes the point stationary
    q = 1;
    sa[0] = fpa;
    sb[0] = fpb;
    slam[0] = fl1;
    lvalid = false;
    info.iters = 1;
    int owner, kk;
    pair_owner_g<G>(fpa, fpb, owner, kk);
    if (i == owner) own_act |= 1u << kk;
    ccx[0] = i == fpa ? T(-2) * fdx : (i == fpb ? T(2) * fdx : T(0));
    ccy[0] = i == fpa ? T(-2) * fdy : (i == fpb ? T(2) * fdy : T(0));
    if (on && (i == fpa || i == fpb)) {
      const T vx = uhx - fl1 * ccx[0];
      const T vy = uhy - fl1 * ccy[0];
      ux = tclamp(vx, lox, hix);
      uy = tclamp(vy, loy, hiy);
      fx = vx > hix ? 1 : (vx < lox ? -1 : 0);
      mux = vx > hix ? vx - hix : (vx < lox ? lox - vx : T(0));
      fy = vy > hiy ? 1 : (vy < loy ? -1 : 0);
      muy = vy > hiy ? vy - hiy : (vy < loy ? loy - vy : T(0));
    }
  }
  const bool run_gi = true;

  // --- active-set loop ---------------------------------------------------------
  // One flat loop. Without a pending row an iteration picks the most violated
  // row p; with one it takes a step toward satisfying p: a full step makes p
  // active, a partial step releases the blocking active row or fixed bound.
  // Unused slots hold zero coefficients and identity rows of the factor, so
  // the slot algebra runs over all kQR slots as straight-line code.
  bool pend = false;
  bool p_pair = false;
  int pa = 0, pb = 0, pk = 0, psig = 0;
  T cpx = T(0), cpy = T(0), bp = T(0), lam_p = T(0);
#pragma unroll
  for (int a = 0; a < kQR; ++a) {
    if (a >= q) {
      L[tri(a, a)] = T(1);
      Linv[a] = T(1);
    }
  }
  bool go = run_gi && !dead;
  [[maybe_unused]] bool first = true;  // FP32: the first pick may take the caller's row
  while (go) {
    if constexpr (std::is_same<T, float>::value) {
      // FP32: the caller hands over the row its closed-form stages found most
      // violated at this start: with a seed, through the group's scratch
      // (H[0..3]: row id a << 4 | b, D = p_a - p_b, b); without one, the rows
      // of a rejected guess (or four or more rows violated at u0) start at
      // u0, where the row (fpa, fpb, fdx, fdy) is the most violated one, its
      // b from the same formula as the geometry above. It enters without a scan once its
      // violation here is confirmed; otherwise (or with no row handed over)
      // the first pick scans as usual.
      if (first) {
        first = false;
        int pid = fpa >= 0 ? (fpa << 4 | fpb) : -1;
        T rdx = fdx, rdy = fdy;
        const T rd2 = fdx * fdx + fdy * fdy;
        const T rh = rd2 - C.rs2;
        T rb = C.gamma * (rh * rh * rh);
        if (seed) {
          const floatx4 pr = *(const __attribute__((address_space(3))) floatx4 *)sh->H;
          pid = __float_as_int(pr.x);
          rdx = pr.y;
          rdy = pr.z;
          rb = pr.w;
        }
        const int ea = pid >> 4, eb = pid & 15;
        const T sgn = i == ea ? T(-2) : (i == eb ? T(2) : T(0));
        const T ex = on ? sgn * rdx : T(0), ey = on ? sgn * rdy : T(0);
        const T v0 = gsum<G>(ex * ux + ey * uy) - rb;
        if (pid >= 0 && v0 > T(0)) {
          if (++info.iters > cap) { info.status = 2; break; }
          p_pair = true;
          pa = ea;
          pb = eb;
          pk = 0;
          psig = 0;
          cpx = ex;
          cpy = ey;
          bp = rb;
          lam_p = T(0);
          pend = true;
        }
      }
    }
    if (!pend) {
      // --- most violated constraint (argmax carries the row's data) --------
      T best = C.tol_add, bdx = T(0), bdy = T(0), bbb = T(0);
      int bid = -1;
      if (on) {
        if (fx == 0) {
          const T su = ux - hix, sl = lox - ux;
          if (su > best) { best = su; bid = 256 + 4 * i; }
          else if (sl > best) { best = sl; bid = 256 + 4 * i + 1; }
        }
        if (fy == 0) {
          const T su = uy - hiy, sl = loy - uy;
          if (su > best) { best = su; bid = 256 + 4 * i + 2; }
          else if (sl > best) { best = sl; bid = 256 + 4 * i + 3; }
        }
      }
      static_for<1, KH + 1>([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        const T uxj = grot<G, K>(ux, lane), uyj = grot<G, K>(uy, lane);
        if (cpid[K - 1] >= 0 && !((own_act >> K) & 1u)) {
          const bool ia = i < ((i + K) & (G - 1));
          const T dux = ia ? uxj - ux : ux - uxj;
          const T duy = ia ? uyj - uy : uy - uyj;
          const T sn = (T(2) * (cdx[K - 1] * dux + cdy[K - 1] * duy) - cb[K - 1]) * crn[K - 1];
          if (sn > best) {
            best = sn;
            bid = cpid[K - 1];
            bdx = cdx[K - 1];
            bdy = cdy[K - 1];
            bbb = cb[K - 1];
          }
        }
      });
      gargmax_payload<G>(best, bid, bdx, bdy, bbb);
      if (bid < 0) break;  // optimal
      if (++info.iters > cap) { info.status = 2; break; }
      p_pair = bid < 256;
      pa = p_pair ? (bid >> 4) : ((bid - 256) >> 2);
      pb = p_pair ? (bid & 15) : -1;
      pk = p_pair ? 0 : (((bid - 256) >> 1) & 1);
      psig = p_pair ? 0 : (((bid - 256) & 1) ? -1 : 1);
      // entering row's coefficients at my robot
      const T sgn = i == pa ? T(-2) : (i == pb ? T(2) : T(0));
      cpx = p_pair ? sgn * bdx : ((i == pa && pk == 0) ? T(psig) : T(0));
      cpy = p_pair ? sgn * bdy : ((i == pa && pk == 1) ? T(psig) : T(0));
      if (!on) cpx = cpy = T(0);
      bp = bbb;
      lam_p = T(0);
      pend = true;
    }
    const bool frx = fx == 0, fry = fy == 0;
    // slots in use by some group of the wavefront: the algebra of the slots
    // beyond them (zero rows, identity rows of the factor) is skipped, which
    // leaves every group's values exactly as if it had run
    int qw = 0;
#pragma unroll
    for (int k = 1; k <= kQR; ++k) qw = __ballot(q >= k) ? k : qw;
    if (!lvalid) {
      // refactor the Gram system over the current free coordinates
      bool pd = true;
#pragma unroll
      for (int a = 0; a < kQR; ++a) {
        if (a < qw) {
#pragma unroll
          for (int b = 0; b <= a; ++b) {
            T sgm = gsum<G>((frx ? ccx[a] * ccx[b] : T(0)) + (fry ? ccy[a] * ccy[b] : T(0)));
#pragma unroll
            for (int k2 = 0; k2 < b; ++k2) sgm -= L[tri(a, k2)] * L[tri(b, k2)];
            if (b == a) {
              sgm = a < q ? sgm : T(1);
              pd = pd && (sgm > T(0));
              const T rs = rsqrt_t(tmax(sgm, T(1e-30)));
              L[tri(a, a)] = sgm * rs;
              Linv[a] = rs;
            } else {
              L[tri(a, b)] = sgm * Linv[b];
            }
          }
        } else {
#pragma unroll
          for (int b = 0; b < a; ++b) L[tri(a, b)] = T(0);
          L[tri(a, a)] = T(1);
          Linv[a] = T(1);
        }
      }
      if (!pd) { restart = true; break; }
      lvalid = true;
    }
    // g = C_S^free c_p, w = L^-1 g, r = L^-T w (zero on unused slots)
    T w[kQR], rv[kQR];
#pragma unroll
    for (int a = 0; a < kQR; ++a) {
      if (a < qw) {
        T g = gsum<G>((frx ? ccx[a] * cpx : T(0)) + (fry ? ccy[a] * cpy : T(0)));
#pragma unroll
        for (int k2 = 0; k2 < a; ++k2) g -= L[tri(a, k2)] * w[k2];
        w[a] = g * Linv[a];
      } else {
        w[a] = T(0);
      }
    }
#pragma unroll
    for (int a = kQR - 1; a >= 0; --a) {
      T sgm = w[a];
#pragma unroll
      for (int k2 = a + 1; k2 < kQR; ++k2) sgm -= L[tri(k2, a)] * rv[k2];
      rv[a] = sgm * Linv[a];
    }
    // C_S^T r at my robot, the primal direction z (free coordinates) and the
    // direction of my fixed bounds' multipliers
    T crx = T(0), cry = T(0);
#pragma unroll
    for (int a = 0; a < kQR; ++a) {
      crx += rv[a] * ccx[a];
      cry += rv[a] * ccy[a];
    }
    const T zx = frx ? cpx - crx : T(0);
    const T zy = fry ? cpy - cry : T(0);
    const T rfx = frx ? T(0) : T(fx) * (cpx - crx);
    const T rfy = fry ? T(0) : T(fy) * (cpy - cry);
    const T zz = gsum<G>(zx * zx + zy * zy);
    const T cpn2 = gsum<G>((frx ? cpx * cpx : T(0)) + (fry ? cpy * cpy : T(0)));
    // blocking step t1 over active rows (uniform) and my fixed bounds
    T t1 = BIG;
    int drop = -1;
#pragma unroll
    for (int a = 0; a < kQR; ++a) {
      const T ratio = qdiv(slam[a], rv[a]);
      const bool ok = a < q && rv[a] > C.eps_r && ratio < t1;
      t1 = ok ? ratio : t1;
      drop = ok ? a : drop;
    }
    {
      const T rx = qdiv(mux, rfx), ry = qdiv(muy, rfy);
      const bool okx = on && !frx && rfx > C.eps_r && (rx < t1 || (rx == t1 && drop < 0));
      t1 = okx ? rx : t1;
      drop = okx ? 1024 + 2 * i : drop;
      const bool oky = on && !fry && rfy > C.eps_r && (ry < t1 || (ry == t1 && drop < 0));
      t1 = oky ? ry : t1;
      drop = oky ? 1024 + 2 * i + 1 : drop;
    }
    gargmin<G>(t1, drop);
    // current violation of p
    T contrib = p_pair ? cpx * ux + cpy * uy : T(0);
    if (!p_pair && on && i == pa)
      contrib = pk ? (psig > 0 ? uy - hiy : loy - uy) : (psig > 0 ? ux - hix : lox - ux);
    const T sp = gsum<G>(contrib) - (p_pair ? bp : T(0));
    const bool z_ok = zz > C.eps_z * cpn2;
    const T t2 = z_ok ? qdiv(sp, zz) : BIG;
    if (drop < 0 && !z_ok) { dead = true; break; }
    const bool full = z_ok && (drop < 0 || t2 <= t1);
    const T t = full ? t2 : t1;
    if (full && p_pair && q == kQR) { restart = carry = true; break; }  // no slot left
    const T tz = z_ok ? t : T(0);
    ux -= tz * zx;
    uy -= tz * zy;
#pragma unroll
    for (int a = 0; a < kQR; ++a) slam[a] -= a < q ? t * rv[a] : T(0);
    mux -= t * rfx;
    muy -= t * rfy;
    lam_p += t;
    if (full && p_pair) {
      // append p at slot q and extend the factor: L[q] = [w, |z|]
      const T rz = rsqrt_t(zz);
#pragma unroll
      for (int a = 0; a < kQR; ++a) {
        const bool here = a == q;
        sa[a] = here ? pa : sa[a];
        sb[a] = here ? pb : sb[a];
        slam[a] = here ? lam_p : slam[a];
        ccx[a] = here ? cpx : ccx[a];
        ccy[a] = here ? cpy : ccy[a];
#pragma unroll
        for (int k2 = 0; k2 < a; ++k2) L[tri(a, k2)] = here ? w[k2] : L[tri(a, k2)];
        L[tri(a, a)] = here ? zz * rz : L[tri(a, a)];
        Linv[a] = here ? rz : Linv[a];
      }
      ++q;
      int owner, kk;
      pair_owner_g<G>(pa, pb, owner, kk);
      if (i == owner) own_act |= 1u << kk;
    } else if (full) {
      // p is a bound: fix the coordinate
      if (i == pa) {
        if (pk) { fy = psig; muy = lam_p; uy = psig > 0 ? hiy : loy; }
        else { fx = psig; mux = lam_p; ux = psig > 0 ? hix : lox; }
      }
      lvalid = false;
    } else if (drop >= 1024) {
      const int r = (drop - 1024) >> 1, cc2 = (drop - 1024) & 1;
      if (i == r) {
        if (cc2) { fy = 0; muy = T(0); } else { fx = 0; mux = T(0); }
      }
      lvalid = false;
    } else {
      // release active row `drop`: shift the later slots down
      int owner = 0, kk = 0;
#pragma unroll
      for (int a = 0; a < kQR; ++a)
        if (a == drop) pair_owner_g<G>(sa[a], sb[a], owner, kk);
      if (i == owner) own_act &= ~(1u << kk);
#pragma unroll
      for (int a = 0; a < kQR; ++a) {
        const bool mv = a >= drop && a + 1 < q;
        const bool clr = a >= drop && !mv;
        if (a + 1 < kQR) {
          sa[a] = mv ? sa[a + 1] : (clr ? -1 : sa[a]);
          sb[a] = mv ? sb[a + 1] : (clr ? -1 : sb[a]);
          slam[a] = mv ? slam[a + 1] : (clr ? T(0) : slam[a]);
          ccx[a] = mv ? ccx[a + 1] : (clr ? T(0) : ccx[a]);
          ccy[a] = mv ? ccy[a + 1] : (clr ? T(0) : ccy[a]);
        } else if (clr) {
          sa[a] = sb[a] = -1;
          slam[a] = ccx[a] = ccy[a] = T(0);
        }
      }
      --q;
      lvalid = false;
    }
    if (full) pend = false;
    if (++info.iters > cap) { info.status = 2; break; }
  }

  QPLoopOut<T> out;
  out.in_lds = 0;
  if (dead) {
    info.status = 1;
    q = 0;
    if (on) {
      ux = lox <= hix ? tmin(tmax(uhx, lox), hix) : T(0.5) * (lox + hix);
      uy = loy <= hiy ? tmin(tmax(uhy, loy), hiy) : T(0.5) * (loy + hiy);
    }
  } else if (restart) {
    // more active rows than register slots: the general solver carries on
    // from this active set; a degenerate Gram system: it starts from the clip
    typedef __attribute__((address_space(3))) T LdsT;
    out.in_lds = carry ? 2 : 1;
    LdsT *hv = handover<kHandover>(sh) + i;
    const T v[kHandover] = {uhx, uhy, lox, hix, loy, hiy, T(fx), T(fy), mux, muy};
#pragma unroll
    for (int c = 0; c < kHandover; ++c) hv[c * G] = v[c];
    if constexpr (G > 2) {
      if (carry) {
#pragma unroll
        for (int a = 0; a < kQR; ++a)
          if (i == sb[a])
            sh->row[a] = (typename QPRow<T>::vec){T(sa[a] | sb[a] << 8), ccx[a], ccy[a], slam[a]};
        if (i == pb) {
          sh->row[kQR] = (typename QPRow<T>::vec){T(pa | pb << 8), cpx, cpy, bp};
          *(LdsT *)(sh->row + kQR + 1) = lam_p;
        }
      }
    }
    wave_lds_fence();
  }
  out.ux = ux;
  out.uy = uy;
  out.status = info.status;
  out.iters = info.iters;
  out.q = q;
  if (want_rows && !out.in_lds) {
    if (i == 0) {
#pragma unroll
      for (int a = 0; a < kQR; ++a) {
        if (a < q) {
          sh->row[a].x = T(sa[a] | (sb[a] << 8));
          sh->lam[a] = slam[a];
        }
      }
    }
    wave_lds_fence();
  }
  if (__ballot(out.in_lds != 0) != 0)  // wavefront-uniform: a tail call
    [[clang::musttail]] return qp_general<T, G>(
        sh, lane, out.in_lds | out.status << 8 | out.q << 16, N, true, T(0), T(0), out.ux, out.uy,
        T(0), T(0), T(0), T(0), false, out.iters, 0, T(0), T(0), T(0), rs2, gamma, vmax4, tol_add,
        eps_z, eps_r, qp_cap, false);
  __builtin_amdgcn_s_setprio(0);
  return out;
}

template <typename T, int G, typename KT>
__device__ __forceinline__ QPInfo qp_solve(QPScratch<T, G> *sh, const KT &K, int qp_cap, int lane, int i, int N,
                           bool on, T px, T py, T uhx, T uhy, T lox, T hix, T loy, T hiy, T &ux,
                           T &uy, QPActive<T> *act_out = nullptr) {
  const auto &C = *K.get();  // the solver's constants, loaded for this phase
  constexpr int KH = G / 2;
  const T BIG = big_v<T>();
  QPInfo info{0, 0, 0, 0, kStBox};

  // --- box clip u0 (every bound holds there) ---------------------------------
  ux = uhx;
  uy = uhy;
  if (on) {
    ux = uhx > hix ? hix : (uhx < lox ? lox : uhx);
    uy = uhy > hiy ? hiy : (uhy < loy ? loy : uhy);
  }

  // --- geometry of the owned pairs and their violations at u0 ---------------
  // (the partner's position and command are fetched together)
  T cdx[KH], cdy[KH], cb[KH], crn[KH], snk[KH];
  int cpid[KH];
  bool coincide = false, viol = false;
  // FP32 8-lane groups take the partner's (p, u0) from one 16-byte LDS
  // exchange in the group's scratch (free here) instead of four DPP
  // rotations of two moves and a select each
  constexpr bool kLdsX = std::is_same<T, float>::value && G == 8;
  // the FP32 closed-form guesses beyond two rows (every group width alike, so
  // that results do not depend on the schedule)
  constexpr bool kGuess = std::is_same<T, float>::value;
  // A wavefront in which no row is violated at u0 leaves before the
  // normalisation, the row search and its exchanges. That is four steps of
  // five with one or two 8-robot envs per wavefront (FP64 steps of one
  // 4-robot env: 1.43 -> 1.21 us), but one of five with eight of them, where
  // the test costs what it saves (0.3% of the headline rollout).
  constexpr bool kEarly = !std::is_same<T, float>::value || G <= 4 ||
                          std::is_same<KT, ConstReg<T>>::value;
  float4 *xq = reinterpret_cast<float4 *>(sh);
  static_assert(!kGuess || sizeof(QPScratch<T, G>) >= G * (sizeof(float4) + 3 * sizeof(float2)),
                "the exchange fits in the group's scratch");
  if constexpr (kLdsX) {
    xq[i] = make_float4(px, py, ux, uy);
    wave_lds_fence();
  }
  static_for<1, KH + 1>([&](auto kc) {
    constexpr int K = decltype(kc)::value;
    T pxj, pyj, uxj, uyj;
    if constexpr (kLdsX) {
      const float4 v = xq[(i + K) & (G - 1)];
      pxj = v.x; pyj = v.y; uxj = v.z; uyj = v.w;
    } else {
      pxj = grot<G, K>(px, lane); pyj = grot<G, K>(py, lane);
      uxj = grot<G, K>(ux, lane); uyj = grot<G, K>(uy, lane);
    }
    const int j = (i + K) & (G - 1);
    const bool valid = on && j < N && !(2 * K == G && i >= KH);
    // D = p_i - p_j as this lane sees the pair. The row's own D runs from
    // its lower-index robot, which only flips the sign: the distance, the
    // pruning test and the violation do not see it, and it is applied when
    // the row is picked.
    const T dx = px - pxj, dy = py - pyj;
    const T d2 = dx * dx + dy * dy;
    const T h = d2 - C.rs2;
    const T bb = C.gamma * (h * h * h);
    const bool cand = valid && (C.vmax4 * (tabs(dx) + tabs(dy)) > bb);
    cdx[K - 1] = dx;
    cdy[K - 1] = dy;
    cb[K - 1] = bb;
    cpid[K - 1] = (cand && d2 > T(0)) ? (min(i, j) << 4 | max(i, j)) : -1;
    if (cand && !(d2 > T(0)) && bb < T(0)) coincide = true;
    // violation 2 D.(u_j - u_i) - b, to be taken over |c| = 2 sqrt(2) |D| (a
    // pair with D = 0 is no candidate: its value is never used)
    crn[K - 1] = kEarly ? d2 : T(0.35355339059327373) * rsqrt_t(d2);
    const T sv = T(2) * (dx * (uxj - ux) + dy * (uyj - uy)) - bb;
    snk[K - 1] = cpid[K - 1] >= 0 ? (kEarly ? sv : sv * crn[K - 1]) : -BIG;
    if constexpr (kEarly) viol = viol | (snk[K - 1] > T(0));
  });
  bool dead = group_any<G>(coincide || (on && (lox > hix || loy > hiy)), lane);

  // outcome of the closed-form stages: rows accepted (fq = 1 or 2), or a
  // one-row start for the active-set loop (seed)
  int fq = 0, fpa = -1, fpb = -1, fqa = -1, fqb = -1, fra = -1, frb = -1;
  T fl1 = T(0), fl2 = T(0), fl3 = T(0), fdx = T(0), fdy = T(0);
  bool seed = false;

  // --- closed-form stages --------------------------------------------------------
  // Every bound holds at the box clip u0. If at most two pairwise rows are
  // violated there, the solution is guessed in closed form and accepted when it
  // satisfies every row through the robots it moves (rows away from them keep
  // their values at u0, where only the guessed rows were violated): being the
  // minimiser over a superset of the feasible set, a feasible guess is the
  // solution.
  //  * One row p = (a, b), or two rows on four distinct robots: each row's
  //    projection onto box & {c.u <= b} is u(l) = clip(u_nom - l c), with
  //    l >= 0 the root of the non-increasing, piecewise linear
  //    phi(l) = c.u(l) - b; its breakpoints are where a coordinate of the
  //    row's two robots meets a bound.
  //  * Two rows through a shared robot: assuming no bound binds on the three
  //    robots, the multipliers solve the 2 x 2 Gram system; the guess also
  //    needs both multipliers >= 0 and the three commands inside their bounds.
  //  * FP32 only: after a rejected one-row guess, rows p and r (the row that
  //    guess violates) both active, or r alone when p's multiplier comes out
  //    negative; and for exactly three violated rows, all three active. Each
  //    solves its rows' Gram system with no bound binding and is accepted
  //    when the multipliers are >= 0, the moved robots stay inside their
  //    boxes and every other row holds: the KKT conditions of the QP.
  // A rejected one-row guess (with p active and the clipped coordinates fixed)
  // is a dual-feasible start for the active-set loop below; otherwise the loop
  // starts from u0.
  const bool some = !kEarly || __ballot(viol) != 0;
  bool run_gi = !dead && some;
  if (kEarly && some)
    static_for<1, KH + 1>([&](auto kc) {
      constexpr int K = decltype(kc)::value;
      crn[K - 1] = T(0.35355339059327373) * rsqrt_t(crn[K - 1]);
      snk[K - 1] = cpid[K - 1] >= 0 ? snk[K - 1] * crn[K - 1] : -BIG;
    });
  if (run_gi) {
    const T thr = C.tol_add;
    const int gbase = lane & ~(G - 1);
    T bdx = T(0), bdy = T(0), bbb = T(0);
    int bid = -1, nv = 0;
    if constexpr (kGuess) {
      // FP32: most violated row of the group by one integer key per row (the
      // score's float bits truncated by a byte, 255 - row id in the low byte:
      // a positive float orders like its bits), the maximum over the owned
      // rows, then over the group by one butterfly. The winner does not depend
      // on which lane owns which row, so it is the same for every group width.
      // Its D and b are recomputed from the two robots' projection points, by
      // the formulas of the scan (the same values the owner holds).
      uint32_t bkey = 0u;
      int nviol = 0;
      static_for<1, KH + 1>([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        const bool v = snk[K - 1] > thr;
        nviol += v ? 1 : 0;
        const uint32_t k =
            v ? ((__float_as_uint((float)snk[K - 1]) & 0xFFFFFF00u) | (uint32_t)(255 - cpid[K - 1]))
              : 0u;
        bkey = k > bkey ? k : bkey;
      });
      const int key =
          gred<G>((int)bkey, [](int a, int b) { return (uint32_t)a > (uint32_t)b ? a : b; });
      nv = gsum<G>(nviol);
      bid = key == 0 ? -1 : 255 - (key & 255);
      const int ra = bid < 0 ? 0 : bid >> 4, rb = bid < 0 ? 0 : bid & 15;
      T pax, pay, pbx, pby;
      if constexpr (kLdsX) {
        const float4 va = xq[ra], vb = xq[rb];
        pax = va.x; pay = va.y; pbx = vb.x; pby = vb.y;
      } else {
        pax = __shfl(px, gbase + ra, 64); pay = __shfl(py, gbase + ra, 64);
        pbx = __shfl(px, gbase + rb, 64); pby = __shfl(py, gbase + rb, 64);
      }
      bdx = pax - pbx;
      bdy = pay - pby;
      const T d2 = bdx * bdx + bdy * bdy;
      const T h = d2 - C.rs2;
      bbb = C.gamma * (h * h * h);
    } else {
      T best = thr;
      int nviol = 0;
      static_for<1, KH + 1>([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        nviol += snk[K - 1] > thr ? 1 : 0;
        if (snk[K - 1] > best) {
          best = snk[K - 1];
          bid = cpid[K - 1];
          bdx = cdx[K - 1];
          bdy = cdy[K - 1];
          bbb = cb[K - 1];
        }
      });
      // most violated row of the group: winner lane by one integer
      // butterfly, its row's data read from that lane
      const int wl = group_argmax_lane<G>(best, bid >= 0, i);
      nv = gsum<G>(nviol);
      const int src = gbase + (wl < 0 ? 0 : wl);
      bid = wl < 0 ? -1 : __shfl(bid, src, 64);
      bdx = __shfl(bdx, src, 64);
      bdy = __shfl(bdy, src, 64);
      bbb = __shfl(bbb, src, 64);
      // orient D from the row's lower-index robot (the owner is either end)
      const bool flip = wl != (bid >> 4);
      bdx = flip ? -bdx : bdx;
      bdy = flip ? -bdy : bdy;
    }
    if (bid < 0) {
      run_gi = false;  // u0 is the solution
    } else if (nv == 3 && kGuess) {
      if constexpr (kGuess) {
        // Three rows violated at u0 (FP32): guess all three
        // active with no bound binding, from their 3 x 3 Gram system, and
        // accept as the two-row stages do; otherwise the loop starts from u0.
        T sx[2] = {T(0), T(0)}, sy[2] = {T(0), T(0)}, sb[2] = {T(0), T(0)};
        int sid[2] = {-1, -1};
        static_for<0, 2>([&](auto rc) {
          constexpr int R = decltype(rc)::value;
          T b2 = thr, e2x = T(0), e2y = T(0), beta2 = T(0);
          int id2 = -1;
          static_for<1, KH + 1>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            const int id = cpid[K - 1];
            const bool taken = id == bid || (R == 1 && id == sid[0]);
            if (!taken && snk[K - 1] > b2) {
              b2 = snk[K - 1];
              id2 = id;
              e2x = cdx[K - 1];
              e2y = cdy[K - 1];
              beta2 = cb[K - 1];
            }
          });
          const int w2 = group_argmax_lane<G>(b2, id2 >= 0, i);
          const int src = gbase + (w2 < 0 ? 0 : w2);
          id2 = w2 < 0 ? -1 : __shfl(id2, src, 64);
          e2x = __shfl(e2x, src, 64);
          e2y = __shfl(e2y, src, 64);
          beta2 = __shfl(beta2, src, 64);
          const bool flip2 = w2 != (id2 >> 4);
          sx[R] = flip2 ? -e2x : e2x;
          sy[R] = flip2 ? -e2y : e2y;
          sb[R] = beta2;
          sid[R] = id2;
        });
        const int pa = bid >> 4, pb = bid & 15;
        const int qa = sid[0] >> 4, qb = sid[0] & 15, ra = sid[1] >> 4, rb = sid[1] & 15;
        const bool all3 = sid[0] >= 0 && sid[1] >= 0;
        auto coef = [&](int a, int b, T dx, T dy, T &cx, T &cy) {
          cx = i == a ? T(-2) * dx : (i == b ? T(2) * dx : T(0));
          cy = i == a ? T(-2) * dy : (i == b ? T(2) * dy : T(0));
        };
        T c1x, c1y, c2x, c2y, c3x, c3y;
        coef(pa, pb, bdx, bdy, c1x, c1y);
        coef(qa, qb, sx[0], sy[0], c2x, c2y);
        coef(ra, rb, sx[1], sy[1], c3x, c3y);
        const T g11 = T(8) * (bdx * bdx + bdy * bdy);
        const T g22 = T(8) * (sx[0] * sx[0] + sy[0] * sy[0]);
        const T g33 = T(8) * (sx[1] * sx[1] + sy[1] * sy[1]);
        const T g12 = gsum<G>(c1x * c2x + c1y * c2y);
        const T g13 = gsum<G>(c1x * c3x + c1y * c3y);
        const T g23 = gsum<G>(c2x * c3x + c2y * c3y);
        const T h1 = gsum<G>(c1x * uhx + c1y * uhy) - bbb;
        const T h2 = gsum<G>(c2x * uhx + c2y * uhy) - sb[0];
        const T h3 = gsum<G>(c3x * uhx + c3y * uhy) - sb[1];
        // Cramer's rule on the symmetric 3 x 3 system
        const T m11 = g22 * g33 - g23 * g23, m12 = g12 * g33 - g23 * g13, m13 = g12 * g23 - g22 * g13;
        const T det = g11 * m11 - g12 * m12 + g13 * m13;
        const T idet = qdiv(T(1), det);
        const T l1 = (h1 * m11 - g12 * (h2 * g33 - g23 * h3) + g13 * (h2 * g23 - g22 * h3)) * idet;
        const T l2 = (g11 * (h2 * g33 - g23 * h3) - h1 * m12 + g13 * (g12 * h3 - h2 * g13)) * idet;
        const T l3 = (g11 * (g22 * h3 - h2 * g23) - g12 * (g12 * h3 - h2 * g13) + h1 * m13) * idet;
        bool ok3 = all3 && det > T(1e-6) * g11 * g22 * g33 && l1 >= T(0) && l2 >= T(0) && l3 >= T(0);
        const bool mv = i == pa || i == pb || i == qa || i == qb || i == ra || i == rb;
        const T vx = uhx - l1 * c1x - l2 * c2x - l3 * c3x;
        const T vy = uhy - l1 * c1y - l2 * c2y - l3 * c3y;
        const bool outb = on && mv && (vx < lox || vx > hix || vy < loy || vy > hiy);
        ok3 = ok3 && !group_any<G>(outb, lane);
        const T wx = (on && mv) ? vx : ux, wy = (on && mv) ? vy : uy;  // unmoved: u0
        float2 *xw = reinterpret_cast<float2 *>(sh) + 2 * G;
        xw[i] = make_float2(wx, wy);
        wave_lds_fence();
        bool bad3 = !ok3;
        static_for<1, KH + 1>([&](auto kc) {
          constexpr int K = decltype(kc)::value;
          const float2 v = xw[(i + K) & (G - 1)];
          const int id = cpid[K - 1];
          const T sn = (T(2) * (cdx[K - 1] * (v.x - wx) + cdy[K - 1] * (v.y - wy)) - cb[K - 1]) *
                       crn[K - 1];
          bad3 = bad3 | ((id >= 0) & (id != bid) & (id != sid[0]) & (id != sid[1]) &
                         (sn > C.tol_add));
        });
        const bool accept3 = !group_any<G>(bad3, lane);
        if (accept3) {
          ux = wx;
          uy = wy;
          fq = 3;
          fpa = pa; fpb = pb; fl1 = l1;
          fqa = qa; fqb = qb; fl2 = l2;
          fra = ra; frb = rb; fl3 = l3;
          info.stage = kStShared;
          info.iters = 3;
          run_gi = false;
        } else {
          // the loop starts at u0, where p is the most violated row
          fpa = pa; fpb = pb; fdx = bdx; fdy = bdy;
        }
      }
    } else if (nv <= 2) {
      // the other violated row, if any
      T b2 = thr, e2x = T(0), e2y = T(0), beta2 = T(0);
      int id2 = -1;
      if (nv == 2) {
        static_for<1, KH + 1>([&](auto kc) {
          constexpr int K = decltype(kc)::value;
          if (cpid[K - 1] != bid && snk[K - 1] > b2) {
            b2 = snk[K - 1];
            id2 = cpid[K - 1];
            e2x = cdx[K - 1];
            e2y = cdy[K - 1];
            beta2 = cb[K - 1];
          }
        });
        const int w2 = group_argmax_lane<G>(b2, id2 >= 0, i);
        const int src = gbase + (w2 < 0 ? 0 : w2);
        id2 = w2 < 0 ? -1 : __shfl(id2, src, 64);
        e2x = __shfl(e2x, src, 64);
        e2y = __shfl(e2y, src, 64);
        beta2 = __shfl(beta2, src, 64);
        const bool flip2 = w2 != (id2 >> 4);
        e2x = flip2 ? -e2x : e2x;
        e2y = flip2 ? -e2y : e2y;
      }
      const bool two = nv == 2 && id2 >= 0;
      const int pa = bid >> 4, pb = bid & 15;
      const int qa = two ? id2 >> 4 : pa, qb = two ? id2 & 15 : pb;
      const bool shared = two && (qa == pa || qa == pb || qb == pa || qb == pb);
      bool ok = true;
      T lam1 = T(0), lam2 = T(0);
      T nux = ux, nuy = uy;  // my command under the guess (u0 unless I move)
      // projection onto box & one half-space for each row, on its own two
      // robots; rows one after the other (a true loop keeps the registers of
      // one row) with a trip count uniform over the wavefront
      const int trips = __ballot(two && !shared) ? 2 : 1;
#pragma unroll 1
      for (int rr = 0; rr < trips; ++rr) {
        const bool r2 = rr == 1;
        const bool use = !shared && (!r2 || two);  // this group solves this row
        const int ra = r2 ? qa : pa, rb = r2 ? qb : pb;
        const T dx = r2 ? e2x : bdx, dy = r2 ? e2y : bdy;
        const T beta = r2 ? beta2 : bbb;
        // projection onto the row's hyperplane with every coordinate free: the
        // row's solution whenever it lands inside the box of both its robots
        // (each group takes it then, whatever the other groups need)
        const T cix = i == ra ? T(-2) * dx : (i == rb ? T(2) * dx : T(0));
        const T ciy = i == ra ? T(-2) * dy : (i == rb ? T(2) * dy : T(0));
        const T lamf = (gsum<G>(cix * uhx + ciy * uhy) - beta) * qdiv(T(1), T(8) * (dx * dx + dy * dy));
        const T fvx = uhx - lamf * cix, fvy = uhy - lamf * ciy;
        const bool end_ab = use && (i == ra || i == rb);
        const bool fbad = end_ab && (fvx < lox || fvx > hix || fvy < loy || fvy > hiy);
        const bool free_ok = use && lamf > T(0) && !group_any<G>(fbad, lane);
        if (__ballot(use && !free_ok) == 0) {  // every row of the wave: the free solution
          nux = end_ab ? fvx : nux;
          nuy = end_ab ? fvy : nuy;
          lam2 = r2 ? lamf : lam2;
          lam1 = r2 ? lam1 : lamf;
          continue;
        }
        const int la = gbase + ra, lb = gbase + rb;
        const T cc[4] = {T(-2) * dx, T(-2) * dy, T(2) * dx, T(2) * dy};
        const T un[4] = {__shfl(uhx, la, 64), __shfl(uhy, la, 64), __shfl(uhx, lb, 64),
                         __shfl(uhy, lb, 64)};
        const T lo[4] = {__shfl(lox, la, 64), __shfl(loy, la, 64), __shfl(lox, lb, 64),
                         __shfl(loy, lb, 64)};
        const T hi[4] = {__shfl(hix, la, 64), __shfl(hiy, la, 64), __shfl(hix, lb, 64),
                         __shfl(hiy, lb, 64)};
        auto phi = [&](T lm) {
          T acc = -beta;
#pragma unroll
          for (int k = 0; k < 4; ++k) acc += cc[k] * tclamp(un[k] - lm * cc[k], lo[k], hi[k]);
          return acc;
        };
        // the root lies between the largest breakpoint (or 0) where phi is
        // still positive, (llo, plo), and the smallest one where it is not,
        // (lhi, phi_hi): no breakpoint falls in between, so phi is linear
        // there. The eight breakpoints are shared out over the group's lanes
        // and both ends found by one butterfly (equal breakpoints give equal
        // phi). No breakpoint with phi <= 0: the row cannot be met in the box.
        T llo = T(0), plo = phi(T(0));
        T lhi = BIG, phh = T(0);
        {
          T bl = T(-1), bv = T(0);
          for (int b = i; b < 8; b += G) {
            // breakpoint b: the multiplier where coordinate k = b / 2 meets
            // its upper (b even) or lower (b odd) bound; a coordinate the row
            // does not move gives 0
            const int k = b >> 1;
            auto pick = [&](const T *v) {
              const T lo2 = (k & 1) ? v[1] : v[0], hi2 = (k & 1) ? v[3] : v[2];
              return (k & 2) ? hi2 : lo2;
            };
            const T ck = pick(cc), uk = pick(un), bk = (b & 1) ? pick(lo) : pick(hi);
            const T ek = ck != T(0) ? (uk - bk) * qdiv(T(1), ck) : T(0);
            const T pk = phi(ek);
            const bool pos = pk > T(0);
            const bool better = pos & (ek > bl);
            bl = better ? ek : bl;
            bv = better ? pk : bv;
            const bool upper = !pos & (ek < lhi);
            lhi = upper ? ek : lhi;
            phh = upper ? pk : phh;
          }
          auto merge = [&](auto c) {
            constexpr int CT = decltype(c)::value;
            const T w = dpp<CT>(bl), q = dpp<CT>(bv);
            const bool better = w > bl;
            bl = better ? w : bl;
            bv = better ? q : bv;
            const T wu = dpp<CT>(lhi), qu = dpp<CT>(phh);
            const bool lower = wu < lhi;
            lhi = lower ? wu : lhi;
            phh = lower ? qu : phh;
          };
          merge(std::integral_constant<int, 0xB1>{});
          if constexpr (G >= 4) merge(std::integral_constant<int, 0x4E>{});
          if constexpr (G >= 8) merge(std::integral_constant<int, 0x141>{});
          if constexpr (G >= 16) merge(std::integral_constant<int, 0x140>{});
          plo = bl > llo ? bv : plo;
          llo = bl > llo ? bl : llo;
        }
        ok = ok && (!use || free_ok || lhi < BIG);
        const T lam = free_ok ? lamf : llo + plo * (tmin(lhi, BIG) - llo) * qdiv(T(1), plo - phh);
        const bool ma = use && i == ra, mb = use && i == rb;
        const T ax = tclamp(un[0] - lam * cc[0], lo[0], hi[0]);
        const T ay = tclamp(un[1] - lam * cc[1], lo[1], hi[1]);
        const T bx = tclamp(un[2] - lam * cc[2], lo[2], hi[2]);
        const T by = tclamp(un[3] - lam * cc[3], lo[3], hi[3]);
        nux = free_ok ? (end_ab ? fvx : nux) : (ma ? ax : (mb ? bx : nux));
        nuy = free_ok ? (end_ab ? fvy : nuy) : (ma ? ay : (mb ? by : nuy));
        lam2 = r2 ? lam : lam2;
        lam1 = r2 ? lam1 : lam;
      }
      if (shared) {
        // two rows through a shared robot r; j is p2's other end. With no
        // bound binding on a, b, j: u = u_nom - lam1 c1 - lam2 c2 there.
        const T c1x = i == pa ? T(-2) * bdx : (i == pb ? T(2) * bdx : T(0));
        const T c1y = i == pa ? T(-2) * bdy : (i == pb ? T(2) * bdy : T(0));
        const T c2x = i == qa ? T(-2) * e2x : (i == qb ? T(2) * e2x : T(0));
        const T c2y = i == qa ? T(-2) * e2y : (i == qb ? T(2) * e2y : T(0));
        const T g11 = T(8) * (bdx * bdx + bdy * bdy);
        const T g22 = T(8) * (e2x * e2x + e2y * e2y);
        const T g12 = gsum<G>(c1x * c2x + c1y * c2y);
        const T h1 = gsum<G>(c1x * uhx + c1y * uhy) - bbb;
        const T h2 = gsum<G>(c2x * uhx + c2y * uhy) - beta2;
        const T det = g11 * g22 - g12 * g12;
        const T idet = qdiv(T(1), det);
        lam1 = (g22 * h1 - g12 * h2) * idet;
        lam2 = (g11 * h2 - g12 * h1) * idet;
        ok = det > T(1e-6) * g11 * g22 && lam1 >= T(0) && lam2 >= T(0);
        const bool mv = i == pa || i == pb || i == qa || i == qb;
        const T vx = uhx - lam1 * c1x - lam2 * c2x;
        const T vy = uhy - lam1 * c1y - lam2 * c2y;
        nux = mv ? vx : nux;
        nuy = mv ? vy : nuy;
        const bool out = mv && (vx < lox || vx > hix || vy < loy || vy > hiy);
        ok = ok && !group_any<G>(out, lane);
      }
      // check every candidate row at the guess, except the guessed ones, from
      // the geometry of the scan: a row with both ends unmoved keeps its value
      // at u0 (below the threshold), and a pruned row holds anywhere in the
      // speed box, which contains every guess
      bool bad = !ok;
      float2 *xv = reinterpret_cast<float2 *>(sh) + 2 * G;  // past the scan's exchange
      if constexpr (kLdsX) {
        xv[i] = make_float2(nux, nuy);
        wave_lds_fence();
      }
      static_for<1, KH + 1>([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        T uxj, uyj;
        if constexpr (kLdsX) {
          const float2 v = xv[(i + K) & (G - 1)];
          uxj = v.x; uyj = v.y;
        } else {
          uxj = grot<G, K>(nux, lane); uyj = grot<G, K>(nuy, lane);
        }
        const int id = cpid[K - 1];
        const bool guessed = (id == bid) | (two & (id == id2));
        const T sn = (T(2) * (cdx[K - 1] * (uxj - nux) + cdy[K - 1] * (uyj - nuy)) - cb[K - 1]) *
                     crn[K - 1];
        bad = bad | ((id >= 0) & !guessed & (sn > C.tol_add));
      });
      bool accept = !group_any<G>(bad, lane);
      bool seeded = !accept && !two && ok;
      bool second = false;  // accepted on the second guess below
      bool lone = false;    // accepted with the violated row alone
      int sqa = qa, sqb = qb, spa = pa, spb = pb;
      if constexpr (kGuess) {
        // A rejected one-row guess violates some row r, which shares a robot
        // with p (only p's robots moved). Second guess: p and r both active
        // with no bound binding, from their 2 x 2 Gram system, accepted by
        // the checks of the shared-robot stage (wave-uniform branch: only
        // wavefronts with such a group pay for it). The guess's commands go
        // through the group's LDS exchange (xv).
        if (__ballot(seeded) != 0) {
          if constexpr (!kLdsX) {  // the guess's commands into the exchange
            xv[i] = make_float2(nux, nuy);
            wave_lds_fence();
          }
          T rbest = C.tol_add, rdx = T(0), rdy = T(0), rbb = T(0);
          int rid = -1;
          static_for<1, KH + 1>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            const float2 v = xv[(i + K) & (G - 1)];
            const int id = cpid[K - 1];
            const T sn = (T(2) * (cdx[K - 1] * (v.x - nux) + cdy[K - 1] * (v.y - nuy)) - cb[K - 1]) *
                         crn[K - 1];
            if (seeded && id >= 0 && id != bid && sn > rbest) {
              rbest = sn;
              rid = id;
              rdx = cdx[K - 1];
              rdy = cdy[K - 1];
              rbb = cb[K - 1];
            }
          });
          const int wr = group_argmax_lane<G>(rbest, rid >= 0, i);
          const int src = gbase + (wr < 0 ? 0 : wr);
          rid = wr < 0 ? -1 : __shfl(rid, src, 64);
          rdx = __shfl(rdx, src, 64);
          rdy = __shfl(rdy, src, 64);
          rbb = __shfl(rbb, src, 64);
          const bool flipr = wr != (rid >> 4);
          rdx = flipr ? -rdx : rdx;
          rdy = flipr ? -rdy : rdy;
          // a seeded loop starts at this guess, where r is the most violated
          // row: handed over through the group's scratch (H[0..3])
          if (seeded && i == 0)
            *reinterpret_cast<floatx4 *>(sh->H) = (floatx4){__int_as_float(rid), rdx, rdy, rbb};
          const int ra = rid >> 4, rb = rid & 15;
          const bool try2 =
              seeded && rid >= 0 && (ra == pa || ra == pb || rb == pa || rb == pb);
          const T c1x = i == pa ? T(-2) * bdx : (i == pb ? T(2) * bdx : T(0));
          const T c1y = i == pa ? T(-2) * bdy : (i == pb ? T(2) * bdy : T(0));
          const T c2x = i == ra ? T(-2) * rdx : (i == rb ? T(2) * rdx : T(0));
          const T c2y = i == ra ? T(-2) * rdy : (i == rb ? T(2) * rdy : T(0));
          const T g11 = T(8) * (bdx * bdx + bdy * bdy);
          const T g22 = T(8) * (rdx * rdx + rdy * rdy);
          const T g12 = gsum<G>(c1x * c2x + c1y * c2y);
          const T h1 = gsum<G>(c1x * uhx + c1y * uhy) - bbb;
          const T h2 = gsum<G>(c2x * uhx + c2y * uhy) - rbb;
          const T det = g11 * g22 - g12 * g12;
          const T idet = qdiv(T(1), det);
          const T m1 = (g22 * h1 - g12 * h2) * idet;
          const T m2 = (g11 * h2 - g12 * h1) * idet;
          bool ok2 = try2 && det > T(1e-6) * g11 * g22 && m1 >= T(0) && m2 >= T(0);
          const bool mv = i == pa || i == pb || i == ra || i == rb;
          const T vx = uhx - m1 * c1x - m2 * c2x;
          const T vy = uhy - m1 * c1y - m2 * c2y;
          const bool outb = on && mv && (vx < lox || vx > hix || vy < loy || vy > hiy);
          ok2 = ok2 && !group_any<G>(outb, lane);
          const T wx = (on && mv) ? vx : ux, wy = (on && mv) ? vy : uy;  // unmoved: u0
          float2 *xw = xv + G;  // past the guess's exchange
          xw[i] = make_float2(wx, wy);
          wave_lds_fence();
          bool bad2 = !ok2;
          static_for<1, KH + 1>([&](auto kc) {
            constexpr int K = decltype(kc)::value;
            const float2 v = xw[(i + K) & (G - 1)];
            const int id = cpid[K - 1];
            const T sn = (T(2) * (cdx[K - 1] * (v.x - wx) + cdy[K - 1] * (v.y - wy)) - cb[K - 1]) *
                         crn[K - 1];
            bad2 = bad2 | ((id >= 0) & (id != bid) & (id != rid) & (sn > C.tol_add));
          });
          second = try2 && !group_any<G>(bad2, lane);
          if (second) {
            nux = wx;
            nuy = wy;
            lam1 = m1;
            lam2 = m2;
            sqa = ra;
            sqb = rb;
            accept = true;
            seeded = false;
          }
          // p's multiplier came out negative: r alone, projected with every
          // coordinate free, p then checked like every other row
          const bool try3 = try2 && !second && m1 < T(0);
          if (__ballot(try3) != 0) {
            const T lr = qdiv(h2, g22);
            const bool mv3 = i == ra || i == rb;
            const T v3x = uhx - lr * c2x, v3y = uhy - lr * c2y;
            const bool outb3 = on && mv3 && (v3x < lox || v3x > hix || v3y < loy || v3y > hiy);
            const bool ok3 = try3 && lr > T(0) && !group_any<G>(outb3, lane);
            const T w3x = (on && mv3) ? v3x : ux, w3y = (on && mv3) ? v3y : uy;
            float2 *x3 = xw + G;  // past the second guess's exchange
            x3[i] = make_float2(w3x, w3y);
            wave_lds_fence();
            bool bad3 = !ok3;
            static_for<1, KH + 1>([&](auto kc) {
              constexpr int K = decltype(kc)::value;
              const float2 v = x3[(i + K) & (G - 1)];
              const int id = cpid[K - 1];
              const T sn = (T(2) * (cdx[K - 1] * (v.x - w3x) + cdy[K - 1] * (v.y - w3y)) - cb[K - 1]) *
                           crn[K - 1];
              bad3 = bad3 | ((id >= 0) & (id != rid) & (sn > C.tol_add));
            });
            lone = try3 && !group_any<G>(bad3, lane);
            if (lone) {
              nux = w3x;
              nuy = w3y;
              lam1 = lr;
              spa = ra;
              spb = rb;
              accept = true;
              seeded = false;
            }
          }
        }
      }
      // accepted: the guess is the solution; one rejected row with ok: start
      // the loop from u(l) with p active; otherwise from u0 (unchanged)
      ux = (accept || seeded) ? nux : ux;
      uy = (accept || seeded) ? nuy : uy;
      fq = accept ? ((two || second) ? 2 : 1) : fq;
      info.stage = (two || second) ? ((shared || second) ? kStShared : kStTwoRows) : kStOneRow;
      seed = seeded;
      fpa = spa; fpb = spb; fl1 = lam1; fdx = bdx; fdy = bdy;
      fqa = sqa; fqb = sqb; fl2 = lam2;
      run_gi = !accept;
      info.iters = (two || second) ? 2 : 1;
    } else {
      if constexpr (kGuess) {
        // four or more rows violated at u0, where the loop starts: p is the
        // most violated one
        fpa = bid >> 4; fpb = bid & 15; fdx = bdx; fdy = bdy;
      }
    }
  }

  if (__builtin_expect(run_gi, 0)) {
    const QPLoopOut<T> r = qp_active_set<T, G>((LdsScratch<T, G> *)sh, lane, i, N, on, px, py, uhx, uhy, lox, hix,
                                               loy, hiy, seed, fpa, fpb, fl1, fdx, fdy, C.rs2,
                                               C.gamma, C.vmax4, C.tol_add, C.eps_z, C.eps_r,
                                               qp_cap, act_out != nullptr);
    ux = r.ux;
    uy = r.uy;
    info.status = r.status;
    info.iters = r.iters;
    info.q = r.q;
    info.in_lds = r.in_lds;
    info.stage = r.in_lds ? kStGeneral : kStActiveSet;
    if (act_out) {
      act_out->q = r.q;
      act_out->rows_in_lds = 1;
    }
    return info;
  }
  if (dead) {
    info.status = 1;
    info.stage = kStBox;
    fq = 0;
    if (on) {
      ux = lox <= hix ? tmin(tmax(uhx, lox), hix) : T(0.5) * (lox + hix);
      uy = loy <= hiy ? tmin(tmax(uhy, loy), hiy) : T(0.5) * (loy + hiy);
    }
  }
  info.q = fq;
  if (act_out) {
    act_out->q = fq;
    act_out->rows_in_lds = 0;
    act_out->sa[0] = fq > 0 ? fpa : -1;
    act_out->sb[0] = fq > 0 ? fpb : -1;
    act_out->slam[0] = fq > 0 ? fl1 : T(0);
    act_out->sa[1] = fq > 1 ? fqa : -1;
    act_out->sb[1] = fq > 1 ? fqb : -1;
    act_out->slam[1] = fq > 1 ? fl2 : T(0);
    act_out->sa[2] = fq > 2 ? fra : -1;
    act_out->sb[2] = fq > 2 ? frb : -1;
    act_out->slam[2] = fq > 2 ? fl3 : T(0);
#pragma unroll
    for (int a = 3; a < kQR; ++a) {
      act_out->sa[a] = -1;
      act_out->sb[a] = -1;
      act_out->slam[a] = T(0);
    }
  }
  return info;
}

}  // namespace rs
